// Chunk table of packed variable-length calls (App. C.6): every sequence of a
// packed batch is cut into chunks of its own (C = 64 tokens, the last one
// partial), so that the state restarts at each sequence boundary.  One
// 1024-thread workgroup: 1024 sequences at a time, a scan of their chunk counts
// gives coff, and every chunk slot of theirs finds its sequence by bisection in
// LDS; a counting sort orders the sequences longest first for the scans.
//
// The kernel stands between the caller and the first chunk kernel and is all
// latency: what counts is its chain of dependent steps.  The scans are wave
// shuffles with one exchange of the 16 wave totals; a serial pass over the
// sort's 4096 bins and a thread per sequence writing all its chunks took 36 us
// for 9 sequences (38 for 30), this 4.7 (5.7).

#include "gdr2_kernels.hpp"

namespace gdr2 {

// Inclusive sum over the 1024 threads; wt: 16 words of LDS.  All threads call it.
__device__ __forceinline__ int scan1024(int x, int* wt, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wt[wave] = x;
  __syncthreads();
  int off = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) off += i < wave ? wt[i] : 0;
  __syncthreads();
  return x + off;
}

__global__ __launch_bounds__(1024) void varlen_table_kernel(const int* cu, int nseq, int T, int ncmax, int* coff,
                                                            int* ct0, int* clen, int* sorder) {
  constexpr int NTHR = 1024;
  constexpr int NBIN = 4096;  // chunk counts >= NBIN - 1 share the first bin
  __shared__ int wt[NTHR / 64];
  __shared__ int sEnd[NTHR], sT0[NTHR], sT1[NTHR];  // of this pass's sequences: chunks up to their end, tokens
  __shared__ int hist[NBIN];
  const int tid = threadIdx.x;
  for (int i = tid; i < NBIN; i += NTHR) hist[i] = 0;
  // tokens [t0, t1) of sequence s, clamped into [0, T]; its chunk count
  const auto tokens = [&](int s, int& t0, int& t1) {
    t0 = min(max(cu[s], 0), T);
    t1 = min(max(cu[s + 1], t0), T);
    return (t1 - t0 + CH - 1) / CH;
  };
  const auto bin_of = [&](int n) { return NBIN - 1 - min(n, NBIN - 1); };
  __syncthreads();
  int carry = 0;  // chunks before this pass's sequences (clamped to ncmax), the same in every thread
  for (int base = 0; base < nseq; base += NTHR) {
    const int s = base + tid;
    int n = 0, t0 = 0, t1 = 0;
    if (s < nseq) {
      n = tokens(s, t0, t1);
      atomicAdd(&hist[bin_of(n)], 1);
    }
    const int end = min(carry + scan1024(n, wt, tid), ncmax);
    sEnd[tid] = end;
    sT0[tid] = t0;
    sT1[tid] = t1;
    __syncthreads();
    if (s < nseq) coff[s] = tid > 0 ? sEnd[tid - 1] : carry;
    const int last = sEnd[NTHR - 1];
    for (int c = carry + tid; c < last; c += NTHR) {
      int lo = 0, hi = NTHR - 1;  // the first sequence whose end lies behind chunk c
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (sEnd[mid] > c)
          hi = mid;
        else
          lo = mid + 1;
      }
      const int t = sT0[lo] + (c - (lo > 0 ? sEnd[lo - 1] : carry)) * CH;
      ct0[c] = t;
      clen[c] = min(CH, sT1[lo] - t);
    }
    carry = last;
    __syncthreads();
  }
  if (tid == 0) coff[nseq] = carry;
  // scan order: counting sort by decreasing chunk count (bin NBIN-1-count);
  // the order within a bin is whatever the LDS atomics give -- it only decides
  // when a scan starts, never what it computes
  {
    constexpr int PER = NBIN / NTHR;
    int x[PER], run = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      x[i] = hist[PER * tid + i];
      run += x[i];
    }
    int before = scan1024(run, wt, tid) - run;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      hist[PER * tid + i] = before;
      before += x[i];
    }
  }
  __syncthreads();
  for (int s = tid; s < nseq; s += NTHR) {
    int t0, t1;
    const int n = tokens(s, t0, t1);
    sorder[atomicAdd(&hist[bin_of(n)], 1)] = s;
  }
}

hipError_t launch_varlen_table(const int* cu, int nseq, int T, int ncmax, int* coff, int* ct0, int* clen,
                               int* sorder, hipStream_t st) {
  hipLaunchKernelGGL(varlen_table_kernel, dim3(1), dim3(1024), 0, st, cu, nseq, T, ncmax, coff, ct0, clen, sorder);
  return hipGetLastError();
}

}  // namespace gdr2
