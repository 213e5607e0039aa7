// Segment chaining of the sequence-parallel state scans (gfx950).
//
// The chunk recursion of the state (eq. eq_gdn2_chunk_state with R from
// eq. eq_app_residual_matrix) is affine in the state:
//     S_{n+1} = (Diag(gamma_C) - Ktail^T Y) S_n + Ktail^T U,
// so a segment of chunks maps its start state X to M X + N, where M is the
// product of the chunk transitions (obtained by scanning identity columns with
// U = 0) and N the segment's end state from a zero start.  The reverse scan of
// the gradient is affine the same way (App. B.1).  This kernel walks the
// segments of each sequence in order (forward) or backwards (reverse),
// X <- M_k X + N_k, and writes the value entering every segment; the segments
// are then re-scanned in parallel from those values.  With no input a chunk's
// reverse step, dS <- Diag(gamma_C) dS - Y^T (Ktail dS), is the transpose of
// its forward step, so the reverse chain of a square state can use the
// forward's maps as M_k^T (transpose_m).
//
// The chain is serial and short, so its length counts: one workgroup per
// (sequence, 16-wide value slice) with a wave per key block of X, each wave's rows
// of M_k and N_k loaded straight into its registers two links ahead, fp32 MFMA
// (no splitting; 32 products deep at Dk = 128), X handed round through LDS with
// one barrier a link.  The slices of a sequence share their XCD (state_slot).
// 16 sequences x 8 segments at 128 x 128: 21 us (39 with split-bf16 products on
// 64-wide slices and M_k loaded where it is used, 4.7 us a link).

#include "gdr2_kernels.hpp"

namespace gdr2 {

template <int DK, int DV>
__global__ __launch_bounds__(4 * DK) void segcombine_kernel(SegCombineArgs a) {
  constexpr int LX = DK + 4;
  __shared__ __align__(16) float sX[2][16 * LX];  // X [v][c], by link parity
  int seq, vs;
  if (!state_slot<DV / 16>(blockIdx.x, a.nseq, seq, vs)) return;
  const int lane = threadIdx.x & 63, cb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lg = lane >> 4, v0 = 16 * vs + lr, nseg = a.nseg;
  const size_t o = (size_t)(16 * cb + 4 * lg) * DV + v0;  // the lane's X[16 cb + 4 lg + u][v0], u = 0
  const auto seg = [&](int step) { return (size_t)seq * nseg + (a.reverse ? nseg - 1 - step : step); };

  struct Ops {
    f4 m[DK / 16];  // M[16 cb + lr][16 j + 4 lg ..] (transposed: M[16 j + 4 lg ..][16 cb + lr])
    f4 n;           // N's tile
  };
  const auto load = [&](Ops& x, int step) {
    const size_t sk = seg(min(step, nseg - 1));  // past the last link: unused
    const float *M = a.M + sk * DK * DK, *N = a.N + sk * DK * DV + o;
    if (a.transpose_m) {
#pragma unroll
      for (int j = 0; j < DK / 16; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t) x.m[j][t] = M[(size_t)(16 * j + 4 * lg + t) * DK + 16 * cb + lr];
    } else {
#pragma unroll
      for (int j = 0; j < DK / 16; ++j) x.m[j] = *reinterpret_cast<const f4*>(M + (16 * cb + lr) * DK + 16 * j + 4 * lg);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) x.n[u] = N[(size_t)u * DV];
    asm volatile("" ::: "memory");  // the loads stay here: the compiler would sink them to their use
  };
  f4 x = f4{0.f, 0.f, 0.f, 0.f};
  if (a.X0 != nullptr) {
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = a.X0[(size_t)seq * DK * DV + o + (size_t)u * DV];
  }
  const auto enter = [&](int step) {  // the value entering segment `step`
    float* xs = a.Xs + seg(step) * DK * DV + o;
#pragma unroll
    for (int u = 0; u < 4; ++u) xs[(size_t)u * DV] = x[u];
  };
  const auto link = [&](Ops& w, int step) {  // then X <- M X + N
    enter(step);
    float* X = sX[step & 1] + lr * LX;
    *reinterpret_cast<f4*>(X + 16 * cb + 4 * lg) = x;
    __syncthreads();  // (the readers of the link before last are done, or they had not met the last link's)
    f4 x2 = f4{0.f, 0.f, 0.f, 0.f};
    x = w.n;
#pragma unroll
    for (int j = 0; j < DK / 16; ++j) {
      const f4 y = *reinterpret_cast<const f4*>(X + 16 * j + 4 * lg);
      x = mfma4(w.m[j][0], y[0], x);
      x2 = mfma4(w.m[j][1], y[1], x2);
      x = mfma4(w.m[j][2], y[2], x);
      x2 = mfma4(w.m[j][3], y[3], x2);
    }
    x += x2;
    load(w, step + 2);
  };
  Ops oa, ob;
  load(oa, 0);
  load(ob, 1);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the loop's waits then count its own loads and stores alone
  int step = 0;
  for (; step + 2 < nseg; step += 2) {
    link(oa, step);
    link(ob, step + 1);
  }
  if (step + 1 < nseg) link(oa, step++);
  enter(step);  // nothing follows the last segment
}

template <int DK, int DV>
hipError_t launch_segcombine(const SegCombineArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((segcombine_kernel<DK, DV>), dim3(state_slots<DV / 16>(a.nseq)), dim3(4 * DK), 0, st, a);
  return hipGetLastError();
}

template hipError_t launch_segcombine<64, 64>(const SegCombineArgs&, hipStream_t);
template hipError_t launch_segcombine<64, 128>(const SegCombineArgs&, hipStream_t);
template hipError_t launch_segcombine<128, 64>(const SegCombineArgs&, hipStream_t);
template hipError_t launch_segcombine<128, 128>(const SegCombineArgs&, hipStream_t);

}  // namespace gdr2
