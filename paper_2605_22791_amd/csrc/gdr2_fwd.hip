// Forward kernels of the chunkwise WY GDR-2 operator (gfx950).
//
//   fwd_intra  one workgroup per (chunk, head, batch): the decay scan, the
//              gate-absorbed tiles, the Gram T and scores A_qk on MFMA, the
//              fp32 WY solve and the auxiliaries Y = A Ebar, U = A (W*V)
//              (Sec. 3.3; App. A; App. C.2: the intra-chunk products, the WY
//              solve and the construction of the auxiliaries).
//   fwd_state  one workgroup per (sequence, head) and one or two 16-column value
//              slices: the sequential inter-chunk recurrence (eq.
//              eq_gdn2_chunk_state) with the fp32 state in registers, fused with
//              the chunk output (eq. eq_gdn2_chunk_output).  Columns of S evolve
//              independently, so the value axis is split across workgroups.

#include "gdr2_kernels.hpp"

#include <type_traits>

namespace gdr2 {

// ---------------------------------------------------------------------------
// fwd_intra.  Workspace written per chunk-head `ch`:
//   Y[ch]   (64 x DK)  Y = A Ebar,   Ebar = gamma*(b*k)
//   U[ch]   (64 x DV)  U = A Z,      Z = w*v
//   Kt[ch]  (64 x DK)  Ktail rows (gamma_C / gamma_r) * k_r
//   Qg[ch]  (64 x DK)  gamma_r * q_r
//   Aqk[ch] (64 x 64)  causal scores, zero above the diagonal
//   GC[ch]  (DK)       gamma_C
template <int DK, int DV>
__global__ __launch_bounds__(512) void fwd_intra_kernel(IntraArgs a) {
  constexpr int NTHR = 512;
  constexpr int LS = DK + 4;
  ChunkPos cp;
  if (!chunk_pos(a.vl, blockIdx.x, blockIdx.y, blockIdx.z, a.T, a.H, a.NT, cp)) return;
  const int h = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int H = a.H;
  const size_t rs = (size_t)(H / a.G) * DK, rsv = (size_t)H * DV;  // key side on the H / G key heads
  const size_t row0 = cp.row0;
  const int len = cp.len;  // rows in use: the rest read as zero and are not written
  const size_t kbase = row0 * rs + (size_t)(h / a.G) * DK;
  const size_t vbase = row0 * rsv + (size_t)h * DV;
  const size_t ch = cp.ch;

  extern __shared__ float smem[];
  float* sR0 = smem;                      // G (64 x LS), later T (64 x LD64)
  float* sLe = sR0 + CH * LS;             // b*k times its left factor (chunk_refs)
  float* sLq = sLe + CH * LS;             // q times it; later Z and solve scratch
  float* sRk = sLq + CH * LS;             // k times its right factor
  float* sA = sRk + CH * LS;              // A (64 x LD64)
  float* eP = sA + CH * LD64;             // 4 x DK
  float* brg = eP + 4 * DK;               // 10 x DK
  float* eGC = brg + 10 * DK;             // DK
  int* split = reinterpret_cast<int*>(eGC + DK);
  float* sG = sR0;
  float* sT = sR0;

  if (tid < 4) split[tid] = 0;
  chunk_cumsum<DK, NTHR>(a.g + kbase, rs, sG, tid, len);
  chunk_refs<DK, NTHR>(sG, eP, brg, eGC, split, tid);

  // gate-absorbed tiles; Qg and Ktail go straight to the workspace
  float* Qg = a.Qg + ch * CH * DK;
  float* Kt = a.Kt + ch * CH * DK;
  for (int e = tid; e < CH * DK / 4; e += NTHR) {
    const int r = e / (DK / 4), c4 = (e % (DK / 4)) * 4, i = r >> 4;
    const float4 kk = ld4z(a.k + kbase + r * rs + c4, r < len);
    const float4 bv = ld4z(a.b + kbase + r * rs + c4, r < len);
    const float4 qq = ld4z(a.q + kbase + r * rs + c4, r < len);
    float4 qg, kt;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c4 + u;
      const float G = sG[r * LS + c];
      const float lf = expf(G - sG[left_row(split, i) * LS + c]);
      const float rf = expf(sG[right_row(split, i) * LS + c] - G);
      const float kv = f4at(kk, u), qv = f4at(qq, u);
      sLe[r * LS + c] = f4at(bv, u) * kv * lf;
      sLq[r * LS + c] = qv * lf;
      sRk[r * LS + c] = kv * rf;
      const float gq = qv * expf(G), gk = kv * expf(sG[(CH - 1) * LS + c] - G);
      if (u == 0) { qg.x = gq; kt.x = gk; }
      if (u == 1) { qg.y = gq; kt.y = gk; }
      if (u == 2) { qg.z = gq; kt.z = gk; }
      if (u == 3) { qg.w = gq; kt.w = gk; }
    }
    *reinterpret_cast<float4*>(Qg + r * DK + c4) = qg;
    *reinterpret_cast<float4*>(Kt + r * DK + c4) = kt;
  }
  for (int c = tid; c < DK; c += NTHR) a.GC[ch * DK + c] = eGC[c];
  __syncthreads();  // sG dead from here on; region reused for T

  // T (strict lower) and A_qk (lower incl. diagonal): 10 + 10 tiles of 16x16
  float* Aqk = a.Aqk + ch * CH * CH;
  for (int it = wave; it < 20; it += NTHR / 64) {
    const bool isT = it < 10;
    int i, j;
    pair_of(isT ? it : it - 10, i, j);
    f4 acc;
    if (i == j && split[i] == kSplitNone) {
      acc = isT ? diag_tile_direct<DK>(a.b + kbase, a.k + kbase, a.k + kbase, a.g + kbase, rs, i, lane, true, len)
                : diag_tile_direct<DK>(a.q + kbase, nullptr, a.k + kbase, a.g + kbase, rs, i, lane, false, len);
    } else {
      acc = gram_tile<DK>(isT ? sLe : sLq, sRk, brg, split, i, j, lane);
    }
    const int ccol = 16 * j + (lane & 15);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 16 * i + 4 * (lane >> 4) + u;
      if (isT) {
        sT[r * LD64 + ccol] = (r > ccol) ? acc[u] : 0.f;
      } else {
        Aqk[r * CH + ccol] = (r >= ccol) ? acc[u] : 0.f;
      }
    }
  }
  // zero the strictly-upper score tiles
  for (int e = tid; e < CH * CH; e += NTHR) {
    const int r = e / CH, s = e % CH;
    if ((s >> 4) > (r >> 4)) Aqk[r * CH + s] = 0.f;
  }
  __syncthreads();

  wy_solve<NTHR>(sT, sA, sLq, tid);  // sLq is free: used as solve scratch

  // Z = w * v into the sLq region (row stride DV + 4)
  float* sZ = sLq;
  constexpr int LZ = DV + 4;
  for (int e = tid; e < CH * DV / 4; e += NTHR) {
    const int r = e / (DV / 4), c4 = (e % (DV / 4)) * 4;
    const float4 wv = ld4z(a.w + vbase + r * rsv + c4, r < len);
    const float4 vv = ld4z(a.v + vbase + r * rsv + c4, r < len);
    float* d = sZ + r * LZ + c4;
    d[0] = wv.x * vv.x; d[1] = wv.y * vv.y; d[2] = wv.z * vv.z; d[3] = wv.w * vv.w;
  }
  __syncthreads();

  // Y = A Ebar (Ebar = Le * eP[block]) and U = A Z, lower-triangular A
  float* Yo = a.Y + ch * CH * DK;
  float* Uo = a.U + ch * CH * DV;
  constexpr int NCB = DK / 16 + DV / 16;
  for (int it = wave; it < NCB; it += NTHR / 64) {
    const bool isY = it < DK / 16;
    const int cb = isY ? it : it - DK / 16;
    const int col = 16 * cb + (lane & 15);
    for (int i = 0; i < 4; ++i) {
      f4 acc = {0.f, 0.f, 0.f, 0.f};
      const float* pa = sA + (16 * i + (lane & 15)) * LD64 + 4 * (lane >> 4);
      for (int kb = 0; kb <= i; ++kb) {
        const float4 av = ld4(pa + 16 * kb);
        const int s0 = 16 * kb + 4 * (lane >> 4);
        float bv[4];
        if (isY) {
          const float ep = eP[kb * DK + col];
#pragma unroll
          for (int u = 0; u < 4; ++u) bv[u] = sLe[(s0 + u) * LS + col] * ep;
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) bv[u] = sZ[(s0 + u) * LZ + col];
        }
        acc = mfma4(av.x, bv[0], acc);
        acc = mfma4(av.y, bv[1], acc);
        acc = mfma4(av.z, bv[2], acc);
        acc = mfma4(av.w, bv[3], acc);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 16 * i + 4 * (lane >> 4) + u;
        if (isY)
          Yo[r * DK + col] = acc[u];
        else
          Uo[r * DV + col] = acc[u];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// fwd_state: S carried across chunks, one workgroup per (sequence, head) and
// 16-column slice of the values.  Per chunk:
//   R   = U - Y S                         (eq. eq_app_residual_matrix)
//   O   = scale * (Qg S + Aqk R)          (eq. eq_app_chunk_output)  [WITH_O]
//   S  <- Diag(gamma_C) S + Ktail^T R     (eq. eq_app_chunk_state)
// With STORE_H the chunk-start states h_n and R are kept for the backward.
//
// A chunk is a serial chain and few sequences leave most of the chip idle, so
// what counts is the chain's length: narrow slices (a product is 32 fp32 MFMAs
// deep at most), waves 0-3 forming R while waves 4-7 form Qg S, one 16 x 16 tile
// of S per wave kept in its registers, two barriers a chunk, and every operand
// loaded straight into the registers of the wave that multiplies it two chunks
// ahead.  S and R meet the other waves through LDS transposed ([v][c], [v][r]),
// so that four K-steps' values are one 16-byte access without bank conflicts.
// 8 sequences x 16 chunks at 128 x 128: 59 us, without the output 40 (32 columns
// a workgroup, four waves, operands loaded where they are used: 160 and 110; the
// two roles in one body, whose waits then counted the barer role: 95 and 45).
// The slices of a sequence share their XCD (state_slot), hence its L2.
//
// Many pairs fill the chip whatever a slice's width, and then every slice's reading of
// the key-side tiles counts: two slices a workgroup (NV = 2, the same sums).  Forward
// calls, 128 x 128, NV = 1 / 2: 128 pairs of 256 tokens 136 / 118 us, 64 of 512 128 / 113,
// 32 of 1000 (256 slices, one a CU) 126 / 150, 4 of 512 63 / 76.
template <int DK, int DV, bool WITH_O, bool STORE_H, int NV>
__global__ __launch_bounds__(512) void fwd_state_kernel(StateArgs a) {
  constexpr int NCB = DK / 16;      // key blocks: S tiles, one per wave
  constexpr int LT = DK + 4, LR = CH + 4;
  int q, vs;
  if (!state_slot<DV / (16 * NV)>(blockIdx.x, a.nq, q, vs)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4, v0 = 16 * NV * vs + lr;
  const size_t seq = (size_t)scan_pair(a.vl, q, a.H);  // (sequence, head) pair
  const int h = (int)(seq % a.H);
  const ScanRange rng = scan_range(a.vl, (int)seq, a.H, a.T, a.NT);
  const bool low = wave < 4, own = NCB == 8 || low;
  const int i = wave & 3, cb = own ? wave : 0;  // row block of the products; key block of the S tile

  __shared__ __align__(16) float sS[16 * NV * LT];  // [v][c]
  __shared__ __align__(16) float sR[16 * NV * LR];  // [v][r]

  f4 st[NV];  // S[16 cb + 4 lg + u][v0 + 16 t]
  const size_t so = (seq * DK + 16 * cb + 4 * lg) * DV + v0;
#pragma unroll
  for (int t = 0; t < NV; ++t) {
    st[t] = f4{0.f, 0.f, 0.f, 0.f};
    if (own && a.S0 != nullptr) {
#pragma unroll
      for (int u = 0; u < 4; ++u) st[t][u] = a.S0[so + (size_t)u * DV + 16 * t];
    }
    if (own) *reinterpret_cast<f4*>(sS + (16 * t + lr) * LT + 16 * cb + 4 * lg) = st[t];
  }

  // the two roles as code of their own: on each the same loads and stores go out
  // every chunk, so that a wait for one chunk's operands leaves the rest in flight
  const auto run = [&](auto LOWC) {
    constexpr bool LOW = decltype(LOWC)::value, OWN = NCB == 8 || LOW;
    struct Ops {
      float4 p[DK / 16];  // row 16 i + lr of Y (waves 0-3) or Qg, channels 16 j + 4 lg ..
      float4 x[4];        // waves 4-7: Aqk row 16 i + lr, keys 16 j + 4 lg ..; waves 0-3: x[t] = U's tiles
      float k[4][4];      // Ktail[16 j + 4 lg + t][16 cb + lr]
      float4 g;           // gamma_C of channels 16 cb + 4 lg ..
    };
    const auto load = [&](Ops& o, int n) {
      // past the end the last chunk again, unused, one cache line a load: with each
      // lane's own line it was twice the traffic for a sequence of two chunks (512 pairs
      // of 128 tokens 341 us, 312)
      const size_t ch = rng.chs + min(n, rng.c1 - 1);
      const int all = n < rng.c1 ? -1 : 0;
      const float* P = (LOW ? a.Y : a.Qg) + ch * CH * DK + (((16 * i + lr) * DK + 4 * lg) & all);
      if (LOW || WITH_O) {
#pragma unroll
        for (int j = 0; j < DK / 16; ++j) o.p[j] = ld4(P + 16 * j);
      }
      if (LOW) {
        const float* U = a.U + ch * CH * DV + (((16 * i + 4 * lg) * DV + v0) & all);
#pragma unroll
        for (int t = 0; t < NV; ++t)
          o.x[t] = make_float4(U[16 * t], U[DV + 16 * t], U[2 * DV + 16 * t], U[3 * DV + 16 * t]);
      } else if (WITH_O) {
        const float* A = a.Aqk + ch * CH * CH + (((16 * i + lr) * CH + 4 * lg) & all);
#pragma unroll
        for (int j = 0; j < 4; ++j) o.x[j] = ld4(A + 16 * min(j, i));
      }
      if (OWN) {
        const float* K = a.Kt + ch * CH * DK + ((4 * lg * DK + 16 * cb + lr) & all);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int t = 0; t < 4; ++t) o.k[j][t] = K[(16 * j + t) * DK];
        o.g = ld4(a.GC + ch * DK + 16 * cb + 4 * lg);
      }
    };
    const auto step = [&](Ops& o, int n, auto FETCH) {
      const size_t ch = rng.chs + n;
      if (STORE_H && OWN) {
        float* Hn = a.Hs + (ch * DK + 16 * cb + 4 * lg) * DV + v0;
#pragma unroll
        for (int t = 0; t < NV; ++t)
#pragma unroll
          for (int u = 0; u < 4; ++u) Hn[u * DV + 16 * t] = st[t][u];
      }
      // Y S (waves 0-3), Qg S (waves 4-7): two accumulators, so that a product does not wait for the one before
      f4 acc[NV], ac2[NV];
#pragma unroll
      for (int t = 0; t < NV; ++t) acc[t] = ac2[t] = f4{0.f, 0.f, 0.f, 0.f};
      if (LOW || WITH_O) {
#pragma unroll
        for (int j = 0; j < DK / 16; ++j) {
          const float4 y = o.p[j];
#pragma unroll
          for (int t = 0; t < NV; ++t) {
            const float4 s = ld4(sS + (16 * t + lr) * LT + 16 * j + 4 * lg);
            acc[t] = mfma4(y.x, s.x, acc[t]);
            ac2[t] = mfma4(y.y, s.y, ac2[t]);
            acc[t] = mfma4(y.z, s.z, acc[t]);
            ac2[t] = mfma4(y.w, s.w, ac2[t]);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < NV; ++t) {
        acc[t] += ac2[t];
        if (LOW) {
          const f4 R = f4{o.x[t].x, o.x[t].y, o.x[t].z, o.x[t].w} - acc[t];
          *reinterpret_cast<f4*>(sR + (16 * t + lr) * LR + 16 * i + 4 * lg) = R;
          if (STORE_H) {
            float* Rn = a.Rs + (ch * CH + 16 * i + 4 * lg) * DV + v0 + 16 * t;
#pragma unroll
            for (int u = 0; u < 4; ++u) Rn[u * DV] = R[u];
          }
        }
      }
      __syncthreads();  // R is there, and nobody reads this chunk's S any more
      float4 r[NV][4];
#pragma unroll
      for (int t = 0; t < NV; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) r[t][j] = ld4(sR + (16 * t + lr) * LR + 16 * j + 4 * lg);
      if (OWN) {
        f4 s2[NV];
#pragma unroll
        for (int t = 0; t < NV; ++t) {
          st[t] = f4{o.g.x * st[t][0], o.g.y * st[t][1], o.g.z * st[t][2], o.g.w * st[t][3]};
          s2[t] = f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int t = 0; t < NV; ++t) {
            st[t] = mfma4(o.k[j][0], r[t][j].x, st[t]);
            s2[t] = mfma4(o.k[j][1], r[t][j].y, s2[t]);
            st[t] = mfma4(o.k[j][2], r[t][j].z, st[t]);
            s2[t] = mfma4(o.k[j][3], r[t][j].w, s2[t]);
          }
#pragma unroll
        for (int t = 0; t < NV; ++t) {
          st[t] += s2[t];
          *reinterpret_cast<f4*>(sS + (16 * t + lr) * LT + 16 * cb + 4 * lg) = st[t];
        }
      }
      if (WITH_O && !LOW) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (j > i) break;
#pragma unroll
          for (int t = 0; t < NV; ++t) {
            acc[t] = mfma4(o.x[j].x, r[t][j].x, acc[t]);
            acc[t] = mfma4(o.x[j].y, r[t][j].y, acc[t]);
            acc[t] = mfma4(o.x[j].z, r[t][j].z, acc[t]);
            acc[t] = mfma4(o.x[j].w, r[t][j].w, acc[t]);
          }
        }
        size_t row0;
        int len;
        scan_rows(rng, n, row0, len);
        // rows past the chunk's end go over U's, which nobody reads any more: a
        // store on every path (waits count stores too)
        float* O = a.o + ((row0 + 16 * i + 4 * lg) * a.H + h) * DV + v0;
        float* X = const_cast<float*>(a.U) + (ch * CH + 16 * i + 4 * lg) * DV + v0;
#pragma unroll
        for (int t = 0; t < NV; ++t)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            *(16 * i + 4 * lg + u < len ? O + (size_t)u * a.H * DV + 16 * t : X + u * DV + 16 * t) = a.scale * acc[t][u];
      }
      if constexpr (decltype(FETCH)::value) load(o, n + 2);
      __syncthreads();
    };
    if (NV == 2 && rng.c0 + 1 == rng.c1) {  // a single chunk: nothing else to fetch (256 pairs of 64 tokens 73 / 67 us)
      Ops oa;
      load(oa, rng.c0);
      __syncthreads();
      step(oa, rng.c0, std::false_type{});
    } else if (rng.c0 < rng.c1) {
      Ops oa, ob;
      load(oa, rng.c0);
      load(ob, rng.c0 + 1);
      __syncthreads();
      for (int n = rng.c0; n < rng.c1; n += 2) {
        step(oa, n, std::true_type{});
        if (n + 1 < rng.c1) step(ob, n + 1, std::true_type{});
      }
    }
  };
  if (low)
    run(std::true_type{});
  else
    run(std::false_type{});
  if (a.ST != nullptr && own) {
#pragma unroll
    for (int t = 0; t < NV; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) a.ST[so + (size_t)u * DV + 16 * t] = st[t][u];
  }
}

// ---------------------------------------------------------------------------
template <int DK, int DV>
hipError_t launch_fwd_intra(const IntraArgs& a, int B, hipStream_t st) {
  constexpr size_t lds = sizeof(float) * (4 * CH * (DK + 4) + CH * LD64 + 15 * DK) + 4 * sizeof(int);
  // Z (row stride DV+4) reuses the dead sLq + sRk regions
  static_assert(CH * (DV + 4) <= 2 * CH * (DK + 4), "Z tile fits the freed regions");
  static_assert(CH * LD64 <= CH * (DK + 4), "T tile fits the G region");
  hipError_t e = hipFuncSetAttribute((const void*)fwd_intra_kernel<DK, DV>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  dim3 grid(a.vl.ct0 ? a.vl.ncmax : a.NT, a.H, a.vl.ct0 ? 1 : B);
  hipLaunchKernelGGL((fwd_intra_kernel<DK, DV>), grid, dim3(512), lds, st, a);
  return hipGetLastError();
}

template <int DK, int DV, bool WITH_O, bool STORE_H>
hipError_t launch_fwd_state(const StateArgs& a, hipStream_t st) {
  if ((long long)a.nq * (DV / 16) <= 256)  // a CU for each narrow slice
    hipLaunchKernelGGL((fwd_state_kernel<DK, DV, WITH_O, STORE_H, 1>), dim3(state_slots<DV / 16>(a.nq)), dim3(512),
                       0, st, a);
  else
    hipLaunchKernelGGL((fwd_state_kernel<DK, DV, WITH_O, STORE_H, 2>), dim3(state_slots<DV / 32>(a.nq)), dim3(512),
                       0, st, a);
  return hipGetLastError();
}

#define GDR2_INST_FWD(DK, DV)                                                               \
  template hipError_t launch_fwd_intra<DK, DV>(const IntraArgs&, int, hipStream_t);         \
  template hipError_t launch_fwd_state<DK, DV, true, false>(const StateArgs&, hipStream_t); \
  template hipError_t launch_fwd_state<DK, DV, false, true>(const StateArgs&, hipStream_t); \
  template hipError_t launch_fwd_state<DK, DV, true, true>(const StateArgs&, hipStream_t);

GDR2_INST_FWD(64, 64)
GDR2_INST_FWD(64, 128)
GDR2_INST_FWD(128, 64)
GDR2_INST_FWD(128, 128)

}  // namespace gdr2
