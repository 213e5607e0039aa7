// Backward kernels of the chunkwise WY GDR-2 operator (gfx950), App. B / App. C.3.
//
//   bwd_state  reverse inter-chunk scan (state and output paths, App. B.1):
//                dR_n  = scale * Aqk^T dO_n + Ktail dS_{n+1}
//                dS_n  = Diag(gamma_C) dS_{n+1} + scale * Qg^T dO_n - Y^T dR_n
//              one workgroup per (sequence, head) and 16-column value slice.
//   bwd_wy     the gate-aware WY vector-Jacobian product (App. B.2, the
//              method-specific step): dA_qk, dY = -dR S0^T, dZ = A^T dR (-> dw,
//              dv), dEbar = A^T dY, dA = dR Z^T + dY Ebar^T with the gates inside
//              the products, dT = -tril(A^T dA A^T, -1).
//   bwd_intra  the score / Gram / tail-key VJPs and the elementwise decay chain
//              (App. B.3 - B.5): dq, dk, db and dlog_alpha by a reverse
//              cumulative sum over the chunk.
//
// Every gamma^{-1} of App. B is paired with a gamma of the same channel so that
// only ratios exp(G_r - G_s), r >= s, appear; they are formed with the block
// factorisation described in gdr2_device.hpp.  Writing dEg = dEbar*gamma,
// dKg = dKbar/gamma and dq = dQg*gamma, App. B.4 becomes
//     db = dEg*k,  dk = dEg*b + dKg,  dG = dq*q - dKg*k + dEg*b*k,
// and d gamma_C (App. B.1, B.3) is added to the last row of dG (gamma_C is
// gamma at row C) before the reverse cumulative sum.

#include "gdr2_kernels.hpp"

#include <type_traits>

namespace gdr2 {

// ---------------------------------------------------------------------------
// The forward state kernel's plan (gdr2_fwd.hip) run backwards: 16 value columns
// a workgroup, a dS tile per wave in registers, operands two chunks ahead.  Waves
// 0-3 form dR while waves 4-7 form Qg^T dO, which needs no dS, for their own tile
// and for that of wave - 4.  8 sequences x 16 chunks at 128 x 128: 65 us (385
// with 32 columns, four waves and operands loaded where they are used).
template <int DK, int DV>
__global__ __launch_bounds__(512) void bwd_state_kernel(BwdStateArgs a) {
  constexpr int NCB = DK / 16;
  constexpr int LT = DK + 4, LR = CH + 4;
  int q, vs;
  if (!state_slot<DV / 16>(blockIdx.x, a.nq, q, vs)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4, v0 = 16 * vs + lr;
  const size_t seq = (size_t)scan_pair(a.vl, q, a.H);  // (sequence, head) pair
  const int h = (int)(seq % a.H);
  const ScanRange rng = scan_range(a.vl, (int)seq, a.H, a.T, a.NT);
  const bool low = wave < 4, own = NCB == 8 || low;
  const int i = wave & 3, cb = own ? wave : 0;

  __shared__ __align__(16) float sS[16 * LT];     // dS [v][c]
  __shared__ __align__(16) float sO[2][16 * LR];  // scale dO [v][r], by chunk parity
  __shared__ __align__(16) float sR[16 * LR];     // dR [v][r]
  __shared__ __align__(16) f4 sQ[4][64];          // Qg^T dO tiles of waves 0-3

  f4 st = f4{0.f, 0.f, 0.f, 0.f};  // dS[16 cb + 4 lg + u][v0]
  const size_t so = (seq * DK + 16 * cb + 4 * lg) * DV + v0;
  if (own) {
    if (a.dST != nullptr) {
#pragma unroll
      for (int u = 0; u < 4; ++u) st[u] = a.dST[so + (size_t)u * DV];
    }
    *reinterpret_cast<f4*>(sS + lr * LT + 16 * cb + 4 * lg) = st;
  }

  // the two roles as code of their own (as in the forward kernel)
  const auto run = [&](auto LOWC) {
    constexpr bool LOW = decltype(LOWC)::value, OWN = NCB == 8 || LOW;
    struct Ops {
      // waves 0-3: row 16 i + lr of Ktail; waves 4-7: Qg[16 j + 4 lg + t][16 wave + lr] in p[j],
      // the same of key block wave - 4 in p[4 + j] (DK = 64: that one alone, in p[j])
      float4 p[8];
      float x[4][4];  // waves 0-3: Aqk[16 j + 4 lg + t][16 i + lr]
      float y[4][4];  // Y[16 j + 4 lg + t][16 cb + lr]
      float4 g;       // gamma_C of channels 16 cb + 4 lg ..
      float2 d;       // dO row tid / 8, columns 2 (tid % 8) .. of the slice
      bool in;        // the row is one of the chunk's
    };
    const auto cols = [&](const float* P, int ld, float (&o)[4][4]) {  // P at row 4 lg
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t) o[j][t] = P[(16 * j + t) * ld];
    };
    const auto col4 = [&](const float* P) { return make_float4(P[0], P[DK], P[2 * DK], P[3 * DK]); };
    const auto load = [&](Ops& o, int n) {
      n = max(n, rng.c0);  // past the start: the first chunk again, unused
      const size_t ch = rng.chs + n;
      size_t row0;
      int len;
      scan_rows(rng, n, row0, len);
      // rows past the chunk's end read its last row; put_dO makes them zero
      const int r = tid >> 3;
      o.in = r < len;
      o.d = *reinterpret_cast<const float2*>(a.dout + ((row0 + min(r, len - 1)) * a.H + h) * DV + 16 * vs + 2 * (tid & 7));
      if (LOW) {
        const float* K = a.Kt + (ch * CH + 16 * i + lr) * DK + 4 * lg;
#pragma unroll
        for (int j = 0; j < DK / 16; ++j) o.p[j] = ld4(K + 16 * j);
        cols(a.Aqk + (ch * CH + 4 * lg) * CH + 16 * i + lr, CH, o.x);
      } else {
        const float* Q = a.Qg + (ch * CH + 4 * lg) * DK + lr;
#pragma unroll
        for (int j = 0; j < 4; ++j) o.p[j] = col4(Q + 16 * j * DK + 16 * (OWN ? wave : wave - 4));
        if (OWN) {
#pragma unroll
          for (int j = 0; j < 4; ++j) o.p[4 + j] = col4(Q + 16 * j * DK + 16 * (wave - 4));
        }
      }
      if (OWN) {
        cols(a.Y + (ch * CH + 4 * lg) * DK + 16 * cb + lr, DK, o.y);
        o.g = ld4(a.GC + ch * DK + 16 * cb + 4 * lg);
      }
    };
    const auto put_dO = [&](const Ops& o, int par) {
      float* d = sO[par] + 2 * (tid & 7) * LR + (tid >> 3);
      d[0] = o.in ? a.scale * o.d.x : 0.f;
      d[LR] = o.in ? a.scale * o.d.y : 0.f;
    };
    // nx: the next chunk's operands
    const auto step = [&](Ops& o, const Ops& nx, int n, int par) {
      const size_t ch = rng.chs + n;
      if (OWN) {
        float* Hn = a.DH + (ch * DK + 16 * cb + 4 * lg) * DV + v0;
#pragma unroll
        for (int u = 0; u < 4; ++u) Hn[u * DV] = st[u];
      }
      const float* dO = sO[par] + lr * LR + 4 * lg;
      f4 acc = f4{0.f, 0.f, 0.f, 0.f}, ac2 = acc;
      if (LOW) {  // dR = Ktail dS + Aqk^T dO, rows of block i
#pragma unroll
        for (int j = 0; j < DK / 16; ++j) {
          const float4 k = o.p[j], s = ld4(sS + lr * LT + 16 * j + 4 * lg);
          acc = mfma4(k.x, s.x, acc);
          ac2 = mfma4(k.y, s.y, ac2);
          acc = mfma4(k.z, s.z, acc);
          ac2 = mfma4(k.w, s.w, ac2);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (j < i) continue;
          const float4 d = ld4(dO + 16 * j);
          acc = mfma4(o.x[j][0], d.x, acc);
          ac2 = mfma4(o.x[j][1], d.y, ac2);
          acc = mfma4(o.x[j][2], d.z, acc);
          ac2 = mfma4(o.x[j][3], d.w, ac2);
        }
        acc += ac2;
        *reinterpret_cast<f4*>(sR + lr * LR + 16 * i + 4 * lg) = acc;
        float* Rn = a.DR + (ch * CH + 16 * i + 4 * lg) * DV + v0;
#pragma unroll
        for (int u = 0; u < 4; ++u) Rn[u * DV] = acc[u];
      } else {  // Qg^T dO: this wave's tile in acc, that of wave - 4 through LDS
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 d = ld4(dO + 16 * j), x = o.p[j], y = o.p[4 + j];
          acc = mfma4(x.x, d.x, acc);
          if (OWN) ac2 = mfma4(y.x, d.x, ac2);
          acc = mfma4(x.y, d.y, acc);
          if (OWN) ac2 = mfma4(y.y, d.y, ac2);
          acc = mfma4(x.z, d.z, acc);
          if (OWN) ac2 = mfma4(y.z, d.z, ac2);
          acc = mfma4(x.w, d.w, acc);
          if (OWN) ac2 = mfma4(y.w, d.w, ac2);
        }
        sQ[i][lane] = OWN ? ac2 : acc;
      }
      __syncthreads();  // dR and the tiles are there, and nobody reads this chunk's dS any more
      if (OWN) {
        // dS <- Diag(gamma_C) dS + Qg^T dO - Y^T dR
        const f4 qd = LOW ? sQ[i][lane] : acc;
        st = f4{o.g.x * st[0], o.g.y * st[1], o.g.z * st[2], o.g.w * st[3]} + qd;
        f4 y1 = f4{0.f, 0.f, 0.f, 0.f}, y2 = y1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 r = ld4(sR + lr * LR + 16 * j + 4 * lg);
          y1 = mfma4(o.y[j][0], r.x, y1);
          y2 = mfma4(o.y[j][1], r.y, y2);
          y1 = mfma4(o.y[j][2], r.z, y1);
          y2 = mfma4(o.y[j][3], r.w, y2);
        }
        st -= y1 + y2;
        *reinterpret_cast<f4*>(sS + lr * LT + 16 * cb + 4 * lg) = st;
      }
      put_dO(nx, par ^ 1);
      load(o, n - 2);
      __syncthreads();
    };
    if (rng.c0 < rng.c1) {
      Ops oa, ob;
      load(oa, rng.c1 - 1);
      load(ob, rng.c1 - 2);
      put_dO(oa, 0);
      __syncthreads();
      for (int n = rng.c1 - 1; n >= rng.c0; n -= 2) {
        step(oa, ob, n, 0);
        if (n - 1 >= rng.c0) step(ob, oa, n - 1, 1);
      }
    }
  };
  if (low)
    run(std::true_type{});
  else
    run(std::false_type{});
  if (a.dS0 != nullptr && own) {
#pragma unroll
    for (int u = 0; u < 4; ++u) a.dS0[so + (size_t)u * DV] = st[u];
  }
}

// ---------------------------------------------------------------------------
// Gate-aware WY VJP.  Writes dv, dw (final), and per chunk-head workspace:
//   DAqk (64x64) = tril(scale dO R^T),  DT (64x64) strict lower,
//   DEg (64xDK)  = (A^T dY) * gamma  with dY = -dR S0^T.
template <int DK, int DV>
__global__ __launch_bounds__(512) void bwd_wy_kernel(BwdChunkArgs a) {
  constexpr int NTHR = 512, NW = 8;
  constexpr int LS = DK + 4;
  ChunkPos cp;
  if (!chunk_pos(a.vl, blockIdx.x, blockIdx.y, blockIdx.z, a.T, a.H, a.NT, cp)) return;
  const int h = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int H = a.H;
  const size_t rs = (size_t)(H / a.G) * DK, rsv = (size_t)H * DV;  // key side on the H / G key heads
  const size_t row0 = cp.row0;
  const int len = cp.len;  // rows in use: the rest read as zero and are not written
  const size_t kbase = row0 * rs + (size_t)(h / a.G) * DK;
  const size_t vbase = row0 * rsv + (size_t)h * DV;
  const size_t ch = cp.ch;

  extern __shared__ float smem[];
  float* sR0 = smem;                // G, later X = A^T dA (LD64)
  float* sLe = sR0 + CH * LS;       // b*k times its left factor (chunk_refs)
  float* sRk = sLe + CH * LS;       // k times its right factor; later solve scratch, then dY
  float* sTd = sRk + CH * LS;       // T, later dA (LD64)
  float* sA = sTd + CH * LD64;      // A (LD64)
  float* eP = sA + CH * LD64;
  float* brg = eP + 4 * DK;
  float* eGC = brg + 10 * DK;
  int* split = reinterpret_cast<int*>(eGC + DK);
  float* sG = sR0;
  float* sX = sR0;
  float* sdY = sRk;

  const float* Hn = a.Hs + ch * DK * DV;
  const float* Rn = a.Rs + ch * CH * DV;
  const float* DRn = a.DR + ch * CH * DV;
  float* DAqk = a.DAqk + ch * CH * CH;
  float* DT = a.DT + ch * CH * CH;
  float* DEg = a.DEg + ch * CH * DK;

  if (tid < 4) split[tid] = 0;
  chunk_cumsum<DK, NTHR>(a.g + kbase, rs, sG, tid, len);
  chunk_refs<DK, NTHR>(sG, eP, brg, eGC, split, tid);
  for (int e = tid; e < CH * DK / 4; e += NTHR) {
    const int r = e / (DK / 4), c4 = (e % (DK / 4)) * 4, i = r >> 4;
    const float4 kk = ld4z(a.k + kbase + r * rs + c4, r < len);
    const float4 bv = ld4z(a.b + kbase + r * rs + c4, r < len);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c4 + u;
      const float G = sG[r * LS + c];
      const float kv = f4at(kk, u);
      sLe[r * LS + c] = f4at(bv, u) * kv * expf(G - sG[left_row(split, i) * LS + c]);
      sRk[r * LS + c] = kv * expf(sG[right_row(split, i) * LS + c] - G);
    }
  }
  __syncthreads();

  // T tiles (10) into sTd, and the 16 tiles of dA_qk = tril(scale dO R^T)
  for (int it = wave; it < 26; it += NW) {
    if (it < 10) {
      int i, j;
      pair_of(it, i, j);
      const f4 acc = (i == j && split[i] == kSplitNone)
                         ? diag_tile_direct<DK>(a.b + kbase, a.k + kbase, a.k + kbase,
                                                     a.g + kbase, rs, i, lane, true, len)
                         : gram_tile<DK>(sLe, sRk, brg, split, i, j, lane);
      const int s = 16 * j + lr;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 16 * i + 4 * lg + u;
        sTd[r * LD64 + s] = (r > s) ? acc[u] : 0.f;
      }
    } else {
      const int i = (it - 10) >> 2, j = (it - 10) & 3;
      f4 acc = {0.f, 0.f, 0.f, 0.f};
      if (j <= i) {
        const float* pd = a.dout + vbase + (16 * i + lr) * rsv + 4 * lg;
        const bool pdin = 16 * i + lr < len;
        const float* pr = Rn + (16 * j + lr) * DV + 4 * lg;
        for (int kk = 0; kk < DV; kk += 16) {
          const float4 dv4 = ld4z(pd + kk, pdin), r4 = ld4(pr + kk);
          acc = mfma4(dv4.x, r4.x, acc);
          acc = mfma4(dv4.y, r4.y, acc);
          acc = mfma4(dv4.z, r4.z, acc);
          acc = mfma4(dv4.w, r4.w, acc);
        }
      }
      const int s = 16 * j + lr;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 16 * i + 4 * lg + u;
        DAqk[r * CH + s] = (r >= s) ? a.scale * acc[u] : 0.f;
      }
    }
  }
  __syncthreads();

  wy_solve<NTHR>(sTd, sA, sRk, tid);  // sRk is dead after T; used as scratch

  // dY = -dR S0^T  (64 x DK) into sdY
  for (int it = wave; it < 4 * (DK / 16); it += NW) {
    const int i = it / (DK / 16), cb = it % (DK / 16);
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    const float* pa = DRn + (16 * i + lr) * DV + 4 * lg;
    const float* pb = Hn + (16 * cb + lr) * DV + 4 * lg;
    for (int kk = 0; kk < DV; kk += 16) {
      const float4 x = ld4(pa + kk), y = ld4(pb + kk);
      acc = mfma4(-x.x, y.x, acc);
      acc = mfma4(-x.y, y.y, acc);
      acc = mfma4(-x.z, y.z, acc);
      acc = mfma4(-x.w, y.w, acc);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) sdY[(16 * i + 4 * lg + u) * LS + 16 * cb + lr] = acc[u];
  }
  __syncthreads();

  // dZ = A^T dR (-> dw = dZ*v, dv = dZ*w) and dEg = (A^T dY) * gamma
  for (int it = wave; it < 4 * (DV / 16) + 4 * (DK / 16); it += NW) {
    const bool isZ = it < 4 * (DV / 16);
    const int idx = isZ ? it : it - 4 * (DV / 16);
    const int NB = isZ ? DV / 16 : DK / 16;
    const int i = idx / NB, cb = idx % NB;
    const int col = 16 * cb + lr;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int kk = 16 * i; kk < CH; kk += 4) {
      const int r = kk + lg;
      const float av = sA[r * LD64 + 16 * i + lr];
      const float bv = isZ ? DRn[r * DV + col] : sdY[r * LS + col];
      acc = mfma4(av, bv, acc);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int s = 16 * i + 4 * lg + u;
      if (isZ) {
        const size_t off = vbase + s * rsv + col;
        if (s < len) {
          a.dw[off] = acc[u] * a.v[off];
          a.dv[off] = acc[u] * a.w[off];
        }
      } else {
        DEg[s * DK + col] = acc[u] * expf(sG[s * LS + col]);
      }
    }
  }
  __syncthreads();  // sG and T dead from here on

  // dA = dR Z^T + dY Ebar^T, strictly lower part, into sTd
  for (int it = wave; it < 16; it += NW) {
    const int i = it >> 2, j = it & 3;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    if (j <= i) {
      const float* pa = DRn + (16 * i + lr) * DV + 4 * lg;
      const float* pw = a.w + vbase + (16 * j + lr) * rsv + 4 * lg;
      const float* pv = a.v + vbase + (16 * j + lr) * rsv + 4 * lg;
      const bool jin = 16 * j + lr < len;
      for (int kk = 0; kk < DV; kk += 16) {
        const float4 x = ld4(pa + kk), w4 = ld4z(pw + kk, jin), v4 = ld4z(pv + kk, jin);
        acc = mfma4(x.x, w4.x * v4.x, acc);
        acc = mfma4(x.y, w4.y * v4.y, acc);
        acc = mfma4(x.z, w4.z * v4.z, acc);
        acc = mfma4(x.w, w4.w * v4.w, acc);
      }
      const float* py = sdY + (16 * i + lr) * LS + 4 * lg;
      const float* pe = sLe + (16 * j + lr) * LS + 4 * lg;
      const float* pp = eP + j * DK + 4 * lg;
      for (int kk = 0; kk < DK; kk += 16) {
        const float4 x = ld4(py + kk), e4 = ld4(pe + kk), p4 = ld4(pp + kk);
        acc = mfma4(x.x, e4.x * p4.x, acc);
        acc = mfma4(x.y, e4.y * p4.y, acc);
        acc = mfma4(x.z, e4.z * p4.z, acc);
        acc = mfma4(x.w, e4.w * p4.w, acc);
      }
    }
    const int s = 16 * j + lr;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 16 * i + 4 * lg + u;
      sTd[r * LD64 + s] = (r > s) ? acc[u] : 0.f;
    }
  }
  __syncthreads();

  // X = A^T dA, lower tiles
  for (int it = wave; it < 10; it += NW) {
    int i, j;
    pair_of(it, i, j);
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int kk = 16 * i; kk < CH; kk += 4) {
      const int p = kk + lg;
      acc = mfma4(sA[p * LD64 + 16 * i + lr], sTd[p * LD64 + 16 * j + lr], acc);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) sX[(16 * i + 4 * lg + u) * LD64 + 16 * j + lr] = acc[u];
  }
  __syncthreads();

  // dT = -tril(X A^T, -1)
  for (int it = wave; it < 16; it += NW) {
    const int i = it >> 2, j = it & 3;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    if (j <= i) {
      for (int kb = 0; kb <= j; ++kb) {
        const float4 x = ld4(sX + (16 * i + lr) * LD64 + 16 * kb + 4 * lg);
        const float4 y = ld4(sA + (16 * j + lr) * LD64 + 16 * kb + 4 * lg);
        acc = mfma4(x.x, y.x, acc);
        acc = mfma4(x.y, y.y, acc);
        acc = mfma4(x.z, y.z, acc);
        acc = mfma4(x.w, y.w, acc);
      }
    }
    const int s = 16 * j + lr;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 16 * i + 4 * lg + u;
      DT[r * CH + s] = (r > s) ? -acc[u] : 0.f;
    }
  }
}

// ---------------------------------------------------------------------------
// Intra-chunk VJP and decay chain: dq, dk, db, dlog_alpha.
template <int DK, int DV>
__global__ __launch_bounds__(512) void bwd_intra_kernel(BwdChunkArgs a) {
  constexpr int NTHR = 512, NW = 8;
  constexpr int LS = DK + 4;
  constexpr int NCB = DK / 16;
  constexpr int NITEM = 4 * NCB;
  constexpr int IPW = NITEM / NW;
  constexpr int NSPLIT = NTHR / DK;
  static_assert(NITEM % NW == 0, "items per wave");
  ChunkPos cp;
  if (!chunk_pos(a.vl, blockIdx.x, blockIdx.y, blockIdx.z, a.T, a.H, a.NT, cp)) return;
  const int h = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int H = a.H;
  const size_t rs = (size_t)(H / a.G) * DK, rsv = (size_t)H * DV;  // key side on the H / G key heads
  const size_t row0 = cp.row0;
  const int len = cp.len;  // rows in use: the rest read as zero and are not written
  const size_t kbase = row0 * rs + (size_t)(h / a.G) * DK;
  // key-side gradients: with grouped value heads (G > 1) this value head's
  // contribution goes, on the value-head axis, to the fp32 partials the group
  // reduction sums
  const size_t rso = a.G > 1 ? (size_t)H * DK : rs;
  const size_t kobase = a.G > 1 ? row0 * rso + (size_t)h * DK : kbase;
  const size_t vbase = row0 * rsv + (size_t)h * DV;
  const size_t ch = cp.ch;

  extern __shared__ float smem[];
  float* sG = smem;
  float* sLe = sG + CH * LS;
  float* sLq = sLe + CH * LS;
  float* sRk = sLq + CH * LS;
  float* eP = sRk + CH * LS;
  float* brg = eP + 4 * DK;
  float* eGC = brg + 10 * DK;
  float* colp = eGC + DK;          // [4 row blocks][4 lane groups][DK]
  float* dgp = colp + 16 * DK;     // [DK][NSPLIT]
  int* split = reinterpret_cast<int*>(dgp + DK * NSPLIT);
  float* sdG = sLq;                // reused after the item loop

  const float* Hn = a.Hs + ch * DK * DV;
  const float* DHn = a.DH + ch * DK * DV;
  const float* Rn = a.Rs + ch * CH * DV;
  const float* DAqk = a.DAqk + ch * CH * CH;
  const float* DT = a.DT + ch * CH * CH;
  const float* DEg = a.DEg + ch * CH * DK;

  if (tid < 4) split[tid] = 0;
  chunk_cumsum<DK, NTHR>(a.g + kbase, rs, sG, tid, len);
  chunk_refs<DK, NTHR>(sG, eP, brg, eGC, split, tid);
  for (int e = tid; e < CH * DK / 4; e += NTHR) {
    const int r = e / (DK / 4), c4 = (e % (DK / 4)) * 4, i = r >> 4;
    const float4 kk = ld4z(a.k + kbase + r * rs + c4, r < len);
    const float4 bv = ld4z(a.b + kbase + r * rs + c4, r < len);
    const float4 qq = ld4z(a.q + kbase + r * rs + c4, r < len);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c4 + u;
      const float G = sG[r * LS + c];
      const float lf = expf(G - sG[left_row(split, i) * LS + c]);
      const float kv = f4at(kk, u);
      sLe[r * LS + c] = f4at(bv, u) * kv * lf;
      sLq[r * LS + c] = f4at(qq, u) * lf;
      sRk[r * LS + c] = kv * expf(sG[right_row(split, i) * LS + c] - G);
    }
  }
  // state part of d gamma_C: rowsum(dS_C * S0) per key channel
  for (int e = tid; e < DK * NSPLIT; e += NTHR) {
    const int c = e / NSPLIT, part = e % NSPLIT;
    float acc = 0.f;
    for (int v = part * (DV / NSPLIT); v < (part + 1) * (DV / NSPLIT); ++v)
      acc += DHn[c * DV + v] * Hn[c * DV + v];
    dgp[c * NSPLIT + part] = acc;
  }
  __syncthreads();

  float keep[IPW][4];
#pragma unroll
  for (int q = 0; q < IPW; ++q) {
    const int it = wave + q * NW;
    const int i = it / NCB, cb = it % NCB;
    const int c = 16 * cb + lr;
    f4 P1 = {0.f, 0.f, 0.f, 0.f}, P2 = P1, P3 = P1, dQs = P1, dKt = P1;
    const bool diag_direct = split[i] == kSplitNone, mid = split[i] == kSplitMiddle;
    // P1 / P2: sum_{s<=r} M[r][s] k_s exp(G_r - G_s), without the left factor
    for (int j = 0; j <= i; ++j) {
      if (j == i && diag_direct) break;
      const float d = j == i && mid ? 1.f : brg[pair_index(i, j) * DK + c];
      const float cl = j < i && split[j] == kSplitMiddle ? brg[pair_index(j, j) * DK + c] : 1.f;
      const float4 mt = ld4(DT + (16 * i + lr) * CH + 16 * j + 4 * lg);
      const float4 mq = ld4(DAqk + (16 * i + lr) * CH + 16 * j + 4 * lg);
      const int s0 = 16 * j + 4 * lg;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float bv = sRk[(s0 + u) * LS + c] * cl * d;
        P1 = mfma4(f4at(mt, u), bv, P1);
        P2 = mfma4(f4at(mq, u), bv, P2);
      }
    }
    // P3: sum_{r>=s} (dT[r][s] (b k)_r + dAqk[r][s] q_r) exp(G_r - G_s), without the right factor
    for (int i2 = i; i2 < 4; ++i2) {
      if (i2 == i && diag_direct) continue;
      const float d = i2 == i && mid ? 1.f : brg[pair_index(i2, i) * DK + c];
      const float cl = i2 > i && mid ? brg[pair_index(i, i) * DK + c] : 1.f;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 16 * i2 + 4 * lg + u;
        P3 = mfma4(DT[r * CH + 16 * i + lr], sLe[r * LS + c] * d * cl, P3);
        P3 = mfma4(DAqk[r * CH + 16 * i + lr], sLq[r * LS + c] * d * cl, P3);
      }
    }
    // dQs = dO S0^T and dKt = R dS_C^T
    {
      const float* pd = a.dout + vbase + (16 * i + lr) * rsv + 4 * lg;
      const bool pdin = 16 * i + lr < len;
      const float* pr = Rn + (16 * i + lr) * DV + 4 * lg;
      const float* ph = Hn + (16 * cb + lr) * DV + 4 * lg;
      const float* pdh = DHn + (16 * cb + lr) * DV + 4 * lg;
      for (int kk = 0; kk < DV; kk += 16) {
        const float4 x = ld4z(pd + kk, pdin), y = ld4(ph + kk);
        const float4 rr = ld4(pr + kk), z = ld4(pdh + kk);
        dQs = mfma4(x.x, y.x, dQs);
        dQs = mfma4(x.y, y.y, dQs);
        dQs = mfma4(x.z, y.z, dQs);
        dQs = mfma4(x.w, y.w, dQs);
        dKt = mfma4(rr.x, z.x, dKt);
        dKt = mfma4(rr.y, z.y, dKt);
        dKt = mfma4(rr.z, z.z, dKt);
        dKt = mfma4(rr.w, z.w, dKt);
      }
    }
    float tailpart = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 16 * i + 4 * lg + u;
      const float G = sG[r * LS + c];
      const float lf = expf(G - sG[left_row(split, i) * LS + c]);
      const float rf = expf(sG[right_row(split, i) * LS + c] - G);
      const float gam = expf(G);
      const float tail = expf(sG[(CH - 1) * LS + c] - G);
      const size_t off = kbase + r * rs + c, offo = kobase + r * rso + c;
      const bool rin = r < len;
      const float kv = ldz(a.k + off, rin), bv = ldz(a.b + off, rin), qv = ldz(a.q + off, rin);
      float dEg = DEg[r * DK + c] + lf * P1[u];
      float dq = a.scale * gam * dQs[u] + lf * P2[u];
      float dKg = rf * P3[u] + tail * dKt[u];
      if (diag_direct) {
        for (int s = 16 * i; s < 16 * i + 16; ++s) {
          const size_t so = kbase + s * rs + c;
          const float Gs = sG[s * LS + c];
          if (s <= r) {
            const float e = expf(G - Gs);   // r >= s: <= 1
            const float ks = ldz(a.k + so, s < len);
            if (s < r) dEg += DT[r * CH + s] * ks * e;
            dq += DAqk[r * CH + s] * ks * e;
          }
          if (s >= r) {
            const float e = expf(Gs - G);   // s >= r: <= 1
            if (s > r) dKg += DT[s * CH + r] * ldz(a.b + so, s < len) * ldz(a.k + so, s < len) * e;
            dKg += DAqk[s * CH + r] * ldz(a.q + so, s < len) * e;
          }
        }
      }
      if (rin) {
        a.db[offo] = dEg * kv;
        a.dk[offo] = dEg * bv + dKg;
        a.dq[offo] = dq;
      }
      keep[q][u] = dq * qv - dKg * kv + dEg * bv * kv;
      tailpart += dKt[u] * kv * tail;
    }
    colp[(i * 4 + lg) * DK + c] = tailpart;
  }
  __syncthreads();  // every read of sLq / sRk / sLe is done

#pragma unroll
  for (int q = 0; q < IPW; ++q) {
    const int it = wave + q * NW;
    const int i = it / NCB, cb = it % NCB;
#pragma unroll
    for (int u = 0; u < 4; ++u) sdG[(16 * i + 4 * lg + u) * LS + 16 * cb + lr] = keep[q][u];
  }
  __syncthreads();
  // d gamma_C * gamma_C joins the last row of dG
  for (int c = tid; c < DK; c += NTHR) {
    float st = 0.f;
    for (int p = 0; p < NSPLIT; ++p) st += dgp[c * NSPLIT + p];
    float tl = 0.f;
    for (int p = 0; p < 16; ++p) tl += colp[p * DK + c];
    sdG[(CH - 1) * LS + c] += eGC[c] * st + tl;
  }
  __syncthreads();
  // dlog_alpha_i = sum_{r >= i} dG_r (eq. eq_app_dg_reverse_cumsum), segmented scan
  {
    constexpr int NSEG = NTHR / DK;
    constexpr int RPS = CH / NSEG;
    const int c = tid % DK, seg = tid / DK;
    float run = 0.f;
    for (int r = (seg + 1) * RPS - 1; r >= seg * RPS; --r) {
      run += sdG[r * LS + c];
      sdG[r * LS + c] = run;
    }
    __syncthreads();
    float off = 0.f;
    for (int s = seg + 1; s < NSEG; ++s) off += sdG[(s * RPS) * LS + c];
    __syncthreads();
    for (int r = seg * RPS; r < (seg + 1) * RPS; ++r)
      if (r < len) a.dg[kobase + r * rso + c] = sdG[r * LS + c] + off;
  }
}

// ---------------------------------------------------------------------------
template <int DK, int DV>
hipError_t launch_bwd_state(const BwdStateArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((bwd_state_kernel<DK, DV>), dim3(state_slots<DV / 16>(a.nq)), dim3(512), 0, st, a);
  return hipGetLastError();
}

template <int DK, int DV>
hipError_t launch_bwd_wy(const BwdChunkArgs& a, int B, hipStream_t st) {
  constexpr size_t lds = sizeof(float) * (3 * CH * (DK + 4) + 2 * CH * LD64 + 15 * DK) + 4 * sizeof(int);
  hipError_t e = hipFuncSetAttribute((const void*)bwd_wy_kernel<DK, DV>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  dim3 grid(a.vl.ct0 ? a.vl.ncmax : a.NT, a.H, a.vl.ct0 ? 1 : B);
  hipLaunchKernelGGL((bwd_wy_kernel<DK, DV>), grid, dim3(512), lds, st, a);
  return hipGetLastError();
}

template <int DK, int DV>
hipError_t launch_bwd_intra(const BwdChunkArgs& a, int B, hipStream_t st) {
  constexpr int NSPLIT = 512 / DK;
  constexpr size_t lds = sizeof(float) * (4 * CH * (DK + 4) + 15 * DK + 16 * DK + DK * NSPLIT) + 4 * sizeof(int);
  hipError_t e = hipFuncSetAttribute((const void*)bwd_intra_kernel<DK, DV>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  dim3 grid(a.vl.ct0 ? a.vl.ncmax : a.NT, a.H, a.vl.ct0 ? 1 : B);
  hipLaunchKernelGGL((bwd_intra_kernel<DK, DV>), grid, dim3(512), lds, st, a);
  return hipGetLastError();
}

#define GDR2_INST_BWD(DK, DV)                                                          \
  template hipError_t launch_bwd_state<DK, DV>(const BwdStateArgs&, hipStream_t);      \
  template hipError_t launch_bwd_wy<DK, DV>(const BwdChunkArgs&, int, hipStream_t);    \
  template hipError_t launch_bwd_intra<DK, DV>(const BwdChunkArgs&, int, hipStream_t);

GDR2_INST_BWD(64, 64)
GDR2_INST_BWD(64, 128)
GDR2_INST_BWD(128, 64)
GDR2_INST_BWD(128, 128)

}  // namespace gdr2
