// Inter-chunk state scan of the bf16 path for few sequences (gfx950): the
// products of gdr2_scan_bf16.hip in the same order (the results are the same
// bits), one workgroup of 8 to 16 waves per (sequence, head) and 32-wide value slice.
//
// With 64-wide slices a scan of few heads leaves half the chip or more idle and
// is bound by the length of a step: 3.3 us, most of it LDS traffic (every
// operand block staged there, the state's fragments read by all waves) and one
// product after another in each wave.  Here a step's products have waves of their
// own, four for R, four for Q_g S and A_qk R (with the output), one per key block for
// the state: 16 or 12 waves with the output (Dk = 128, 64), 12 or 8 without.  Every
// operand block goes from memory straight into the registers of the one wave
// that multiplies it, and LDS holds S and R alone.  A step is 1.7 us on 64
// workgroups (16 heads, 16 chunks, 128 x 128: 28 us, the wide scan 52); what is left is
// LDS time of the products' S and R fragments and, with a workgroup on every CU, the
// memory's answer (3 us a step, where the wide kernel takes 4).  With the loads of R's and Q_g's waves in front of
// the barrier they wait at, a step was 2.1 us: the loads of all waves at once take
// 700 cycles to issue.
// scan_slices in gdr2_api.hip says when it is taken.
//
// Precision: as gdr2_scan_bf16.hip.

#include "gdr2_kernels.hpp"
#include "gdr2_bf16.hpp"

#include <type_traits>

namespace gdr2 {

// B fragment of S for Y S in the permuted key order of Y's fragments (stored [v][c])
__device__ __forceinline__ bf8 ld_perm(const __bf16* row, int k0, int g) {
  const bf4 a = *reinterpret_cast<const bf4*>(row + k0 + 4 * g);
  const bf4 b = *reinterpret_cast<const bf4*>(row + k0 + 16 + 4 * g);
  bf8 r;
  r[0] = a[0]; r[1] = a[1]; r[2] = a[2]; r[3] = a[3];
  r[4] = b[0]; r[5] = b[1]; r[6] = b[2]; r[7] = b[3];
  return r;
}

constexpr int nscan_threads(int dk, bool with_o) { return 64 * ((with_o ? 8 : 4) + dk / 16); }

template <int DK, int DV, bool WITH_O, bool STORE_H>
__global__ __launch_bounds__(nscan_threads(DK, WITH_O)) void nscan_bf16_kernel(ScanArgs a) {
  constexpr int DVS = 32, NS = DV / DVS, KS = DK / 32;
  constexpr int W_S = WITH_O ? 8 : 4;      // the first wave of the state's key blocks
  constexpr int LS = DK + 8, LR = 64 + 8;  // S, R rows (hi and lo planes) [v][c], [v][r]
  __shared__ __align__(16) __bf16 sSh[DVS * LS], sSl[DVS * LS];
  __shared__ __align__(16) __bf16 sRh[DVS * LR], sRl[DVS * LR];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int H = a.H;
  if (a.pick > 0 && !packed_narrow(a.vl, a.pick)) return;  // the wide kernel's
  // the slices of the G value heads that read one key head's tiles run on one XCD where the pairs divide
  int q, slice;
  {
    const int units = a.B * H / a.G, per = a.G * NS;
    int unit, rem;
    if ((units & 7) == 0) {
      const int j = blockIdx.x >> 3;
      unit = (j / per) * 8 + (blockIdx.x & 7);
      rem = j % per;
    } else {
      unit = blockIdx.x / per;
      rem = blockIdx.x % per;
    }
    const int HK = H / a.G;
    q = (unit / HK) * H + (unit % HK) * a.G + rem / NS;
    slice = rem % NS;
  }
  const int seq = scan_pair(a.vl, q, H), h = seq % H;  // (sequence, head) pair
  const ScanRange rng = scan_range(a.vl, seq, H, a.T, a.NT);
  const size_t chs = rng.chs;                          // value-head chunks: U, h, R
  const size_t chk = key_ch(a.vl, chs, H, a.G, a.NT);  // key-head chunks: Y, Q_g, A_qk, K_tail, gamma_C
  const int v0 = slice * DVS;
  const int i = wave & 3;  // row block of R's and O's waves

  // One role's walk over the chunks.  Op: a chunk's operands in registers, two
  // chunks of them; load fetches them, before and after do the work on the two
  // sides of a step's first barrier.  The loads go out where the role is idle, since
  // a wave's wait to issue them would lengthen the step: the state's waves (EARLY)
  // fetch the next chunk's while the others form R and Q_g S, the others the one
  // after it while the state is updated.  Past the end the last chunk's again, unused,
  // so that the same loads and stores go out every chunk and a wait for one chunk's
  // operands leaves the rest in flight.
  const auto walk = [&](auto op, auto early, auto&& load, auto&& before, auto&& after) {
    constexpr bool EARLY = decltype(early)::value;
    if (rng.c0 >= rng.c1) return;
    decltype(op) oa, ob;
    // the loads stay where they are put: the compiler would sink them past the barrier to their use
    const auto fetch = [&](decltype(op)& o, int n) {
      asm volatile("" ::: "memory");
      load(o, min(n, rng.c1 - 1));
      asm volatile("" ::: "memory");
    };
    const auto step = [&](decltype(op)& o, decltype(op)& other, int n) {
      if constexpr (EARLY) fetch(other, n + 1);
      before(o, n);
      __syncthreads();  // R is there, and nobody reads this chunk's S any more
      after(o, n);
      if constexpr (!EARLY) fetch(o, n + 2);
      __syncthreads();  // the next chunk's S is there, and nobody reads R any more
    };
    fetch(oa, rng.c0);
    if constexpr (!EARLY) fetch(ob, rng.c0 + 1);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the loop's waits then count its own loads and stores alone
    __syncthreads();
    int n = rng.c0;
    for (; n + 1 < rng.c1; n += 2) {  // one way through: the operands stay in their registers
      step(oa, ob, n);
      step(ob, oa, n + 1);
    }
    if (n < rng.c1) step(oa, ob, n);
  };
  const auto bf = [](u4v x) { return __builtin_bit_cast(bf8, x); };

  if (wave < 4) {  // ---- R = U - Y S, rows of block i
    struct Op {
      u4v y[KS], u[2];
    };
    f4 acc[2];
    walk(
        Op{}, std::false_type{},
        [&](Op& o, int n) {
          const unsigned char* Y = a.Y + (chk + n) * WsBf16::y(DK) + i * KS * 1024 + 16 * lane;
#pragma unroll
          for (int p = 0; p < KS; ++p) o.y[p] = ldg16(Y + 1024 * p);
          const float* U = a.U + (chs + n) * (WsBf16::u(DV) / 4) + ((size_t)(v0 / 16 * 4 + i) * 64 + lane) * 4;
          o.u[0] = ldg16(U);
          o.u[1] = ldg16(U + 4 * 64 * 4);
        },
        [&](Op& o, int n) {
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[t] = __builtin_bit_cast(f4, o.u[t]);
#pragma unroll
          for (int p = 0; p < KS; ++p) {
            const bf8 y = neg8(bf(o.y[p]));
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[t] = mma(y, ld_perm(sSh + (16 * t + r16) * LS, 32 * p, g), acc[t]);
          }
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const int ro = (16 * t + r16) * LR + 16 * i + 4 * g;
            st4split(sRh + ro, sRl + ro, acc[t]);
          }
        },
        [&](Op& o, int n) {
          if constexpr (STORE_H) {  // for the backward: the wave's 16 x 32 tile as one fp16 fragment block
            int sh[1];
            state_shifts<2>(acc, sh);
            const size_t blk = (chs + n) * (WsBf16::rs(DV) / 1024) + (size_t)i * (DV / 32) + v0 / 32;
            store_frag_f16(acc, sh[0], a.Rs + blk * 512, lane);
            a.Rsc[blk] = ldexpf(1.f, -sh[0]);  // every lane: no branch around the store
          }
        });
  } else if (WITH_O && wave < 8) {  // ---- O^T = S^T Q_g^T + R^T A_qk^T (lane: O[16 i + r16][16 t + 4 g + u])
    struct Op {
      u4v q[2 * KS];  // hi and lo
    };
    u4v x[4];  // A_qk's blocks, one chunk ahead (registers for two chunks are not there)
    f4 acc[2];
    __bf16* const oseq = reinterpret_cast<__bf16*>(a.o) + (rng.row0 + 16 * i + r16) * ((size_t)H * DV) +
                         (size_t)h * DV + v0 + 4 * g;
    const auto load_A = [&](int n) {
      // keys 32.. of query rows 0..31 are zero and not stored: the first block again, unused
      const unsigned char* A = a.Aqk + (chk + n) * WsBf16::aqk() + i * 4096 + 16 * lane;
      const int second = i >> 1 ? 2048 : 0;
      x[0] = ldg16(A);
      x[1] = ldg16(A + 1024);
      x[2] = ldg16(A + second);
      x[3] = ldg16(A + second + 1024);
    };
    if (rng.c0 < rng.c1) load_A(rng.c0);
    walk(
        Op{}, std::false_type{},
        [&](Op& o, int n) {
          const unsigned char* Q = a.Qg + (chk + n) * WsBf16::qg(DK) + i * KS * 2048 + 16 * lane;
#pragma unroll
          for (int p = 0; p < 2 * KS; ++p) o.q[p] = ldg16(Q + 1024 * p);
        },
        [&](Op& o, int n) {
          acc[0] = acc[1] = f4zero();
#pragma unroll
          for (int p = 0; p < KS; ++p) {
            const Fr qf = {bf(o.q[2 * p]), bf(o.q[2 * p + 1])};
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              const Fr sf = {ld8(sSh + (16 * t + r16) * LS + 32 * p + 8 * g),
                             ld8(sSl + (16 * t + r16) * LS + 32 * p + 8 * g)};
              acc[t] = mma3(sf, qf, acc[t]);
            }
          }
        },
        [&](Op& o, int n) {
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            if (kb > (i >> 1)) break;  // A_qk is causal
            const Fr af = {bf(x[2 * kb]), bf(x[2 * kb + 1])};
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              const Fr rf = {ld_perm(sRh + (16 * t + r16) * LR, 32 * kb, g),
                             ld_perm(sRl + (16 * t + r16) * LR, 32 * kb, g)};
              acc[t] = mma3(rf, af, acc[t]);
            }
          }
          asm volatile("" ::: "memory");
          load_A(min(n + 1, rng.c1 - 1));
          asm volatile("" ::: "memory");
          const int t0 = (n - rng.c0) * CH;  // the chunk's first token
          // rows past the chunk's end go over the slice's U tiles of this chunk,
          // which nobody reads any more: a store on every path
          __bf16* orow = oseq + t0 * (size_t)(H * DV);
          __bf16* urow = reinterpret_cast<__bf16*>(const_cast<float*>(a.U) + (chs + n) * (WsBf16::u(DV) / 4) +
                                                   ((size_t)(v0 / 16 * 4 + i) * 64 + lane) * 4);
          const bool in = t0 + 16 * i + r16 < rng.rows;
#pragma unroll
          for (int t = 0; t < 2; ++t)
            st4(in ? orow + 16 * t : urow + 4 * t, a.scale * acc[t][0], a.scale * acc[t][1], a.scale * acc[t][2],
                a.scale * acc[t][3]);
        });
  } else {  // ---- S <- Diag(gamma_C) S + Ktail^T R, key block cs
    struct Op {
      u4v k[4];  // hi and lo
      f4 gm;     // gamma_C of channels 16 cs + 4 g ..
    };
    const int cs = wave - W_S;
    f4 st[2] = {f4zero(), f4zero()};  // S[16 cs + 4 g + u][v0 + 16 t + r16]
    const size_t so = ((size_t)seq * DK + 16 * cs + 4 * g) * DV + v0 + r16;
    const auto put_S = [&] {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int o = (16 * t + r16) * LS + 16 * cs + 4 * g;
        st4split(sSh + o, sSl + o, st[t]);
      }
    };
    if (a.S0 != nullptr) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) st[t][u] = a.S0[so + (size_t)u * DV + 16 * t];
    }
    put_S();
    walk(
        Op{}, std::true_type{},
        [&](Op& o, int n) {
          const unsigned char* K = a.KtT + (chk + n) * WsBf16::ktt(DK) + cs * 4096 + 16 * lane;
#pragma unroll
          for (int j = 0; j < 4; ++j) o.k[j] = ldg16(K + 1024 * j);
          o.gm = *reinterpret_cast<const f4*>(a.GC + (chk + n) * (WsBf16::gc(DK) / 4) + 16 * cs + 4 * g);
        },
        [&](Op& o, int n) {
          if constexpr (STORE_H) {  // the chunk-start state for the backward, fp16 with its block scale
            int sh[1];
            state_shifts<2>(st, sh);
            store_state_f16<2>(st, sh, a.Hs + ((chs + n) * DK + 16 * cs) * DV + v0, DV,
                               a.Hsc + (chs + n) * (WsBf16::hsc(DK, DV) / 4) + cs * (DV / 32) + v0 / 32, lane);
          }
        },
        [&](Op& o, int n) {
#pragma unroll
          for (int t = 0; t < 2; ++t) st[t] *= o.gm;
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            const Fr kf = {bf(o.k[2 * kb]), bf(o.k[2 * kb + 1])};
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              const Fr rf = {ld8(sRh + (16 * t + r16) * LR + 32 * kb + 8 * g),
                             ld8(sRl + (16 * t + r16) * LR + 32 * kb + 8 * g)};
              st[t] = mma3(kf, rf, st[t]);
            }
          }
          put_S();
        });
    if (a.ST != nullptr) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) a.ST[so + (size_t)u * DV + 16 * t] = st[t][u];
    }
  }
}

template <int DK, int DV, bool WITH_O, bool STORE_H>
hipError_t launch_nscan_bf16(const ScanArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((nscan_bf16_kernel<DK, DV, WITH_O, STORE_H>), dim3(a.B * a.H * (DV / 32)), dim3(nscan_threads(DK, WITH_O)),
                     0, st, a);
  return hipGetLastError();
}

#define GDR2_INST_NSCAN(DK, DV)                                                             \
  template hipError_t launch_nscan_bf16<DK, DV, true, false>(const ScanArgs&, hipStream_t); \
  template hipError_t launch_nscan_bf16<DK, DV, false, true>(const ScanArgs&, hipStream_t); \
  template hipError_t launch_nscan_bf16<DK, DV, true, true>(const ScanArgs&, hipStream_t);

GDR2_INST_NSCAN(64, 64)
GDR2_INST_NSCAN(64, 128)
GDR2_INST_NSCAN(128, 64)
GDR2_INST_NSCAN(128, 128)

}  // namespace gdr2
