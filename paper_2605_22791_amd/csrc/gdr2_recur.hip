// Recurrent (token-by-token) GDR-2 forward for decoding, App. C.5.  Per token
//     Sbar = Diag(exp g) S,  r = Sbar^T (b*k),  S = Sbar + k (w*v - r)^T,
//     o    = scale * S^T q = scale * (Sbar^T q + (w*v - r) (k . q)),
// for every (batch, head), or (sequence, head) of a packed batch (App. C.6: the
// same cumulative-length layout as the chunk kernels).  The fp32 state stays in
// registers for all T tokens of the call: S is read and written once.
//
// One token (recurrent_one_kernel) is the state's way through memory and back.
// A workgroup takes a (batch, head) and each of its four waves a quarter of the
// rows, one contiguous run, a whole kilobyte an access; the rows' sums meet in
// LDS behind the only barrier (rows_tokens).  B = 256, 16 heads, 128 x 128 (545 MB):
// 103 us, 5.2 TB/s (a large copy runs at 5.1); 108 with five barriers and a wave's
// accesses in two runs 8 KB apart, 111 with a wave per 32 columns.  B = 64
// (within the Infinity Cache): 22.2, 23.1 and 24.4 us.
//
// Several tokens (recurrent_kernel) are bound by a token's latency, or with many
// sequences by the vector instructions (four per state element).  The columns
// of S never meet, so a wave takes CW value columns over all rows and needs
// nothing from another: the sums over rows are DPP steps inside 8 or 16 lanes,
// the key-side factors (exp g, b*k, q, k) are formed once per wave and handed
// round through the wave's own LDS a token ahead, and the token after that is
// on its way from memory: no barrier anywhere.  Two sequences x 16 heads x 128
// x 128: 0.65 us a token, 1.48 with a workgroup per head and five barriers a
// token; 64 sequences of 65 tokens 188 us, 295 before; a packed batch of 48
// sequences of 1 to 16 tokens from raw projections 32.5 us a call, 48.5 before.
//
// A few tokens of many sequences are both: a sequence of up to kRowsTokens goes by
// rows with a barrier a token, whatever its neighbours in a packed batch do (the
// workgroup sees its count).  16 heads, 128 x 128, by columns / by rows: 256 sequences
// of 2 tokens 94.2 / 87.4 us, of 4 107.8 / 100.6, of 8 143 / 138; 64 of 4 30.3 / 28.9, of 6
// 33.2 / 33.6, of 8 37.3 / 38.7; a packed batch of 256 single tokens 89.3 / 81.1.
//
// Fused input stage (a.st.a_log set; App. C.1, App. D.2): q and k are the raw
// projections, L2-normalised per token in fp32 and rounded to the operand
// dtype, as the chunk path does; the log-decay is -exp(a) softplus(f + delta)
// from the decay projection f.

#include "gdr2_kernels.hpp"
#include "gdr2_bf16.hpp"

namespace gdr2 {

// x rounded to the operand dtype (nearest, ties to even)
template <typename TIn>
__device__ __forceinline__ float round_as(float x);
template <>
__device__ __forceinline__ float round_as<float>(float x) { return x; }
template <>
__device__ __forceinline__ float round_as<bf16_t>(float x) { return (float)(__bf16)x; }

// N consecutive values of one token, raw until used (a conversion at the load
// would wait for it there)
template <typename TIn, int N>
struct Raw;
template <>
struct Raw<bf16_t, 1> {
  uint16_t u;
  __device__ __forceinline__ void load(const bf16_t* p) { u = p->x; }
  __device__ __forceinline__ float at(int) const { return __uint_as_float((uint32_t)u << 16); }
};
template <>
struct Raw<bf16_t, 2> {
  uint32_t u;
  __device__ __forceinline__ void load(const bf16_t* p) { u = *reinterpret_cast<const uint32_t*>(p); }
  __device__ __forceinline__ float at(int i) const { return __uint_as_float(i == 0 ? u << 16 : u & 0xffff0000u); }
};
template <>
struct Raw<bf16_t, 4> {
  uint2 u;
  __device__ __forceinline__ void load(const bf16_t* p) { u = *reinterpret_cast<const uint2*>(p); }
  __device__ __forceinline__ float at(int i) const {
    const uint32_t x = i < 2 ? u.x : u.y;
    return __uint_as_float((i & 1) == 0 ? x << 16 : x & 0xffff0000u);
  }
};
template <>
struct Raw<float, 1> {
  float u;
  __device__ __forceinline__ void load(const float* p) { u = *p; }
  __device__ __forceinline__ float at(int) const { return u; }
};
template <>
struct Raw<float, 2> {
  float2 u;
  __device__ __forceinline__ void load(const float* p) { u = *reinterpret_cast<const float2*>(p); }
  __device__ __forceinline__ float at(int i) const { return i == 0 ? u.x : u.y; }
};
template <>
struct Raw<float, 4> {
  f4 u;
  __device__ __forceinline__ void load(const float* p) { u = *reinterpret_cast<const f4*>(p); }
  __device__ __forceinline__ float at(int i) const { return u[i]; }
};
__device__ __forceinline__ void put4(float* p, const float (&x)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(x[0], x[1], x[2], x[3]);
}
__device__ __forceinline__ void put4(bf16_t* p, const float (&x)[4]) {
  st4(reinterpret_cast<__bf16*>(p), x[0], x[1], x[2], x[3]);
}
// sum over the wave's 64 lanes
__device__ __forceinline__ float wave_sum(float x, int lane) {
  x = row_sum(x);
  x += row_partner16(x, (lane & 16) != 0);
  return x + row_partner32(x, lane >= 32);
}

// A wave's part of a token: NK = DK / 64 key-side rows and four value columns per lane
template <int DK, typename TIn, bool FUSED>
struct Token {
  static constexpr int NK = DK / 64;
  Raw<TIn, NK> q, k, b;
  Raw<float, NK> g;
  Raw<TIn, 4> v, w;
  // ok, ov: element offsets of the lane's rows and columns
  __device__ __forceinline__ void load(const RecurArgs<TIn>& a, size_t ok, size_t ov) {
    k.load(a.k + ok);
    q.load(a.q + ok);
    b.load(a.b + ok);
    g.load(a.g + ok);
    v.load(a.v + ov);
    w.load(a.w + ov);
  }
  // put(row, exp g, b k, q, k) for the lane's rows NK lane ..; returns k . q (all lanes)
  template <class Put>
  __device__ __forceinline__ float factors(const Raw<float, NK>& dl, float Adec, float eps, int lane, Put&& put) const {
    float kv[NK], qv[NK];
#pragma unroll
    for (int j = 0; j < NK; ++j) kv[j] = k.at(j), qv[j] = q.at(j);
    if constexpr (FUSED) {
      // y = x (sum x^2 + eps)^(-1/2) in the operand dtype
      float kk = 0.f, qq = 0.f;
#pragma unroll
      for (int j = 0; j < NK; ++j) kk += kv[j] * kv[j], qq += qv[j] * qv[j];
      const float rk = inv_norm(wave_sum(kk, lane), eps), rq = inv_norm(wave_sum(qq, lane), eps);
#pragma unroll
      for (int j = 0; j < NK; ++j) kv[j] = round_as<TIn>(kv[j] * rk), qv[j] = round_as<TIn>(qv[j] * rq);
    }
    float kq = 0.f;
#pragma unroll
    for (int j = 0; j < NK; ++j) {
      const float al = expf(FUSED ? decay_act(g.at(j), dl.at(j), Adec) : g.at(j));
      put(NK * lane + j, al, b.at(j) * kv[j], qv[j], kv[j]);
      kq += kv[j] * qv[j];
    }
    return wave_sum(kq, lane);
  }
};

constexpr int kRowsTokens = 4;

// ---- a workgroup per (sequence, head): one token, or a few ------------------
// n tokens from `row` on of pair seq; MULTI: n may be more than one.  smem: rows_lds bytes
template <int DK, int DV, int NW, bool MULTI>
constexpr int rows_lds() { return 4 * (NW * 4 * DK + (MULTI ? 2 : 1) * 2 * NW * DV); }
template <int DK, int DV, typename TIn, bool FUSED, int NW, bool MULTI>
__device__ __forceinline__ void rows_tokens(const RecurArgs<TIn>& a, int seq, size_t row, int n, unsigned char* smem) {
  constexpr int RW = DK / NW;               // rows per wave
  constexpr int CG = DV / 4, RG = 64 / CG;  // the lanes' column and row groups
  constexpr int RPL = RW / RG;              // rows per lane: RW wave + RG i + rg
  static_assert(RG == 2 || RG == 4, "row groups are halves or quarters of a wave");
  float(*sF)[4 * DK] = reinterpret_cast<float(*)[4 * DK]>(smem);
  // the waves' sums, by token parity: one barrier a token
  float(*sSum)[2][NW][DV] = reinterpret_cast<float(*)[2][NW][DV]>(smem + 4 * NW * 4 * DK);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = seq % a.H;
  const int cg = lane % CG, rg = lane / CG;
  const int HK = a.H / a.G, hk = h / a.G;  // key side (q, k, g, b) on the H / G key heads

  using Tok = Token<DK, TIn, FUSED>;
  const size_t ks = (size_t)HK * DK, vs = (size_t)a.H * DV;  // token strides
  const size_t ok = (row * HK + hk) * DK + Tok::NK * lane;
  const size_t ov = (MULTI ? row * a.H + h : (size_t)seq) * DV + 4 * cg;
  Tok x;
  x.load(a, ok, ov);
  Raw<float, Tok::NK> dl{};
  float Adec = 0.f;
  if constexpr (FUSED) {
    dl.load(a.st.delta + (size_t)hk * DK + Tok::NK * lane);
    Adec = expf(a.st.a_log[hk]);
  }
  float* const Sg = a.S + (size_t)seq * DK * DV + (size_t)RW * DV * wave;
  unsigned ls = rg * DV + 4 * cg;
  f4 S[RPL];
#pragma unroll
  for (int i = 0; i < RPL; ++i) S[i] = *reinterpret_cast<const f4*>(Sg + (ls + RG * i * DV));

  float* const F = sF[wave];
  for (int t = 0; t < (MULTI ? n : 1); ++t) {
    const float kq = x.factors(dl, Adec, a.st.eps, lane, [&](int row, float al, float e, float q, float k) {
      *reinterpret_cast<float4*>(F + 4 * row) = make_float4(al, e, q, k);
    });
    float z[4];
    if constexpr (MULTI) {
#pragma unroll
      for (int u = 0; u < 4; ++u) z[u] = x.v.at(u) * x.w.at(u);
      // the next token (past the last one the last again)
      const size_t d = (size_t)min(t + 1, n - 1);
      x.load(a, ok + d * ks, ov + d * vs);
    }
    __builtin_amdgcn_wave_barrier();
    const float* Fl = F + 4 * (RW * wave + rg);
    f4 pr = f4zero(), pp = f4zero();
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const float4 f = *reinterpret_cast<const float4*>(Fl + 4 * RG * i);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        S[i][u] *= f.x;
        pr[u] += S[i][u] * f.y;
        pp[u] += S[i][u] * f.z;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if constexpr (RG == 4) {
        pr[u] += row_partner16(pr[u], (lane & 16) != 0);
        pp[u] += row_partner16(pp[u], (lane & 16) != 0);
      }
      pr[u] += row_partner32(pr[u], lane >= 32);
      pp[u] += row_partner32(pp[u], lane >= 32);
    }
    float(*sum)[NW][DV] = sSum[MULTI ? t & 1 : 0];
    if (rg == 0) {
      *reinterpret_cast<f4*>(&sum[0][wave][4 * cg]) = pr;
      *reinterpret_cast<f4*>(&sum[1][wave][4 * cg]) = pp;
    }
    __syncthreads();
    float res[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float r = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) r += sum[0][w][4 * cg + u];
      res[u] = (MULTI ? z[u] : x.v.at(u) * x.w.at(u)) - r;
    }
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const float k = Fl[4 * RG * i + 3];
#pragma unroll
      for (int u = 0; u < 4; ++u) S[i][u] += k * res[u];
    }
    if constexpr (!MULTI) {
      asm volatile("" : "+v"(ls));  // addresses anew: kept from the loads they would hold registers
#pragma unroll
      for (int i = 0; i < RPL; ++i) *reinterpret_cast<f4*>(Sg + (ls + RG * i * DV)) = S[i];
    }
    if (wave == 0 && rg == 0) {
      float o4[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float p = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) p += sum[1][w][4 * cg + u];
        o4[u] = a.scale * (p + res[u] * kq);
      }
      put4(a.o + ov + (size_t)t * vs, o4);
    }
    __builtin_amdgcn_wave_barrier();
  }
  if constexpr (MULTI) {
    asm volatile("" : "+v"(ls));
#pragma unroll
    for (int i = 0; i < RPL; ++i) *reinterpret_cast<f4*>(Sg + (ls + RG * i * DV)) = S[i];
  }
}

template <int DK, int DV, typename TIn, bool FUSED>
__global__ __launch_bounds__(256) void recurrent_one_kernel(RecurArgs<TIn> a) {
  __shared__ __align__(16) unsigned char smem[rows_lds<DK, DV, 4, false>()];
  const int seq = blockIdx.x;  // signed, as the remainder in rows_tokens: one division for both
  rows_tokens<DK, DV, TIn, FUSED, 4, false>(a, seq, seq / a.H, 1, smem);
}

// ---- any number of tokens --------------------------------------------------
// ROWS > 0 (a head's waves in one workgroup): a sequence of at most so many tokens
// goes by rows instead (see the top).
template <int DK, int DV, typename TIn, bool FUSED, int CW, int NW, int ROWS = 0>
__global__ __launch_bounds__(64 * NW) void recurrent_kernel(RecurArgs<TIn> a) {
  constexpr int NSL = DV / CW;              // column slices, one per wave
  constexpr int CG = CW / 4, RG = 64 / CG;  // the lanes' column and row groups
  constexpr int RPL = DK / RG;              // rows per lane: RG i + rg
  static_assert(RG == 8 || RG == 16, "row sums within 8 or 16 lanes");
  // floats of one row group's factors: (exp g, b k, q, -) per row, then k of its rows; padded
  constexpr int RGS = 5 * RPL + 4;
  constexpr int LDS_COLS = 4 * NW * 2 * RG * RGS, LDS_ROWS = ROWS > 0 ? rows_lds<DK, DV, NW, true>() : 0;
  __shared__ __align__(16) unsigned char smem[LDS_COLS > LDS_ROWS ? LDS_COLS : LDS_ROWS];
  float(*sF)[2][RG * RGS] = reinterpret_cast<float(*)[2][RG * RGS]>(smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = blockIdx.x * NW + wave;
  const int seq = unit / NSL, v0 = CW * (unit % NSL);
  const int bb = seq / a.H, h = seq % a.H;
  const int rg = lane % RG, cg = lane / RG;
  const int T = a.T, H = a.H;

  // tokens of this sequence: bb's T tokens, or cu[bb] .. cu[bb+1) of a packed batch (clamped into [0, T])
  int t0 = 0, t1 = T;
  size_t rbase = (size_t)bb * T;
  if (a.cu != nullptr) {
    t0 = min(max(a.cu[bb], 0), T);
    t1 = min(max(a.cu[bb + 1], t0), T);
    rbase = 0;
  }
  if (t0 >= t1) return;  // no token: the state stays as it is
  if constexpr (ROWS > 0) {
    static_assert(NW * CW == DV, "a workgroup has a whole head");
    if (t1 - t0 <= ROWS) return rows_tokens<DK, DV, TIn, FUSED, NW, true>(a, seq, rbase + t0, t1 - t0, smem);
  }
  const int HK = H / a.G, hk = h / a.G;  // key side (q, k, g, b) on the H / G key heads
  const size_t ks = (size_t)HK * DK, vs = (size_t)H * DV;  // token strides
  using Tok = Token<DK, TIn, FUSED>;
  const size_t ok = (rbase + t0) * ks + (size_t)hk * DK + Tok::NK * lane;
  const size_t ov = (rbase + t0) * vs + (size_t)h * DV + v0 + 4 * cg;

  // Past the last token the last one is read again, so that every path issues
  // the same loads (waits count them in issue order).
  Tok x;
  const auto fetch = [&](int t) {
    const size_t d = (size_t)(min(t, t1 - 1) - t0);
    x.load(a, ok + d * ks, ov + d * vs);
  };
  fetch(t0);
  Raw<float, Tok::NK> dl{};
  float Adec = 0.f;
  if constexpr (FUSED) {
    dl.load(a.st.delta + (size_t)hk * DK + Tok::NK * lane);
    Adec = expf(a.st.a_log[hk]);
  }
  float* const Sg = a.S + (size_t)seq * DK * DV + v0;
  unsigned ls = rg * DV + 4 * cg;
  f4 S[RPL];
#pragma unroll
  for (int i = 0; i < RPL; ++i) S[i] = *reinterpret_cast<const f4*>(Sg + (ls + RG * i * DV));

  // the fetched token's factors into F for the lanes that hold its rows; its k . q and w * v
  const auto stage = [&](float* F, float& kq, float (&z)[4]) {
    kq = x.factors(dl, Adec, a.st.eps, lane, [&](int row, float al, float e, float q, float k) {
      float* const f = F + (row % RG) * RGS;
      *reinterpret_cast<float4*>(f + 4 * (row / RG)) = make_float4(al, e, q, 0.f);
      f[4 * RPL + row / RG] = k;
    });
#pragma unroll
    for (int u = 0; u < 4; ++u) z[u] = x.v.at(u) * x.w.at(u);
  };
  float kq, z[4];
  stage(sF[wave][0], kq, z);
  fetch(t0 + 1);
  // the state has arrived: later waits are for tokens' operands alone
#pragma unroll
  for (int i = 0; i < RPL; ++i) asm volatile("" : "+v"(S[i]));

  // Token t computes from one half of sF while the next one's factors go into the
  // other and the one after that is on its way from memory.
  for (int t = t0, p = 0; t < t1; ++t, p ^= 1) {
    const float* F = sF[wave][p] + rg * RGS;
    float kqn, zn[4];
    __builtin_amdgcn_wave_barrier();
    stage(sF[wave][p ^ 1], kqn, zn);
    fetch(t + 2);
    __builtin_amdgcn_wave_barrier();

    // decay, the two sums over the rows, update.  Four rows' factors at a time,
    // the next four in flight: all at once would take 64 registers
    float pr[4] = {0.f, 0.f, 0.f, 0.f}, pp[4] = {0.f, 0.f, 0.f, 0.f};
    float4 f[2][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) f[0][j] = *reinterpret_cast<const float4*>(F + 4 * j);
#pragma unroll
    for (int i4 = 0; i4 < RPL / 4; ++i4) {
      if (i4 + 1 < RPL / 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) f[(i4 + 1) & 1][j] = *reinterpret_cast<const float4*>(F + 4 * (4 * i4 + 4 + j));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = 4 * i4 + j;
        const float4 y = f[i4 & 1][j];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          S[i][u] *= y.x;
          pr[u] += S[i][u] * y.y;
          pp[u] += S[i][u] * y.z;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    f4 kr[RPL / 4];
#pragma unroll
    for (int j = 0; j < RPL / 4; ++j) kr[j] = *reinterpret_cast<const f4*>(F + 4 * RPL + 4 * j);
    float res[4], o4[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      res[u] = z[u] - row_sum<RG == 8>(pr[u]);
      o4[u] = a.scale * (row_sum<RG == 8>(pp[u]) + res[u] * kq);
    }
#pragma unroll
    for (int i = 0; i < RPL; ++i)
#pragma unroll
      for (int u = 0; u < 4; ++u) S[i][u] += kr[i / 4][i % 4] * res[u];
    if (rg == 0) put4(a.o + ov + (size_t)(t - t0) * vs, o4);
    kq = kqn;
#pragma unroll
    for (int u = 0; u < 4; ++u) z[u] = zn[u];
  }
  asm volatile("" : "+v"(ls));  // as in rows_tokens
#pragma unroll
  for (int i = 0; i < RPL; ++i) *reinterpret_cast<f4*>(Sg + (ls + RG * i * DV)) = S[i];
}

template <int DK, int DV, typename TIn, bool FUSED>
hipError_t launch_recurrent_t(const RecurArgs<TIn>& a, int B, hipStream_t st) {
  const unsigned seqs = (unsigned)B * a.H;
  if (a.cu == nullptr && a.T == 1) {
    hipLaunchKernelGGL((recurrent_one_kernel<DK, DV, TIn, FUSED>), dim3(seqs), dim3(256), 0, st, a);
  } else if (seqs * (DV / 32) <= 1024) {
    // No more 32-column waves than SIMDs: 16 columns a wave halve a token's
    // instructions (17 tokens, 16 heads, 128 x 128: 2 sequences 17.3 against 19.9
    // us, 16 sequences 24.5 against 25.7; 32 sequences 38.3 against 34.9).  Each in
    // a workgroup of its own while they still have a SIMD each, else a head's
    // together, whose token rows then come from one L1 (16 sequences 27.8 apart).
    constexpr int NW = DV / 16;
    if (seqs * NW <= 1024)
      hipLaunchKernelGGL((recurrent_kernel<DK, DV, TIn, FUSED, 16, 1>), dim3(seqs * NW), dim3(64), 0, st, a);
    else
      hipLaunchKernelGGL((recurrent_kernel<DK, DV, TIn, FUSED, 16, NW>), dim3(seqs), dim3(64 * NW), 0, st, a);
  } else {
    constexpr int NW = DV / 32;
    if (a.cu == nullptr && a.T > kRowsTokens)
      hipLaunchKernelGGL((recurrent_kernel<DK, DV, TIn, FUSED, 32, NW>), dim3(seqs), dim3(64 * NW), 0, st, a);
    else
      hipLaunchKernelGGL((recurrent_kernel<DK, DV, TIn, FUSED, 32, NW, kRowsTokens>), dim3(seqs), dim3(64 * NW), 0, st,
                         a);
  }
  return hipGetLastError();
}

template <int DK, int DV, typename TIn>
hipError_t launch_recurrent(const RecurArgs<TIn>& a, int B, hipStream_t st) {
  return a.st.a_log != nullptr ? launch_recurrent_t<DK, DV, TIn, true>(a, B, st)
                               : launch_recurrent_t<DK, DV, TIn, false>(a, B, st);
}

#define GDR2_INST_REC(DK, DV, TIN) \
  template hipError_t launch_recurrent<DK, DV, TIN>(const RecurArgs<TIN>&, int, hipStream_t);

GDR2_INST_REC(64, 64, float)
GDR2_INST_REC(64, 128, float)
GDR2_INST_REC(128, 64, float)
GDR2_INST_REC(128, 128, float)
GDR2_INST_REC(64, 64, bf16_t)
GDR2_INST_REC(64, 128, bf16_t)
GDR2_INST_REC(128, 64, bf16_t)
GDR2_INST_REC(128, 128, bf16_t)

}  // namespace gdr2
