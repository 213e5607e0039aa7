// Grouped value heads (Sec. 3.5, App. C.1): q, k, the log-decay and b of a key
// head are shared by the G value heads of its group, so their gradients are
// the sums of the per-value-head contributions, which the fp32 chunk backward
// leaves in fp32 on the value-head axis (the bf16 one adds them up itself).
// One thread per 4 consecutive outputs; the G partials are added in a fixed
// order (deterministic).

#include "gdr2_kernels.hpp"

namespace gdr2 {

__global__ __launch_bounds__(256) void group_reduce_kernel(const float* __restrict__ P, float* __restrict__ out,
                                                           size_t n4, int Hk, int G, int D) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
    const size_t e = 4 * i;  // output element (r * Hk + h) * D + c
    const size_t c = e % D, rh = e / D;
    // partial of value head h * G + j at row r: ((r * Hk + h) * G + j) * D + c
    const float* src = P + rh * G * D + c;
    float4 acc = ld4(src);
    for (int j = 1; j < G; ++j) {
      const float4 x = ld4(src + (size_t)j * D);
      acc.x += x.x;
      acc.y += x.y;
      acc.z += x.z;
      acc.w += x.w;
    }
    *reinterpret_cast<float4*>(out + e) = acc;
  }
}

hipError_t launch_group_reduce(const float* P, float* out, size_t rows, int Hk, int G, int D, hipStream_t st) {
  const size_t n4 = rows * Hk * (size_t)D / 4;
  const size_t blocks = (n4 + 255) / 256;
  dim3 grid((unsigned)(blocks < 16384 ? blocks : 16384));
  if (n4 == 0) return hipSuccess;
  hipLaunchKernelGGL(group_reduce_kernel, grid, dim3(256), 0, st, P, out, n4, Hk, G, D);
  return hipGetLastError();
}

}  // namespace gdr2
