// silu(z) = z / (1 + exp(-z)) and its derivative as the network kernels evaluate them, with the IEEE
// quotient.  Host and device, so that the quotient's steps can be compared with the division on a CPU.
#pragma once

#include <hip/hip_runtime.h>

namespace kpsi {
namespace nn {

// q = z / d for the special operands (d infinite, z or d not a number, z infinite), else q.
__host__ __device__ __forceinline__ float fix_quotient(float q, float d, float z) {
#if __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_div_fixupf(q, d, z);
#else
  const bool plain = __builtin_isfinite(z) && __builtin_isfinite(d) && z != 0.0f && d != 0.0f;
  return plain ? q : z / d;
#endif
}
// 1/d from an estimate y0 within one unit in the last place: one Newton step, correctly rounded for all
// but a few d, with an error below that of the estimate by a factor of 2^23.
__host__ __device__ __forceinline__ float newton_rcp(float d, float y0) {
  return __builtin_fmaf(__builtin_fmaf(-d, y0, 1.0f), y0, y0);
}
// z / d from y = newton_rcp(d): one correction of z y by its exact remainder gives the IEEE quotient for
// 1 <= d <= 2^126 (these are the steps of the division without its scaling of extreme operands).  For d
// between 2^126 and infinity the estimate of 1/d can be a denormal that the hardware returns as zero:
// the quotient is then zero in place of at most |z| 2^-126 in size (of silu: 1e-36).
__host__ __device__ __forceinline__ float quotient(float z, float d, float y) {
  const float q = z * y;
  return fix_quotient(__builtin_fmaf(__builtin_fmaf(-d, q, z), y, q), d, z);
}
// silu and silu' = s (1 + z (1 - s)) with s = 1/d, d = 1 + exp(-z), from the estimate y0 of 1/d
__host__ __device__ __forceinline__ float silu_of(float z, float d, float y0) { return quotient(z, d, newton_rcp(d, y0)); }
__host__ __device__ __forceinline__ void silu_both_of(float z, float d, float y0, float& sl, float& ds) {
  const float s = quotient(1.0f, d, newton_rcp(d, y0));
  sl = quotient(z, d, s);
  ds = s * __builtin_fmaf(z, 1.0f - s, 1.0f);
}

}  // namespace nn
}  // namespace kpsi
