// Device arithmetic shared by the per-event kernel and the interference-matrix kernel: the
// hardware reciprocal and reciprocal square root (refined by Newton steps in FP64), the
// normalised Blatt-Weisskopf polynomials, and the angular functions of the K* helicity angle
// (Eq. 4: the small-d functions d^J_{00}, d^J_{10} without their constant factors).  One copy, so
// both kernels evaluate the same lineshape and angular polynomials.  Also the opaque kernel-argument pointer both use in their event loops.
#pragma once

#include <hip/hip_runtime.h>

namespace kpsi {

// 1/x and 1/sqrt(x): the FP32 forms are the hardware instructions (about 1 ulp); the FP64
// forms refine the hardware estimate with two Newton steps to full double precision.
__device__ __forceinline__ float rcp_(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float rsq_(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq_(double x) {
  double r = __builtin_amdgcn_rsq(x);
  double h = 0.5 * x;
  double e = __builtin_fma(-h * r, r, 0.5);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-h * r, r, 0.5);
  return __builtin_fma(r, e, r);
}
__device__ __forceinline__ float sqrt_(float x) { return __builtin_sqrtf(x); }
__device__ __forceinline__ double sqrt_(double x) { return __builtin_sqrt(x); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// M^2 - s, the real part of a Breit-Wigner denominator (Eq. 2).  In FP32 the squared mass is
// carried as M2 plus its rounding remainder M2lo: near a narrow pole M^2 - s is far smaller than
// M^2, and the rounding of M^2 alone would move the pole of every event by the same amount (a
// shift of 0.5 ulp of M^2 is 1e-3 of the statistical error of a K*(892) mass at 3e6 events).
template <typename T> __device__ __forceinline__ T pole_gap(T M2, T M2lo, T s) {
  if constexpr (sizeof(T) == sizeof(float)) return (M2 - s) + M2lo;
  else return M2 - s;
}

// Blatt-Weisskopf polynomial B_L(z), z = (r p)^2, in Horner form: the barrier factor of
// Eq. 2-3 is F_L = sqrt(B_L(z0) / B_L(z)).
template <int L, typename T> __device__ __forceinline__ T bpoly(T z) {
  if constexpr (L == 0) return T(1);
  else if constexpr (L == 1) return T(1) + z;
  else if constexpr (L == 2) return T(9) + z * (T(3) + z);
  else if constexpr (L == 3) return T(225) + z * (T(45) + z * (T(6) + z));
  else return T(11025) + z * (T(1575) + z * (T(135) + z * (T(10) + z)));
}
// Lowest orbital momentum of B -> J/psi K* for a K* of spin J (text below Eq. 3).
template <int J> struct LBof { static constexpr int v = (J == 0) ? 1 : J - 1; };

template <typename T, int n> __device__ __forceinline__ T ipow(T x) {
  T r = T(1);
#pragma unroll
  for (int i = 0; i < n; ++i) r *= x;
  return r;
}

// M^2 - m^2 of a K* from m itself: one fused step leaves only the rounding of the result.
template <typename T> __device__ __forceinline__ T pole_gap_m(T M2, T M2lo, T m) {
  if constexpr (sizeof(T) == sizeof(float)) return fma_(-m, m, M2) + M2lo;
  else return fma_(-m, m, M2);
}

// The kernels' angular functions: d^J_{00}(theta_K) = E0<J> ang0<J> and d^J_{10}(theta_K) / sqrt2 = E1<J> sin
// ang1<J>, with the constants folded into the couplings on the host.  (Each is one rounded number: as products
// of rounded roots they would shift the lambda = +-1 terms of every event by up to 2^-52.)
template <int J> struct AngScale;
template <> struct AngScale<0> { static constexpr double E0 = 1.0, E1 = 0.0; };
template <> struct AngScale<1> { static constexpr double E0 = 1.0, E1 = -0.5; };
template <> struct AngScale<2> { static constexpr double E0 = 1.0, E1 = -0.86602540378443864676; };     // sqrt(3)/2
template <> struct AngScale<3> { static constexpr double E0 = 1.0, E1 = -0.30618621784789726227; };     // sqrt(6)/8
template <> struct AngScale<4> { static constexpr double E0 = 0.125, E1 = -0.39528470752104741649; };   // sqrt(10)/8
template <int J, typename T> __device__ __forceinline__ T ang0(T c) {
  if constexpr (J == 0) return T(1);
  else if constexpr (J == 1) return c;
  else if constexpr (J == 2) return fma_(T(1.5) * c, c, T(-0.5));
  else if constexpr (J == 3) return c * fma_(T(2.5) * c, c, T(-1.5));
  else { const T c2 = c * c; return fma_(c2, fma_(T(35), c2, T(-30)), T(3)); }
}
template <int J, typename T> __device__ __forceinline__ T ang1(T c) {
  if constexpr (J <= 1) return T(1);
  else if constexpr (J == 2) return c;
  else if constexpr (J == 3) return fma_(T(5) * c, c, T(-1));
  else return c * fma_(T(7) * c, c, T(-3));
}

// Opaque copy of a pointer to uniform kernel-argument data.  Re-deriving it inside the
// event loop keeps the compiler from hoisting every per-resonance constant out of the
// loop into vector registers: the constants are re-read with scalar loads instead.
template <typename P> using kconst_ptr = __attribute__((address_space(4))) const P*;
template <typename P> __device__ __forceinline__ kconst_ptr<P> kernarg_laundered() {
  kconst_ptr<P> p = (kconst_ptr<P>)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// First K* slot of spin J in a compiled kernel shape (slots are ordered by spin).
template <class Sh> __host__ __device__ constexpr int slot_base(int J) {
  int b = 0;
  for (int j = 0; j < J; ++j) b += Sh::N[j];
  return b;
}

}  // namespace kpsi
