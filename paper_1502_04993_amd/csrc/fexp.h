// exp in FP64 for the device's epilogues (and, for tests, the host): x = k ln 2 + r with
// |r| <= ln2 / 2 and e^r = 1 + r + r^2 q(r), q of degree 9 interpolating
// (e^r - 1 - r) / r^2 at Chebyshev points (relative error 1.6e-17 before
// rounding; about 1 ulp in all).  Overflow gives infinity, underflow 0
// (through denormals), also at infinite x; NaN stays NaN.  21 instructions
// where the library's exp compiles to 38 here (a move before each fused
// multiply-add, and selects for the special cases).
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define GLMR_EXP_FN __host__ __device__ __forceinline__
#else
#include <math.h>
#define GLMR_EXP_FN inline
#endif

GLMR_EXP_FN double exp_f64(double x) {
  const double c = fmin(fmax(x, -1100.0), 1100.0);
  const double k = __builtin_rint(c * 1.44269504088896338700e+00);
  double r = fma(k, -6.93147180559945286227e-01, c);
  r = fma(k, -2.31904681384629955842e-17, r);
  double q = 2.5100424157005067e-08;
  q = fma(q, r, 2.7620138719733994e-07);
  q = fma(q, r, 2.7557268378684192e-06);
  q = fma(q, r, 2.480152119021773e-05);
  q = fma(q, r, 0.00019841269863105968);
  q = fma(q, r, 0.0013888888917281794);
  q = fma(q, r, 0.008333333333330051);
  q = fma(q, r, 0.04166666666662399);
  q = fma(q, r, 0.16666666666666669);
  q = fma(q, r, 0.5000000000000001);
  const double e = 1.0 + fma(r * r, q, r);
  // the clamp drops a NaN: it comes back as the upper half's bits
  struct Halves {
    unsigned lo, hi;
  } v = __builtin_bit_cast(Halves, __builtin_ldexp(e, (int)k));
  v.hi = x != x ? 0x7ff80000u : v.hi;
  return __builtin_bit_cast(double, v);
}
