// Sines and cosines of RoPE angles p * base^(-2j/d_h) (App. B.1.1).  The angle is formed and reduced to [-pi/4, pi/4] in
// fp64 (pi/2 in two parts), then comes a Taylor series and the quadrant.  Good for angles up to 2^40: every position at a
// base of 1 or more (rope_angles_small).
#pragma once
#include <hip/hip_runtime.h>

namespace gta {

// Frequencies are at most 1.  A smaller base is accepted, but its frequencies grow up to base^-1 and leave the range of
// the reduction: such calls keep to kernels that call the library's sine.
inline bool rope_angles_small(int rope, double base) { return !rope || base >= 1.0; }

// p * f = x + quadrant * pi/2
__device__ __forceinline__ double rope_reduce(int p, double f, int &quadrant) {
  const double ang = (double)p * f, k = rint(ang * 0.6366197723675814);
  quadrant = (int)(k - 4.0 * floor(k * 0.25));   // 0 .. 3
  return fma(-k, 6.123233995736766e-17, fma(-k, 1.5707963267948966, ang));
}

// (cos, sin) rounded once from fp64: the series to degree 11 / 12 (the first terms left out are below 1e-11).  For fp32
// rows and tables.
__device__ __forceinline__ float2 rope_cos_sin(int p, double f) {
  int q;
  const double x = rope_reduce(p, f, q), y = x * x;
  const double s = fma(x * y, fma(y, fma(y, fma(y, fma(y, -1. / 39916800., 1. / 362880.), -1. / 5040.), 1. / 120.), -1. / 6.), x);
  const double c = fma(y, fma(y, fma(y, fma(y, fma(y, fma(y, 1. / 479001600., -1. / 3628800.), 1. / 40320.), -1. / 720.), 1. / 24.), -0.5), 1.);
  const float a = (float)(q & 1 ? c : s), b = (float)(q & 1 ? s : c);
  return make_float2((q + 1) & 2 ? -b : b, q & 2 ? -a : a);
}

// the same for any angle (tables)
__device__ __forceinline__ float2 rope_cos_sin_any(int p, double f) {
  const double ang = (double)p * f;
  if (fabs(ang) < 0x1p40) return rope_cos_sin(p, f);
  double s, c;
  sincos(ang, &s, &c);
  return make_float2((float)c, (float)s);
}

// rope_cos_sin with the series in fp32, to degree 9 / 10 (the first terms left out are below 2e-9 and 2e-10): largest error
// 5.8e-8 against 3.0e-8.  For rows that are rounded to bf16.
__device__ __forceinline__ float2 rope_cos_sin_short(int p, double f) {
  int q;
  const float r = (float)rope_reduce(p, f, q), r2 = r * r;
  const float s = fmaf(r * r2, fmaf(r2, fmaf(r2, fmaf(r2, 1.f / 362880.f, -1.f / 5040.f), 1.f / 120.f), -1.f / 6.f), r);
  const float c = fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, fmaf(r2, -1.f / 3628800.f, 1.f / 40320.f), -1.f / 720.f), 1.f / 24.f), -0.5f), 1.f);
  const float a = q & 1 ? c : s, b = q & 1 ? s : c;
  return make_float2((q + 1) & 2 ? -b : b, q & 2 ? -a : a);
}

}  // namespace gta
