// Device helpers shared by the gfx950 kernel files.
#pragma once

#include <hip/hip_runtime.h>

namespace jam {
namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr double kLog2e = 1.44269504088896340736;

// G in pc (km/s)^2 / Msun: IAU nominal GM_sun over (1 pc in m) * 1e6, with
// 1 pc = 648000/pi au and the IAU au.
constexpr double kGMsun = 1.3271244e20;
constexpr double kAu = 149597870700.0;

__device__ inline double grav_const() { return kGMsun / (kAu * 648000.0 / kPi * 1.0e6); }

__device__ inline double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// FP64 reciprocal and reciprocal square root: the hardware approximations
// refined by two Newton steps (a few FP64 ulp; the coefficients they feed are
// stored as FP32).  Arguments are positive and finite.
__device__ inline double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}
__device__ inline double rsq64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double e = fma(-x * y, y, 1.0);
  y = fma(0.5 * y, e, y);
  e = fma(-x * y, y, 1.0);
  return fma(0.5 * y, e, y);
}

// log of a positive normal number to about 1e-15 (the interpolation variable
// takes no more): mantissa in [sqrt(1/2), sqrt 2), odd series in
// (m - 1) / (m + 1).
__device__ __forceinline__ double log64(double x) {
  int e = __builtin_amdgcn_frexp_exp(x);
  double m = __builtin_amdgcn_frexp_mant(x);         // [1/2, 1)
  const bool low = m < 0.70710678118654752440;
  m = low ? 2.0 * m : m;
  e = low ? e - 1 : e;
  const double t = (m - 1.0) * rcp64(m + 1.0), t2 = t * t;
  double q = 2.0 / 19.0;
  q = fma(q, t2, 2.0 / 17.0);
  q = fma(q, t2, 2.0 / 15.0);
  q = fma(q, t2, 2.0 / 13.0);
  q = fma(q, t2, 2.0 / 11.0);
  q = fma(q, t2, 2.0 / 9.0);
  q = fma(q, t2, 2.0 / 7.0);
  q = fma(q, t2, 2.0 / 5.0);
  q = fma(q, t2, 2.0 / 3.0);
  return fma((double)e, 0.69314718055994530942, t * fma(q, t2, 2.0));
}

// A load through a pointer that the compiler cannot see to be global (one read
// from a descriptor), which would otherwise be a flat load and wait for LDS too.
__device__ __forceinline__ double load_global(const double *p) {
  return *reinterpret_cast<const __attribute__((address_space(1))) double *>(
      reinterpret_cast<uintptr_t>(p));
}

constexpr double kSqrtPi = 1.77245385090551602730;

}  // namespace
}  // namespace jam
