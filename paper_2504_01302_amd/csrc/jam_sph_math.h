// Functions of the spherical kernels' points, from small tables in LDS: a few
// FP64 ulp where the library's cost three to six times the operations.
#pragma once

#include "jam_device.h"
#include "jam_internal.h"

namespace jam {
namespace {

// Evaluated at compile time (series that end below FP64 rounding).
struct alignas(16) SphTables {
  double lg[64][2];                // 1 / c, -log(1 / c) at the centres c of 64 mantissa intervals
  double ex[32];                   // 2^(i / 32)
  double sn[kSphNT];               // sin of the moment table's angles
  double at[65];                   // atan(i / 64)
};
constexpr SphTables sph_tables() {
  SphTables t{};
  for (int i = 0; i < 64; ++i) {
    const double ic = 1.0 / (1.0 + (i + 0.5) / 64.0);
    // -log ic = 2 atanh z
    const double z = (1.0 - ic) / (1.0 + ic), z2 = z * z;
    double p = 0.0;
    for (int n = 41; n >= 1; n -= 2) p = p * z2 + 1.0 / n;
    t.lg[i][0] = ic;
    t.lg[i][1] = 2.0 * z * p;
  }
  for (int i = 0; i < 32; ++i) {
    const double x = i * 0.02166084939249829;    // ln 2 / 32
    double p = 1.0;
    for (int n = 24; n >= 1; --n) p = 1.0 + p * x / n;
    t.ex[i] = p;
  }
  for (int i = 0; i < kSphNT; ++i) {
    const double x = i * (0.5 * kPi / (kSphNT - 1)), x2 = x * x;
    double p = 1.0;
    for (int n = 25; n >= 3; n -= 2) p = 1.0 - p * x2 / (n * (n - 1));
    t.sn[i] = x * p;
  }
  for (int i = 1; i <= 64; ++i) {
    // atan(i / 64) - atan((i - 1) / 64) = atan(z)
    const double z = (1.0 / 64.0) / (1.0 + i * (i - 1) / 4096.0), z2 = z * z;
    double p = 0.0;
    for (int n = 15; n >= 1; n -= 2) p = 1.0 / n - p * z2;
    t.at[i] = t.at[i - 1] + z * p;
  }
  return t;
}
__device__ constexpr SphTables kSphTables = sph_tables();

// A kernel's tables in LDS.  The caller synchronises.
struct alignas(16) PolMath {       // potential grid
  double lg[64][2];
  double ex[32];
  double sn[kSphNT];
};
struct alignas(16) LosMath {       // line of sight
  double lg[64][2];
  double at[65];
};
__device__ inline void pol_math_fill(PolMath &t) {
  for (int e = threadIdx.x; e < 128; e += blockDim.x) (&t.lg[0][0])[e] = (&kSphTables.lg[0][0])[e];
  for (int e = threadIdx.x; e < 32; e += blockDim.x) t.ex[e] = kSphTables.ex[e];
  for (int e = threadIdx.x; e < kSphNT; e += blockDim.x) t.sn[e] = kSphTables.sn[e];
}
__device__ inline void los_math_fill(LosMath &t) {
  for (int e = threadIdx.x; e < 128; e += blockDim.x) (&t.lg[0][0])[e] = (&kSphTables.lg[0][0])[e];
  for (int e = threadIdx.x; e < 65; e += blockDim.x) t.at[e] = kSphTables.at[e];
}

// log of a positive normal w to about 1e-16 absolute (a grid coordinate):
// exponent + table + series in |r| <= 1 / 128.
template <class Tables> __device__ __forceinline__ double pol_log(double w, const Tables &tb) {
  const int hi = __double2hiint(w);
  const double2 c = *reinterpret_cast<const double2 *>(tb.lg[(hi >> 14) & 63]);
  const double m = __hiloint2double((hi & 0xfffff) | 0x3ff00000, __double2loint(w));
  const double r = fma(m, c.x, -1.0);
  double p = fma(r, 1.0 / 7.0, -1.0 / 6.0);
  p = fma(p, r, 1.0 / 5.0);
  p = fma(p, r, -1.0 / 4.0);
  p = fma(p, r, 1.0 / 3.0);
  p = fma(p, r, -1.0 / 2.0);
  return fma((double)((hi >> 20) - 1023), 0.6931471805599453, c.y + fma(r * r, p, r));
}

// exp of x <= 0, relative error a few FP64 ulp (of the argument's rounding).
__device__ __forceinline__ double pol_exp(double x, const PolMath &tb) {
  x = fmax(x, -800.0);
  const double n = rint(x * 46.16624130844683);          // 32 / ln 2
  const double r = fma(n, -7.247021293269686e-19, fma(n, -0.02166084939249829, x));
  double p = fma(r, 1.0 / 720.0, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  const int ni = (int)n;
  const double t = tb.ex[ni & 31];
  return ldexp(fma(t, fma(r * r, p, r), t), ni >> 5);
}

// Angle in [0, pi / 2] of the point (c, s), c, s >= 0 and not both zero:
// table + series in |d| <= 1 / 128.
__device__ __forceinline__ double los_atan(double s, double c, const LosMath &tb) {
  const double hi = fmax(s, c), lo = fmin(s, c);
  const int n = (int)fmaf((float)lo * __builtin_amdgcn_rcpf((float)hi), 64.f, 0.5f);
  const int i = min(max(n, 0), 64);
  const double t = i * (1.0 / 64.0);
  const double d = fma(-t, hi, lo) * rcp64(fma(t, lo, hi)), d2 = d * d;
  double p = fma(d2, -1.0 / 7.0, 1.0 / 5.0);
  p = fma(p, d2, -1.0 / 3.0);
  const double a = tb.at[i] + fma(d * d2, p, d);
  return s <= c ? a : 0.5 * kPi - a;
}

}  // namespace
}  // namespace jam
