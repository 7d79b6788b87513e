"""The kernels' own logarithms, exponential, arc tangent, reciprocal and
reciprocal square root (jam_device.h, jam_sph_math.h), compiled for the host
with the few device names they use, against long double.

Bars: a few FP64 ulp (2.2e-16), absolute for the logarithms and the arc tangent
(coordinates), relative for the others; 1e-15 for log64, which says so.  A
relative error of exp grows with the rounding of x times log2(e) and is taken per
1 + |x| / 8.  The hardware's first approximations are replaced by ones rounded to 24 bits."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2504_01302_amd", "csrc")

STUB = r"""
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __restrict__
struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
struct double2 { double x, y; };
typedef void *hipStream_t;
struct Dim { unsigned x = 0; };
static Dim threadIdx, blockDim;
using std::max;
using std::min;
inline double __shfl_xor(double v, int, int) { return v; }
inline double __builtin_amdgcn_rcp(double x) { return (float)(1.0 / x); }
inline double __builtin_amdgcn_rsq(double x) { return (float)(1.0 / std::sqrt(x)); }
inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
inline int __builtin_amdgcn_frexp_exp(double x) { int e; std::frexp(x, &e); return e; }
inline double __builtin_amdgcn_frexp_mant(double x) { int e; return std::frexp(x, &e); }
inline uint64_t bits(double x) { uint64_t u; std::memcpy(&u, &x, 8); return u; }
inline int __double2hiint(double x) { return (int)(bits(x) >> 32); }
inline int __double2loint(double x) { return (int)(uint32_t)bits(x); }
inline double __hiloint2double(int h, int l) {
  const uint64_t u = (uint64_t)(uint32_t)h << 32 | (uint32_t)l;
  double x;
  std::memcpy(&x, &u, 8);
  return x;
}
"""

MAIN = r"""
#include "jam_sph_math.h"
#include <cstdio>
#include <random>
using namespace jam;
int main() {
  PolMath pm;
  LosMath lm;
  blockDim.x = 1;
  pol_math_fill(pm);
  los_math_fill(lm);
  std::mt19937_64 r(7);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long double lg = 0, l64 = 0, ex = 0, at = 0, rc = 0, rs = 0, sn = 0;
  auto up = [](long double &m, long double e) { m = e < 0 ? std::max(m, -e) : std::max(m, e); };
  for (int i = 0; i < 400000; ++i) {
    const double w = std::exp(60.0 * (u(r) - 0.5)), one = 1.0 + (u(r) - 0.5) * 1e-3;
    for (double v : {w, one}) {
      const long double L = logl((long double)v);
      up(lg, (pol_log(v, pm) - L) / std::max(1.0L, fabsl(L)));
      up(l64, (log64(v) - L) / std::max(1.0L, fabsl(L)));
    }
    const double x = -700.0 * u(r) * u(r);
    up(ex, (pol_exp(x, pm) / expl((long double)x) - 1) / (1 + fabsl((long double)x) / 8));
    const double t = 1.5707963267948966 * u(r), a = std::exp(20.0 * (u(r) - 0.5));
    const double s = a * std::sin(t), c = a * std::cos(t);
    up(at, los_atan(s, c, lm) - atan2l(s, c));
    up(rc, rcp64(w) * (long double)w - 1);
    up(rs, rsq64(w) * sqrtl((long double)w) - 1);
  }
  for (int i = 0; i < kSphNT; ++i)
    up(sn, pm.sn[i] - sinl(i * (0.5L * 3.14159265358979323846264338327950288L / (kSphNT - 1))));
  // ends: below exp's range an exact zero, and the arguments 0 and 1
  const bool ends = pol_exp(-760.0, pm) == 0.0 && pol_exp(-1e300, pm) == 0.0 && pol_exp(0.0, pm) == 1.0 &&
                    std::fabs(pol_log(1.0, pm)) < 1e-16 && std::fabs(log64(1.0)) < 1e-16 &&
                    los_atan(0.0, 1.0, lm) == 0.0 &&
                    std::fabs(los_atan(1.0, 0.0, lm) - 1.5707963267948966) < 1e-15;
  std::printf("%Lg %Lg %Lg %Lg %Lg %Lg %Lg %d\n", lg, l64, ex, at, rc, rs, sn, (int)ends);
}
"""


def test_device_functions_on_the_host(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "math")
    subprocess.run([cxx, "-O2", "-std=c++17", "-w", "-I", str(tmp_path), "-I", CSRC,
                    str(tmp_path / "main.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()
    lg, l64, ex, at, rc, rs, sn = map(float, out[:7])
    print(f"log {lg:.1e}, log64 {l64:.1e}, exp {ex:.1e}, atan {at:.1e}, rcp {rc:.1e}, "
          f"rsq {rs:.1e}, sin {sn:.1e}")
    ulp = 2.3e-16
    assert lg <= 2 * ulp and l64 <= 1e-15 and ex <= 4 * ulp and at <= 2 * ulp
    assert rc <= 2 * ulp and rs <= 2 * ulp and sn <= ulp and out[7] == "1"
