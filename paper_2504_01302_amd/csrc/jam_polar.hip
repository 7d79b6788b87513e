// gfx950 kernels of the spherical model's potential grid: the tracer-free
// (j, u) sums G and G_theta of the characteristic integrals, tabulated on a
// polar grid, the moment table interpolated from it, and the adjoint of both.
//
// A node of tracer k's characteristic through (r, theta) lies at r' = r e^tau,
// where tau belongs to (k, r, node) alone, and sin theta' = sin theta
// (r / r')^(1 - beta).  With the grid's rows at radii (uniform in ln r') and
// its columns over the angle, the interpolation splits: the row weights of a
// node are those of all its 24 angles, so a wave combines the six rows into
// one line of 64 columns (contiguous loads), and the 24 points read their
// eight columns of the line from LDS.  The adjoint is the transpose: points
// onto lines, lines onto rows.
//
// Rows: x = 2 + (ln r' - ln r_0) iX, r_0 the table's first radius, r_max =
// sqrt(r_hi^2 + 50 max sigma_k^2), the farthest node, at x = kPolN - 4.
// Columns: y = iC log(1 + cos^2 theta' / s0) with s0 the smallest h = 1 - e_j^2 u^2
// of the terms, y = kPolC - 8 on the axis; column slot s holds y = s - 3.
// Both variables are analytic with unit scale whatever the model: a term is
// exp(-v r'^2 - d r'^2 cos^2 theta') with d = v (1 / h - 1) <= v (1 / s0 - 1),
// bounded for |Im ln r'| < pi / 4 and |Im y / iC| < pi / 2 (slots 0 .. 2 take cos^2
// theta' down to -s0, where the term is still below one).  Lagrange interpolation on
// 6 x 8 points of the 384 x 64 grid leaves at most 1e-7 of G at q_j >= 0.05
// (FP64 sums, five mass models, 6000 points each) where 4 x 4 points of a 512
// x 512 grid in R and z left 1e-6 to 1e-5; and of G_theta at q_j = 0.05 up to 3e-4 of
// its largest value at the same radius, where that radius is far outside the thin
// Gaussian and a few terms make it up.  s0 has to be that of the terms: the smallest
// q_j^2 goes to zero at the deprojection limit and stretches the columns with it,
// while u < 1 keeps h from it.  Against 64 bits, models of 3 + 12 tracers 1e-4, 1e-6
// and 1e-8 in cos i inside the limit, V / gradient at most: s0 = min q_j^2 8e-7 / 9e-6,
// 4e-5 / 2e-4, 3e-4 / 9e-4, this 5e-7 / 6e-6, 2e-6 / 4e-6, 2e-6 / 4e-6, the R, z grid
// 1e-6 / 2e-6, 3e-6 / 4e-5, 5e-6 / 1e-4.
#include "jam_device.h"
#include "jam_internal.h"
#include "jam_sph_math.h"

#include <hip/hip_runtime.h>
#include <algorithm>
#include <type_traits>

namespace jam {

namespace {

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Orders a wave's own LDS writes before its later reads by other lanes (LDS
// operations of a wave execute in order; this keeps the compiler to it).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Lagrange weights of P equidistant points -(P/2 - 1) .. P/2 at f.
template <int P> __device__ __forceinline__ void lagrange(double f, double (&w)[P]) {
  double d[P], pre[P];
#pragma unroll
  for (int i = 0; i < P; ++i) d[i] = f - (double)(i - (P / 2 - 1));
  pre[0] = 1.0;
#pragma unroll
  for (int i = 1; i < P; ++i) pre[i] = i == 1 ? d[0] : pre[i - 1] * d[i - 1];
  double suf = 1.0;
#pragma unroll
  for (int i = P - 1; i >= 0; --i) {
    double q = 1.0;                        // product of the point distances
    for (int j = 0; j < P; ++j)
      if (j != i) q *= (double)(i - j);
    w[i] = i == 0 ? suf * (1.0 / q) : (i == P - 1 ? pre[i] * (1.0 / q) : pre[i] * suf * (1.0 / q));
    suf = i == P - 1 ? d[i] : suf * d[i];
  }
}

// By value: a conditional of two array elements would select the index.
__device__ __forceinline__ double select(bool on, double a, double b) { return on ? a : b; }
// w[b] = w[(b + Q) % 8] where d has bit Q.
template <int Q> __device__ __forceinline__ void rotate8(double (&w)[8], int d) {
  const bool on = d & Q;
  double u[8];
#pragma unroll
  for (int b = 0; b < 8; ++b) u[b] = select(on, w[(b + Q) & 7], w[b]);
#pragma unroll
  for (int b = 0; b < 8; ++b) w[b] = u[b];
}

// Whether a tracer's density underflows to an exact zero along every
// characteristic from radius r on: its exponent at r' >= r is at least
// min(alpha, alphaq) r^2, and pol_exp gives zero from 746 on.  Such a (tracer,
// radius) adds exact zeros everywhere and is left out: narrow tracers at large
// radii, a fifth of the pairs of 48 models of 10 tracers.  Measured there with
// them / without: moments 800 + 1230 / 684 + 1179 us, spread 1520 / 1240.
// The radius always as pol_radius2: what the moments leave out the spread must not
// read.
__device__ __forceinline__ double pol_radius2(const GeomDev &g, int ir) {
  return exp(2.0 * fma((double)ir, g.sph_dlnr, g.sph_lnr0));
}
__device__ __forceinline__ bool pol_empty(double alpha, double alphaq, double r2) {
  return fmin(alpha, alphaq) * r2 > 750.0;
}

// Grid scales of a model (k_sph_terms): iX, s0, iC.
struct PolScale {
  double iX, s0, iC;
};
__device__ inline PolScale pol_scale(const double *pol, const ModelDev &md) {
  const double *p = pol + md.pol_off;
  return PolScale{p[0], p[1], p[2]};
}
__device__ inline double *pol_parts(double *pol, const ModelDev &md) {
  return pol + md.pol_off + kPolScales;
}
// r'^2 of row i and cos^2 theta' of column slot s.
__device__ inline double pol_row_r2(const GeomDev &g, const PolScale &sc, int i) {
  return exp(2.0 * (g.sph_lnr0 + (i - 2) / sc.iX));
}
__device__ inline double pol_col_c2(const PolScale &sc, int s) {
  return sc.s0 * expm1((s - 3) / sc.iC);
}
// Lower bound over the columns of a term's exponent in units of v r'^2.
__device__ inline double pol_reach(const PolScale &sc) {
  return 1.0 + (1.0 - sc.s0) * expm1(-3.0 / sc.iC);
}
// ---------------------------------------------------------------------------
// The grid: item (m, four rows, term slice); wave = row, lane = column.  The
// term coefficients are uniform over the wave (scalar loads); FP32 sums of 64
// terms folded into FP64, the slice partial stored in FP32 ([N][C][2] per
// slice: G, G_theta).
// The exponent is not a product of a row and a column factor here, so the
// sums run on the VALU: two FP32 operations, an exponential and two
// multiply-adds per term and point, but on 24,576 points where the R, z grid
// took matrix products on 262,144.  Measured (48 models of 1300 terms / one
// of 5248): 683 / 72 us on that grid, 287 / 37 here.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_pol_grid(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  const float4 *__restrict__ terms,
                                                  const int *__restrict__ st_ws,
                                                  const double *__restrict__ pol,
                                                  float *__restrict__ sgrid) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;         // the grid is not read
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const PolScale sc = pol_scale(pol, md);
    const int row = 4 * it.a + wave;
    const double r2 = pol_row_r2(g, sc, row), z2 = r2 * pol_col_c2(sc, lane);
    const float R2 = (float)(r2 - z2), Z2 = (float)z2;
    const int chunks = sph_terms_padded(g.J1, g.n_u) / 64;
    const int c0 = (int)((int64_t)chunks * it.b / md.sgrid_slices);
    const int c1 = (int)((int64_t)chunks * (it.b + 1) / md.sgrid_slices);
    const float4 *tc = terms + md.term_off;
    double acc[2] = {0.0, 0.0};
    for (int ch = c0; ch < c1; ++ch) {
      float f[2] = {0.f, 0.f};
#pragma unroll 16
      for (int t = 64 * ch; t < 64 * ch + 64; ++t) {
        const float4 c = tc[t];
        const float e = fast_exp2(fmaf(c.x, R2, c.y * Z2));
        f[0] = fmaf(c.z, e, f[0]);
        f[1] = fmaf(c.w, e, f[1]);
      }
      acc[0] += (double)f[0];
      acc[1] += (double)f[1];
    }
    float *o = sgrid + md.sgrid_off + (int64_t)it.b * (kPolN * kPolC * 2);
    o[(row * kPolC + lane) * 2] = (float)acc[0];
    o[(row * kPolC + lane) * 2 + 1] = (float)acc[1];
  }
}

// The adjoint's grid: G, G_theta and T_theta = dG_theta / dR'^2 at fixed r' (all
// the adjoint needs beside them: with R'^2 + z'^2 = r'^2 fixed, dG / dR'^2 =
// G_theta / 2), per slice (G, G_theta) [N][C] in FP64 and T_theta [N][C] in FP32.
// A model's inclination derivative is one number in which terms hundreds of times
// larger cancel, so exponents, sums and the stored G, G_theta are FP64; only the
// exponential is FP32, whose rounding differs from term to term.  Relative error of
// that derivative, 24 single models of 40 x 41 Gaussians, largest / geometric mean:
// all FP32 1.4e-5 / 4.5e-7, FP64 sums stored in FP32 4e-6 / 1e-7, FP32 sums of 64
// terms stored in FP64 1e-5 / 2e-7, this 6e-7 / 3e-8, FP64 exponentials as well
// 1e-7 / 3e-9.  T_theta only enters d/dbeta, which does not cancel.  Measured (48
// models of 1300 terms / one of 5248): all FP32 331 / 41 us, this 517 / 75, FP64
// exponentials as well 877 / 105.
__global__ void __launch_bounds__(256) k_pol_grid_adj(const GeomDev *__restrict__ geoms,
                                                      const ModelDev *__restrict__ models,
                                                      const Item *__restrict__ items, int n_it,
                                                      const double *__restrict__ terms64,
                                                      const int *__restrict__ st_ws,
                                                      const double *__restrict__ pol,
                                                      double *__restrict__ sgrid3) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;         // the grid is not read
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const PolScale sc = pol_scale(pol, md);
    const int row = 4 * it.a + wave;
    const double r2 = pol_row_r2(g, sc, row), Z2 = r2 * pol_col_c2(sc, lane), R2 = r2 - Z2;
    const int chunks = sph_terms_padded(g.J1, g.n_u) / 64;
    const int c0 = (int)((int64_t)chunks * it.b / md.sgrid_slices);
    const int c1 = (int)((int64_t)chunks * (it.b + 1) / md.sgrid_slices);
    const SphTerm *tc = reinterpret_cast<const SphTerm *>(terms64 + md.term64_off);
    double G = 0.0, T = 0.0, D = 0.0;
#pragma unroll 8
    for (int t = 64 * c0; t < 64 * c1; ++t) {
      const double e = (double)fast_exp2((float)fma(tc[t].cx, R2, tc[t].cy * Z2));
      G = fma(tc[t].gP, e, G);
      T = fma(tc[t].gT, e, T);
      D = fma(tc[t].gD, e, D);
    }
    double *o = sgrid3 + md.sgrid3_off + (int64_t)it.b * kPolAdjGrid;
    reinterpret_cast<double2 *>(o)[row * kPolC + lane] = make_double2(G, T);
    reinterpret_cast<float *>(o + 2 * kPolN * kPolC)[row * kPolC + lane] = (float)D;
  }
}

// Item (m, block of 1024 grid floats; the adjoint's 256 grid points): the slice
// partials summed in slice order (FP64) into slice 0.
__global__ void __launch_bounds__(256) k_pol_grid_sum(const ModelDev *__restrict__ models,
                                                      const Item *__restrict__ items, int n_it,
                                                      const int *__restrict__ st_ws,
                                                      float *__restrict__ sgrid) {
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;
    const ModelDev md = models[it.m];
    const int64_t len = (int64_t)kPolN * kPolC * 2;
    float4 *base = reinterpret_cast<float4 *>(sgrid + md.sgrid_off) + it.a * 256 + threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int sl = 0; sl < md.sgrid_slices; ++sl) {
      const float4 q = base[sl * (len / 4)];
      v[0] += (double)q.x; v[1] += (double)q.y; v[2] += (double)q.z; v[3] += (double)q.w;
    }
    *base = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
  }
}
__global__ void __launch_bounds__(256) k_pol_grid_sum_adj(const ModelDev *__restrict__ models,
                                                          const Item *__restrict__ items, int n_it,
                                                          const int *__restrict__ st_ws,
                                                          double *__restrict__ sgrid3) {
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;
    const ModelDev md = models[it.m];
    const int e = it.a * 256 + threadIdx.x;
    double *base = sgrid3 + md.sgrid3_off;
    double2 v = make_double2(0.0, 0.0);
    double d = 0.0;
    for (int sl = 0; sl < md.sgrid_slices; ++sl) {
      const double *b = base + (int64_t)sl * kPolAdjGrid;
      const double2 q = reinterpret_cast<const double2 *>(b)[e];
      v.x += q.x;
      v.y += q.y;
      d += (double)reinterpret_cast<const float *>(b + 2 * kPolN * kPolC)[e];
    }
    reinterpret_cast<double2 *>(base)[e] = v;
    reinterpret_cast<float *>(base + 2 * kPolN * kPolC)[e] = (float)d;
  }
}

// ---------------------------------------------------------------------------
// Moments.  A wave per (tracer group, radius), a block four consecutive radii
// (whose lines share rows in the L1): the group's tracers in turn, all 24
// angles.  Set-up with lane = node; then per segment of eight nodes the eight
// lines (lane = column), and the 24 x 8 points in three rounds (lane = 8
// (angle % 8) + node % 8), eight columns each from LDS.  A group's share of
// (A_r, A_theta, A_phi) per cell goes to the partials, which k_pol_table adds
// in order.  FP64 but the grid's values; all sums run in a fixed order.
// kJac: the adjoint's forward pass.  Per (cell, tracer) the node sums of the
// characteristic integrals (fP, fD) and of their derivatives with respect to
// beta_k (bP, bD), alphaq_k (qP, qD) and nu0_k (eP, eD) go to SphAdj::jac,
// none of which depends on the table cotangent (k_sph_rows combines them with
// it), and (s, r'^2, weight) of every node to the node table of k_pol_spread.
// Dependent FP64 operations and LDS reads bound it: the three rounds' sums
// leave registers for two waves a SIMD, whose latencies overlap little (one
// wave takes twice the time), so the compiler is asked to schedule as for
// four; its default order for two costs 930 us where this takes 797, and 1780
// where this takes 1225.  Tried and slower: three waves sharing the lines with
// eight angles each (four waves a SIMD, but barriers and three times the rows
// in the L1), rows prefetched a segment ahead.  Measured (48 models of 10
// tracers / one of 40), a block per four table points and 4 x 4 scattered
// points of the R, z grid before, this after: forward 3444 / 303 -> 684 / 82
// us, the adjoint's pass 6417 / 498 -> 1227 / 152 (1179 / 146 with its grid in
// FP32).
// ---------------------------------------------------------------------------
template <bool kJac> struct PolWave {
  double rp2[64], s[64], w[64], wd[64];   // r'^2, (r / r')^(1 - beta), weights of P and D
  double tau[kJac ? 64 : 1];
  double x[64];                           // row coordinate
  double wx[8][6];                        // a segment's row weights and row offsets
  int row[8], c0[64];                     // and first column
  double2 L[8][kPolC + 1];                // lines (G, G_theta); the odd stride spreads the banks
  double L3[kJac ? 8 : 1][kPolC + 1];     // T_theta
};

// Forward lines: the columns from 64 - 2 LPN on, LPN lanes per node, two
// columns a lane (16 bytes a load: loads issue at four lanes per cycle
// whatever their width), 64 / LPN nodes a step.
template <int LPN>
__device__ __forceinline__ void pol_lines(PolWave<false> &W, const float *__restrict__ sg, int lane) {
  constexpr int kStep = 64 / LPN;
  const int col = kPolC - 2 * LPN + 2 * (lane % LPN), sub = lane / LPN;
#pragma unroll 1
  for (int q = 0; q < 8; q += kStep) {
    const int h = q + sub;
    const float *g0 = sg + W.row[h] + col * 2;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < 6; ++a) {
      const double wx = W.wx[h][a];
      const float4 f = *reinterpret_cast<const float4 *>(g0 + a * (kPolC * 2));
      v[0] = fma(wx, (double)f.x, v[0]);
      v[1] = fma(wx, (double)f.y, v[1]);
      v[2] = fma(wx, (double)f.z, v[2]);
      v[3] = fma(wx, (double)f.w, v[3]);
    }
    W.L[h][col] = make_double2(v[0], v[1]);
    W.L[h][col + 1] = make_double2(v[2], v[3]);
  }
}

// The grid's numbers: the forward's FP32, the adjoint's FP64.
template <bool kJac> using PolGrid = std::conditional_t<kJac, double, float>;

template <bool kJac>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) k_pol_moments(
    const GeomDev *__restrict__ geoms, const ModelDev *__restrict__ models,
    const Item *__restrict__ items, int n_it, const double *__restrict__ gauss,
    const int *__restrict__ st_ws, const PolGrid<kJac> *__restrict__ sgrid,
    double *__restrict__ pol, double *__restrict__ sens, double *__restrict__ pcot) {
  static_assert(kSphNT == 24 && kSphNodes == 64 && kPolC == 64 && kPolPr == 6, "wave layout");
  constexpr int NS = kJac ? 6 : 2;
  __shared__ PolMath mt;
  __shared__ PolWave<kJac> wv[4];
  const int lane = threadIdx.x & 63, nd = lane & 7, tl = lane >> 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  PolWave<kJac> &W = wv[wave];
  pol_math_fill(mt);
  __syncthreads();
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;         // k_pol_table writes the zeros
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const int unit = 4 * it.a + wave, grp = unit / kSphNR, ir = unit % kSphNR;
    const int K = g.K, tg = pol_group_len(K), k0 = grp * tg, k1 = min(K, k0 + tg);
    const double *tab = gauss + md.gauss_off;
    const PolScale sc = pol_scale(pol, md);
    const double rs0 = 1.0 / sc.s0, iC = sc.iC;
    const double lnr = g.sph_lnr0 + ir * g.sph_dlnr, r = exp(lnr), r2 = pol_radius2(g, ir);
    const double glx = g.gl8_x[nd], glw = g.gl8_w[nd];
    const PolGrid<kJac> *sg = sgrid + (kJac ? md.sgrid3_off : md.sgrid_off);
    double Ar[3], At[3], Ap[3];             // lanes nd == 0: cells 8 t + tl
#pragma unroll
    for (int t = 0; t < 3; ++t) Ar[t] = At[t] = Ap[t] = 0.0;
    for (int k = k0; k < k1; ++k) {
      const double alpha = tab[k], alphaq = tab[K + k];
      const double kap2 = alphaq - alpha, kap = 2.0 * kap2;
      double *jac = nullptr;
      if constexpr (kJac)
        jac = sph_adj_layout(sens + md.sens_off, K, g.n_pix, sph_terms_padded(g.J1, g.n_u),
                             md.n_sens_parts).jac + ((int64_t)k * kSphCells + ir * kSphNT) * 8;
      if (pol_empty(alpha, alphaq, r2)) {           // uniform per wave
        if constexpr (kJac)
#pragma unroll
          for (int e = 0; e < 3; ++e) jac[64 * e + lane] = 0.0;
        continue;
      }
      wave_sync();                          // the previous tracer's reads of W
      {
        const double omb = 1.0 / tab[3 * K + k], beta = 1.0 - omb;
        const double hs = 0.5 * log1p(50.0 * (0.5 / alpha) / (r * r)) / kSphSeg;
        const double tau = (tl + 0.5 + 0.5 * glx) * hs;       // node = lane
        const double rp = exp(lnr + tau), rbt = exp(beta * tau), rpb = exp(beta * lnr) * rbt;
        const double wn = 0.5 * glw * hs * rp, s = (r / rp) * rbt;
        const double w = wn * (rp * rpb * rpb);
        W.rp2[lane] = rp * rp;
        W.s[lane] = s;
        W.w[lane] = w;
        W.wd[lane] = w * rpb * rp;
        W.x[lane] = fma(ir * g.sph_dlnr + tau, sc.iX, 2.0);
        if constexpr (kJac) {
          W.tau[lane] = tau;
          double *nt = pcot + md.sgcot_off + ((int64_t)(k * kSphNR + ir) * 64 + lane) * 3;
          nt[0] = s;
          nt[1] = rp * rp;
          nt[2] = wn * rp * rbt * rbt * tab[2 * K + k];
        }
        // cos^2 theta' >= 1 - s^2 at every angle
        const double c2 = fmax(0.0, fma(-s, s, 1.0));
        W.c0[lane] = (int)(pol_log(fma(c2, rs0, 1.0), mt) * iC - 1e-6);
      }
      double S[3][NS];
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int c = 0; c < NS; ++c) S[t][c] = 0.0;
      for (int seg = 0; seg < kSphSeg; ++seg) {
        wave_sync();                        // W written, the previous lines read
        {
          const double x = W.x[8 * seg + nd];
          const int i0 = min(max((int)x, 2), kPolN - 4);
          double wx[6];
          lagrange<6>(x - i0, wx);
          if (tl == 0) {
            W.row[nd] = (i0 - 2) * (kJac ? kPolC : kPolC * 2);
#pragma unroll
            for (int a = 0; a < 6; ++a) W.wx[nd][a] = wx[a];
          }
        }
        wave_sync();
        // far along the characteristic it runs near the axis: a segment needs
        // the columns from its first node's on
        const int c0 = __builtin_amdgcn_readfirstlane(W.c0[8 * seg]);
        if constexpr (kJac) {
          // unneeded columns repeat the first
          const double2 *sl = reinterpret_cast<const double2 *>(sg) + max(lane, c0);
          const float *sd = reinterpret_cast<const float *>(sg + 2 * kPolN * kPolC) + max(lane, c0);
#pragma unroll 4
          for (int h = 0; h < 8; ++h) {
            const int at = __builtin_amdgcn_readfirstlane(W.row[h]);
            double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int a = 0; a < 6; ++a) {
              const double wx = W.wx[h][a];
              const double2 q = sl[at + a * kPolC];
              v[0] = fma(wx, q.x, v[0]);
              v[1] = fma(wx, q.y, v[1]);
              v[2] = fma(wx, (double)sd[at + a * kPolC], v[2]);
            }
            W.L[h][lane] = make_double2(v[0], v[1]);
            W.L3[h][lane] = v[2];
          }
        } else {
          if (c0 >= 48)
            pol_lines<8>(W, sg, lane);
          else if (c0 >= 32)
            pol_lines<16>(W, sg, lane);
          else
            pol_lines<32>(W, sg, lane);
        }
        wave_sync();                        // lines written
        const int n = 8 * seg + nd;
        const double rp2 = W.rp2[n], s = W.s[n], w = W.w[n], wd = W.wd[n];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const double sraw = mt.sn[8 * t + tl] * s, st = fmin(1.0, sraw);
          const double c2 = fma(-st, st, 1.0);
          const double en = pol_exp(-rp2 * fma(kap2, c2, alpha), mt);
          const double y = pol_log(fma(c2, rs0, 1.0), mt) * iC;
          const int l0 = min(max((int)y, 0), kPolC - 8);
          double wy[8];
          lagrange<8>(y - l0, wy);
          const double2 *ln = &W.L[nd][l0];
          double G = 0.0, T = 0.0, D = 0.0;
#pragma unroll
          for (int b = 0; b < 8; ++b) {
            const double2 q = ln[b];
            G = fma(wy[b], q.x, G);
            T = fma(wy[b], q.y, T);
          }
          if constexpr (kJac) {
            const double *l3 = &W.L3[nd][l0];
#pragma unroll
            for (int b = 0; b < 8; ++b) D = fma(wy[b], l3[b], D);
          }
          const double we = w * en, wde = wd * en * st;
          const double H = fma(kap, G, T);      // the integrand's second sum
          S[t][0] = fma(we, G, S[t][0]);
          S[t][1] = fma(wde, H, S[t][1]);
          if constexpr (kJac) {
            // d/dbeta of the node at fixed r': sin theta' = s -> ds = s tau,
            // dR'^2 = -dz'^2 = 2 R'^2 tau
            const double tau = W.tau[n], td = sraw < 1.0 ? tau : 0.0, lrp = lnr + tau;
            const double hR2 = rp2 * (st * st) * td, z2 = rp2 * c2;
            const double dlnu = kap * hR2;      // d ln nu
            const double dG = hR2 * T, dH = fma(2.0 * hR2, D, kap * dG);
            S[t][2] = fma(we, fma(fma(2.0, lrp, dlnu), G, dG), S[t][2]);
            S[t][3] = fma(wde, fma(fma(3.0, lrp, td + dlnu), H, dH), S[t][3]);
            S[t][4] = fma(-we * z2, G, S[t][4]);
            S[t][5] = fma(wde, fma(-z2, H, 2.0 * G), S[t][5]);
          }
        }
      }
      // over the eight nodes of the lanes' groups
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int c = 0; c < NS; ++c) {
          double v = S[t][c];
          v += __shfl_xor(v, 1, 64);
          v += __shfl_xor(v, 2, 64);
          v += __shfl_xor(v, 4, 64);
          S[t][c] = v;
        }
      if (nd == 0) {
        const double omb = 1.0 / tab[3 * K + k], nu0 = tab[2 * K + k];
        const double rbe = exp((1.0 - omb) * lnr), rb2 = rbe * rbe;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const int th = 8 * t + tl;
          const double fP = nu0 * S[t][0], fD = nu0 * S[t][1], P = fP / rb2;
          Ar[t] += P;
          At[t] += omb * P;
          Ap[t] += omb * P + omb * mt.sn[th] * (r / (rb2 * rbe)) * fD;
          if constexpr (kJac) {
            double *o = jac + th * 8;
            o[0] = fP;
            o[1] = fD;
#pragma unroll
            for (int c = 2; c < 6; ++c) o[c] = nu0 * S[t][c];
            o[6] = S[t][0];
            o[7] = S[t][1];
          }
        }
      }
    }
    if (nd == 0) {
      double *o = pol_parts(pol, md) + ((int64_t)grp * kSphCells + ir * kSphNT) * 3;
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const int th = 8 * t + tl;
        o[3 * th] = Ar[t];
        o[3 * th + 1] = At[t];
        o[3 * th + 2] = Ap[t];
      }
    }
  }
}

// The table: per cell the groups' partials in order and -nu R^2 G_phi.  Item
// (m, 16 cells), a wave per cell, four cells each; G_phi's terms (FP32; the
// adjoint's exponents and sums FP64, as its grid's) and the tracer density summed in FP64 over the lanes in a fixed
// order.
template <bool kAdj>
__global__ void __launch_bounds__(256) k_pol_table(
    const GeomDev *__restrict__ geoms, const ModelDev *__restrict__ models,
    const Item *__restrict__ items, int n_it, const double *__restrict__ gauss,
    const float4 *__restrict__ terms, const double *__restrict__ terms64,
    const int *__restrict__ st_ws, double *__restrict__ pol, double *__restrict__ table,
    double *__restrict__ sens) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const int cell0 = 16 * it.a + 4 * wave;
    double *out = table + md.sph_off + (int64_t)cell0 * 3;
    if (st_ws[it.m] != 0) {                 // uniform per block
      if (lane < 12) out[lane] = 0.0;
      continue;
    }
    const int K = g.K, Tp = sph_terms_padded(g.J1, g.n_u);
    const double *tab = gauss + md.gauss_off;
    // lane c of the wave's first four: cell c's coordinates
    double r2c = 0.0, z2c = 0.0;
    {
      const int cell = cell0 + (lane & 3), ir = cell / kSphNT, ith = cell % kSphNT;
      const double r = exp(g.sph_lnr0 + ir * g.sph_dlnr), th = ith * (0.5 * kPi / (kSphNT - 1));
      const double R0 = r * sin(th), z0 = r * cos(th);
      r2c = R0 * R0;
      z2c = z0 * z0;
    }
    // tracer density: lane = 4 (tracer % 16) + cell
    double nu = 0.0;
    for (int k = lane >> 2; k < K; k += 16)
      nu += tab[2 * K + k] * exp(-(tab[k] * r2c + tab[K + k] * z2c));
    for (int o = 4; o < 64; o <<= 1) nu += __shfl_xor(nu, o, 64);
    double accF[4];
    PolGrid<kAdj> R20[4], Z20[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      R20[c] = (PolGrid<kAdj>)__shfl(r2c, c, 64);
      Z20[c] = (PolGrid<kAdj>)__shfl(z2c, c, 64);
      accF[c] = 0.0;
    }
    if constexpr (kAdj) {
      const SphTerm *tc = reinterpret_cast<const SphTerm *>(terms64 + md.term64_off);
#pragma unroll 2
      for (int t = lane; t < Tp; t += 64) {
        const double cx = tc[t].cx, cy = tc[t].cy, f = tc[t].gF;
#pragma unroll
        for (int c = 0; c < 4; ++c) 
          accF[c] = fma(f, (double)fast_exp2((float)fma(cx, R20[c], cy * Z20[c])), accF[c]);
      }
    } else {
      const float4 *tc = terms + md.term_off;
      const float *tf = (const float *)(tc + Tp);
#pragma unroll 4
      for (int t = lane; t < Tp; t += 64) {
        const float4 q = tc[t];
        const float f = tf[t];
#pragma unroll
        for (int c = 0; c < 4; ++c)
          accF[c] += (double)(f * fast_exp2(fmaf(q.x, R20[c], q.y * Z20[c])));
      }
    }
    // the partials: lane = 3 c + moment
    double v = 0.0;
    if (lane < 12) {
      const double *pp = pol_parts(pol, md) + (int64_t)cell0 * 3 + lane;
      for (int q = 0; q < pol_groups(K); ++q) v += pp[(int64_t)q * kSphCells * 3];
    }
    double sub = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double F = wave_sum(accF[c]), nR = __shfl(nu * r2c, c, 64);
      if (lane == 3 * c + 2) sub = nR * F;
      if (kAdj && lane == 0)
        sph_adj_layout(sens + md.sens_off, K, g.n_pix, Tp, md.n_sens_parts).gphi[cell0 + c] = F;
    }
    if (lane < 12) out[lane] = v - sub;
  }
}

// ---------------------------------------------------------------------------
// The adjoint's transpose.  The cotangents phi = dL/dG and psi = dL/dG_theta
// of the points (cell, tracer, node), from the table cotangent, onto the grid:
// item (m, row bin, tracer group), the nodes whose stencil starts in the bin's
// kPolR rows.  A wave looks through its (tracer, radius) pairs, queues their
// nodes of the bin, and takes them eight at a time whatever pair they came
// from: the 24 x 8 points in three rounds (lane = 8 (angle % 8) + node), each
// point's weighted cotangents into its node's line in LDS, then each line (lane = column) times its six row
// weights into kPolR + 5 rows of FP64 accumulators in registers.  The block's
// four waves are added in order; no atomics across waves, no scales, and the
// same result in any batch.
// FP64 issue and the LDS adds bound it.  Measured (48 models of 10 tracers /
// one of 40): the points sorted by tile of an R, z grid and spread with
// fixed-point atomics 5300 / 700 us, this with k_pol_cot_sum 1270 / 201.
// ---------------------------------------------------------------------------
struct SpreadWave {
  double L[2][8][kPolC + 1];              // lines of phi and psi
  double2 wx[8][3];
  double qx[72];
  int qi[72];
};
union SpreadShare {
  SpreadWave w[4];
  double2 tile[3][kPolTile / 2];          // accumulators of waves 1 .. 3, at the end
};

__global__ void __launch_bounds__(256, 3) k_pol_spread(
    const GeomDev *__restrict__ geoms, const ModelDev *__restrict__ models,
    const Item *__restrict__ items, int n_it, const double *__restrict__ gauss,
    const int *__restrict__ st_ws, const double *__restrict__ pol, double *__restrict__ sens,
    double *__restrict__ pcot) {
  __shared__ PolMath mt;
  __shared__ SpreadShare wv;
  const int lane = threadIdx.x & 63, nd = lane & 7, tl = lane >> 3;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SpreadWave &W = wv.w[wave];
  pol_math_fill(mt);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;          // uniform per block
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const double *dtab = sens + md.sens_off;  // SphAdj::dtab
    const double *tab = gauss + md.gauss_off;
    const double *nt = pcot + md.sgcot_off;
    const PolScale sc = pol_scale(pol, md);
    const double rs0 = 1.0 / sc.s0, iC = sc.iC;
    const int K = g.K, tg = pol_cot_len(K), k0 = it.b * tg, k1 = min(K, k0 + tg);
    const int ia = 2 + kPolR * it.a;
    __syncthreads();                         // tables filled; the previous item's sums
#pragma unroll
    for (int h = 0; h < 8; ++h) W.L[0][h][lane] = W.L[1][h][lane] = 0.0;
    double acc[kPolR + 5][2];
#pragma unroll
    for (int q = 0; q < kPolR + 5; ++q) acc[q][0] = acc[q][1] = 0.0;
    const double glx = g.gl8_x[nd];
    int qn = 0;
    const int chunks = 2 * (k1 - k0);        // 64 pairs each: a tracer, every other radius
    for (int ch = wave; ch < chunks || qn > 0; ch += 4) {
      const bool last = ch + 4 >= chunks;
      int k = 0;
      unsigned long long todo = 0;
      double hs = 0.0;
      if (ch < chunks) {
        k = k0 + (ch >> 1);
        const int ir = 2 * lane + (ch & 1);
        const double r2 = pol_radius2(g, ir);
        hs = 0.5 * log1p(50.0 * (0.5 / tab[k]) / r2) / kSphSeg;
        // the pair's nodes lie within [x0, x0 + kSphSeg hs iX]
        const double x0 = fma(ir * g.sph_dlnr, sc.iX, 2.0), x1 = fma(kSphSeg * hs, sc.iX, x0);
        const bool top = ia + kPolR > kPolN - 4;            // the last bin takes what is clamped
        todo = __ballot(x1 >= (double)ia - 1e-6 && (top || x0 <= (double)(ia + kPolR) + 1e-6) &&
                        !pol_empty(tab[k], tab[K + k], r2));
      }
      while (todo != 0 || (last && qn > 0)) {
        if (todo != 0) {
          const int pl = __builtin_ctzll(todo);
          todo &= todo - 1;
          const int ir = 2 * pl + (ch & 1);
          const double hsp = __shfl(hs, pl, 64);
          const double tau = (tl + 0.5 + 0.5 * glx) * hsp;   // node = lane
          const double x = fma(ir * g.sph_dlnr + tau, sc.iX, 2.0);
          const int i0 = min(max((int)x, 2), kPolN - 4);
          const bool in = i0 >= ia && i0 < ia + kPolR;
          const unsigned long long m = __ballot(in);
          if (in) {
            const int at = qn + __popcll(m & ((1ull << lane) - 1ull));
            W.qx[at] = x;
            W.qi[at] = (k * kSphNR + ir) * 64 + lane;
          }
          qn += __popcll(m);
          wave_sync();
        }
        // whole batches of eight, and at the end what is left
        int q0 = 0;
        const bool flush = last && todo == 0;
        while (qn - q0 >= 8 || (flush && qn > q0)) {
          const bool on = q0 + nd < qn;
          const int id = W.qi[on ? q0 + nd : q0];
          const double x = W.qx[on ? q0 + nd : q0];
          const int i0 = min(max((int)x, 2), kPolN - 4);
          const int kk = id / (kSphNR * 64), ir = (id >> 6) % kSphNR;
          const double s = nt[(int64_t)id * 3], rp2 = nt[(int64_t)id * 3 + 1];
          const double A = on ? nt[(int64_t)id * 3 + 2] : 0.0;
          const double alpha = tab[kk], kap2 = tab[K + kk] - alpha, omb = 1.0 / tab[3 * K + kk];
          {
            double wx[6];
            lagrange<6>(x - i0, wx);
            if (tl == 0)
#pragma unroll
              for (int a = 0; a < 3; ++a) W.wx[nd][a] = make_double2(wx[2 * a], wx[2 * a + 1]);
          }
          const double ea = -alpha * rp2, eq = -kap2 * rp2, kap = 2.0 * kap2;
#pragma unroll 1
          for (int t = 0; t < 3; ++t) {
            const int th = 8 * t + tl;
            const double *dt = dtab + 3 * (ir * kSphNT + th);
            const double lr = dt[0], lt = dt[1], lp = dt[2];
            const double sraw = mt.sn[th] * s, st = fmin(1.0, sraw);
            const double c2 = fma(-st, st, 1.0);
            const double Ae = A * pol_exp(fma(eq, c2, ea), mt);
            const double psi = lp * omb * Ae * rp2 * sraw * st;
            const double phi = fma(kap, psi, fma(omb, lt + lp, lr) * Ae);
            const double y = pol_log(fma(c2, rs0, 1.0), mt) * iC;
            const int l0 = min(max((int)y, 0), kPolC - 8);
            double wy[8];
            lagrange<8>(y - l0, wy);
            // Step b adds the stencil column c with c % 8 = (b + tl) % 8: the
            // eight angles of a node, which may share columns, are then at
            // eight different ones, so that the order of the adds is that of
            // the steps.  The weights are rotated into that order.
            const int d = (tl - l0) & 7;
            rotate8<1>(wy, d);
            rotate8<2>(wy, d);
            rotate8<4>(wy, d);
            double *o = &W.L[0][nd][l0];
#pragma unroll
            for (int b = 0; b < 8; ++b) {
              double *c = o + ((b + d) & 7);
              unsafeAtomicAdd(c, wy[b] * phi);
              unsafeAtomicAdd(c + 8 * (kPolC + 1), wy[b] * psi);
            }
          }
          wave_sync();
          const int nb = min(8, qn - q0);
          for (int h = 0; h < nb; ++h) {
            const double2 v = make_double2(W.L[0][h][lane], W.L[1][h][lane]);
            W.L[0][h][lane] = W.L[1][h][lane] = 0.0;
            const double2 a0 = W.wx[h][0], a1 = W.wx[h][1], a2 = W.wx[h][2];
            const int off = __builtin_amdgcn_readlane(i0, h) - ia;
#pragma unroll
            for (int o = 0; o < kPolR; ++o)
              if (off == o) {
                acc[o][0] = fma(a0.x, v.x, acc[o][0]);
                acc[o][1] = fma(a0.x, v.y, acc[o][1]);
                acc[o + 1][0] = fma(a0.y, v.x, acc[o + 1][0]);
                acc[o + 1][1] = fma(a0.y, v.y, acc[o + 1][1]);
                acc[o + 2][0] = fma(a1.x, v.x, acc[o + 2][0]);
                acc[o + 2][1] = fma(a1.x, v.y, acc[o + 2][1]);
                acc[o + 3][0] = fma(a1.y, v.x, acc[o + 3][0]);
                acc[o + 3][1] = fma(a1.y, v.y, acc[o + 3][1]);
                acc[o + 4][0] = fma(a2.x, v.x, acc[o + 4][0]);
                acc[o + 4][1] = fma(a2.x, v.y, acc[o + 4][1]);
                acc[o + 5][0] = fma(a2.y, v.x, acc[o + 5][0]);
                acc[o + 5][1] = fma(a2.y, v.y, acc[o + 5][1]);
              }
          }
          wave_sync();
          q0 += 8;
        }
        // what is left moves to the front (fewer than eight entries)
        q0 = min(q0, qn);
        if (q0 > 0) {
          const int left = qn - q0;
          double x = 0.0;
          int id = 0;
          if (lane < left) { x = W.qx[q0 + lane]; id = W.qi[q0 + lane]; }
          wave_sync();
          if (lane < left) { W.qx[lane] = x; W.qi[lane] = id; }
          qn = left;
          wave_sync();
        }
      }
      if (last) break;
    }
    __syncthreads();                         // every wave has done its nodes
    if (wave > 0)
#pragma unroll
      for (int q = 0; q < kPolR + 5; ++q)
        wv.tile[wave - 1][q * kPolC + lane] = make_double2(acc[q][0], acc[q][1]);
    __syncthreads();
    if (wave == 0) {
      double2 *o = reinterpret_cast<double2 *>(
          pcot + md.sgcot_off + pol_nodes(K) + (int64_t)(it.b * kPolBins + it.a) * kPolTile);
#pragma unroll
      for (int q = 0; q < kPolR + 5; ++q) {
        double2 v = make_double2(acc[q][0], acc[q][1]);
#pragma unroll
        for (int w = 0; w < 3; ++w) {
          const double2 u = wv.tile[w][q * kPolC + lane];
          v.x += u.x;
          v.y += u.y;
        }
        o[q * kPolC + lane] = v;
      }
    }
  }
}

// Item (m, block of 256 grid points): the bins' tiles and the tracer groups
// added in order, to FP32 (phi, psi).
__global__ void __launch_bounds__(256) k_pol_cot_sum(const GeomDev *__restrict__ geoms,
                                                     const ModelDev *__restrict__ models,
                                                     const Item *__restrict__ items, int n_it,
                                                     const int *__restrict__ st_ws,
                                                     double *__restrict__ pcot) {
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;
    const ModelDev md = models[it.m];
    const int K = geoms[md.geom].K, ng = pol_cot_groups(K);
    const double *tiles = pcot + md.sgcot_off + pol_nodes(K);
    float2 *fl = reinterpret_cast<float2 *>(pcot + md.sgcot_off + pol_nodes(K) +
                                            (int64_t)ng * kPolBins * kPolTile);
    const int p = it.a * 256 + threadIdx.x, row = p / kPolC, col = p % kPolC;
    const int b1 = row / kPolR;              // bins whose tile [kPolR b, + kPolR + 5) has the row
    double va = 0.0, vb = 0.0;
    for (int q = 0; q < ng; ++q)
      for (int b = max(0, b1 - 1); b <= min(b1, kPolBins - 1); ++b) {
        const int rr = row - kPolR * b;
        if (rr >= kPolR + 5) continue;
        const double2 v = *reinterpret_cast<const double2 *>(
            tiles + (int64_t)(q * kPolBins + b) * kPolTile + (rr * kPolC + col) * 2);
        va += v.x;
        vb += v.y;
      }
    fl[p] = make_float2((float)va, (float)vb);
  }
}

// Term sensitivities from the grid cotangent: item (m, 512-term tile, part of
// kPolN / kPolParts rows); thread = two terms, which share each point's LDS
// reads (wave-wide broadcasts; with one term per thread the reads are the
// bound).  Per term S_phi = sum phi E, S_psi and their z'^2 moments, FP32 over a
// row of 64 points, FP64 across rows.  On a row r'^2 is fixed: the exponent, in FP64
// as in k_pol_grid_adj, is one multiply-add from c.x r'^2.  An FP64 multiply-add, an
// exponential and four FP32 multiply-adds per term and point bound it.
// Measured (48 models of 1300 terms / one of 5248): on the 512 x 512 grid with
// matrix cores 1132 / 129 us, here 400 / 64 (325 / 52 with FP32 exponents).
__global__ void __launch_bounds__(256) k_pol_sens(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  const double *__restrict__ terms64,
                                                  const int *__restrict__ st_ws,
                                                  const double *__restrict__ pol,
                                                  double *__restrict__ sens,
                                                  const double *__restrict__ pcot) {
  constexpr int kRows = kPolN / kPolParts;
  static_assert(kRows % 4 == 0 && kPolN % kPolParts == 0, "four rows at a time");
  __shared__ float4 pc[4][kPolC];            // (phi, psi, phi z'^2, psi z'^2)
  __shared__ double pz[4][kPolC];            // z'^2
  __shared__ double rr[4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;          // uniform per block
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const PolScale sc = pol_scale(pol, md);
    const int K = g.K, Tp = sph_terms_padded(g.J1, g.n_u);
    const float2 *fl = reinterpret_cast<const float2 *>(
        pcot + md.sgcot_off + pol_nodes(K) + (int64_t)pol_cot_groups(K) * kPolBins * kPolTile);
    const SphTerm *tc = reinterpret_cast<const SphTerm *>(terms64 + md.term64_off);
    double cx[2], dz[2], SP[2], ST[2], ZP[2], ZT[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = it.a * 512 + 256 * u + threadIdx.x;
      cx[u] = t < Tp ? tc[t].cx : 0.0;
      dz[u] = t < Tp ? tc[t].cy - cx[u] : 0.0;
      SP[u] = ST[u] = ZP[u] = ZT[u] = 0.0;
    }
    const double c2 = pol_col_c2(sc, lane), reach = pol_reach(sc);
    double cmax = fmax(cx[0], cx[1]);
    for (int o = 32; o > 0; o >>= 1) cmax = fmax(cmax, __shfl_xor(cmax, o, 64));
    for (int q0 = it.b * kRows; q0 < (it.b + 1) * kRows; q0 += 4) {
      const double r2 = pol_row_r2(g, sc, q0 + wave), z2 = r2 * c2;
      const float2 f = fl[(q0 + wave) * kPolC + lane];
      __syncthreads();                       // the previous rows read
      pc[wave][lane] = make_float4(f.x, f.y, f.x * (float)z2, f.y * (float)z2);
      pz[wave][lane] = z2;
      if (lane == 0) rr[wave] = r2;
      __syncthreads();
      for (int w = 0; w < 4; ++w) {
        // a row where every term of the wave underflows adds exact zeros
        if (cmax * (rr[w] * reach) < -160.0) continue;
        float sP[2] = {0.f, 0.f}, sT[2] = {0.f, 0.f}, zP[2] = {0.f, 0.f}, zT[2] = {0.f, 0.f};
        const double r = rr[w];
        const double a[2] = {cx[0] * r, cx[1] * r};
#pragma unroll 16
        for (int l = 0; l < kPolC; ++l) {
          const float4 p = pc[w][l];
          const double z = pz[w][l];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const float e = fast_exp2((float)fma(dz[u], z, a[u]));
            sP[u] = fmaf(p.x, e, sP[u]);
            sT[u] = fmaf(p.y, e, sT[u]);
            zP[u] = fmaf(p.z, e, zP[u]);
            zT[u] = fmaf(p.w, e, zT[u]);
          }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          SP[u] += (double)sP[u];
          ST[u] += (double)sT[u];
          ZP[u] += (double)zP[u];
          ZT[u] += (double)zT[u];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = it.a * 512 + 256 * u + threadIdx.x;
      if (t >= Tp) continue;
      double *o = sph_adj_layout(sens + md.sens_off, K, g.n_pix, Tp, md.n_sens_parts).sparts +
                  ((int64_t)it.b * Tp + t) * 4;
      o[0] = SP[u];
      o[1] = ST[u];
      o[2] = ZP[u];
      o[3] = ZT[u];
    }
  }
}

}  // namespace

namespace {
unsigned grid_of(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(n, 1 << 22)); }
}  // namespace

void launch_pol_grid(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                     const Item *it_sum, int n_sum, const float4 *terms, const int *st_ws,
                     const double *pol, float *sgrid, hipStream_t st) {
  hipLaunchKernelGGL(k_pol_grid, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, terms,
                     st_ws, pol, sgrid);
  if (n_sum)
    hipLaunchKernelGGL(k_pol_grid_sum, dim3(grid_of(n_sum)), dim3(256), 0, st, m, it_sum, n_sum,
                       st_ws, sgrid);
}
void launch_pol_grid_adj(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                         const Item *it_sum, int n_sum, const double *terms64, const int *st_ws,
                         const double *pol, double *sgrid3, hipStream_t st) {
  hipLaunchKernelGGL(k_pol_grid_adj, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, terms64,
                     st_ws, pol, sgrid3);
  if (n_sum)
    hipLaunchKernelGGL(k_pol_grid_sum_adj, dim3(grid_of(n_sum)), dim3(256), 0, st, m, it_sum, n_sum,
                       st_ws, sgrid3);
}
void launch_pol_moments(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                        const Item *it_tab, int n_tab, const double *gauss, const float4 *terms,
                        const int *st_ws, const float *sgrid, double *pol, double *table,
                        hipStream_t st) {
  hipLaunchKernelGGL(k_pol_moments<false>, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it,
                     gauss, st_ws, sgrid, pol, nullptr, nullptr);
  hipLaunchKernelGGL(k_pol_table<false>, dim3(grid_of(n_tab)), dim3(256), 0, st, g, m, it_tab,
                     n_tab, gauss, terms, nullptr, st_ws, pol, table, nullptr);
}
void launch_pol_moments_adj(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                            const Item *it_tab, int n_tab, const double *gauss,
                            const double *terms64, const int *st_ws, const double *sgrid3,
                            double *pol, double *table, double *sens, double *pcot,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_pol_moments<true>, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it,
                     gauss, st_ws, sgrid3, pol, sens, pcot);
  hipLaunchKernelGGL(k_pol_table<true>, dim3(grid_of(n_tab)), dim3(256), 0, st, g, m, it_tab, n_tab,
                     gauss, nullptr, terms64, st_ws, pol, table, sens);
}
void launch_pol_adjoint(const GeomDev *g, const ModelDev *m, const Item *it_spread, int n_spread,
                        const Item *it_sum, int n_sum, const Item *it_sens, int n_sens,
                        const double *gauss, const double *terms64, const int *st_ws,
                        const double *pol, double *sens, double *pcot, hipStream_t st) {
  hipLaunchKernelGGL(k_pol_spread, dim3(grid_of(n_spread)), dim3(256), 0, st, g, m, it_spread,
                     n_spread, gauss, st_ws, pol, sens, pcot);
  hipLaunchKernelGGL(k_pol_cot_sum, dim3(grid_of(n_sum)), dim3(256), 0, st, g, m, it_sum, n_sum,
                     st_ws, pcot);
  hipLaunchKernelGGL(k_pol_sens, dim3(grid_of(n_sens)), dim3(256), 0, st, g, m, it_sens, n_sens,
                     terms64, st_ws, pol, sens, pcot);
}

}  // namespace jam
