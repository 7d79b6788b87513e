// gfx950 kernels of the JAM-cyl forward model and its adjoint.
//
// The numerator map of eq. (VLos) is, per sky point (x', y'),
//   N = sum_{k,j,n} exp(-c1 x'^2 - gamma y'^2) (C0 + C1 x'^2),
// one term per luminous Gaussian k, mass Gaussian j (BH last) and
// Gauss-Legendre node u_n (the u-integral of the deprojected-MGE potential);
// the term coefficients follow from the App. A deprojection and the
// cylindrically aligned Jeans solution.  Derivation per term, with
// alpha = 1/(2 sigma_k^2), r = 1/(2 sigma_j^2), h = 1 - e_j^2 u^2:
//   c1 = alpha + r u^2,  A = alpha/q_k^2 + r u^2 / h,
//   a = c1 sin^2 i + A cos^2 i,  gamma = c1 A / a,
//   g = nu0 K r u^2 / (A h^{3/2})   (nu v_z^2 amplitude),
//   w = 2 nu0 K r u^2 / h^{1/2}      (nu R^-1 dPhi/dR amplitude),
//   P = (cos^2 i + b sin^2 i) g,  Q = sin^2 i (w - 2 c1 b g),
//   C0 = w_n sqrt(pi/a) P,  C1 = w_n sqrt(pi/a) Q,
// with nu0 the deprojected peak density (App. A), K = sqrt(2/pi) G M/(s sigma_j)
// and b = 1/(1 - beta_k).
//
// Precision: the set-up and term coefficients are FP64 and stored as FP32
// (with log2(e) folded into the exponent coefficients for v_exp_f32); the
// integrand sums run in FP32 per (k, j) group of u-nodes and are folded into
// FP64 accumulators; the surface brightness, bin sums and the final division
// are FP64.
#include "jam_device.h"
#include "jam_internal.h"
#include "jam_sph_math.h"

#include <hip/hip_runtime.h>
#include <algorithm>
#include <cmath>
#include <type_traits>

namespace jam {

namespace {

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Split-term partial maps are stored per slice on the unique-pixel map padded
// to whole 32x32 blocks and transposed (y fastest): element (x, y) at
// x * 32 n_yt + y, 32 n_xt * 32 n_yt doubles per slice.  A wave's MFMA tile
// then stores 32 consecutive y values per instruction.
__device__ inline int64_t part_slice_size(const ModelDev &md) {
  return (int64_t)(32 * md.n_xt) * (32 * md.n_yt);
}
__device__ inline int64_t part_index(const ModelDev &md, const GeomDev &g, int q) {
  return (int64_t)(q % g.n_ux) * (32 * md.n_yt) + q / g.n_ux;
}

// Deterministic block sum of one double over a 256-thread block.
__device__ double block_sum256(double v, double *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) sh[t] += sh[t + s];
    __syncthreads();
  }
  double r = sh[0];
  __syncthreads();
  return r;
}

// Eight wave sums at once, in a fixed order: three halving exchanges (lanes
// 32 apart swap halves of the eight values, then 16 apart, then 8 apart)
// leave each lane a partial of value lane / 8, and three butterflies over
// the lane's group of eight finish it.  Returns the full sum of value
// lane / 8 in every lane of group lane / 8 (10 exchanges instead of 48).
__device__ inline double wave_sum8(const double (&v)[8], int lane) {
  const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
  double w[4], x[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double keep = h5 ? v[i + 4] : v[i], send = h5 ? v[i] : v[i + 4];
    w[i] = keep + __shfl_xor(send, 32, 64);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = h4 ? w[i + 2] : w[i], send = h4 ? w[i] : w[i + 2];
    x[i] = keep + __shfl_xor(send, 16, 64);
  }
  const double keep = h3 ? x[1] : x[0], send = h3 ? x[0] : x[1];
  double y = keep + __shfl_xor(send, 8, 64);
  y += __shfl_xor(y, 4, 64);
  y += __shfl_xor(y, 2, 64);
  y += __shfl_xor(y, 1, 64);
  return y;
}

// ---------------------------------------------------------------------------
// Set-up: App. A deprojection and per-Gaussian derived quantities (FP64),
// per-model validity.
// ---------------------------------------------------------------------------
// One model's set-up; every thread of the block calls it (block-wide ORs).
__device__ void setup_item(const GeomDev *__restrict__ geoms, const ModelDev *__restrict__ models,
                           int m, const ParamsDev &p, double *__restrict__ gauss,
                           int *__restrict__ st_ws, int32_t *__restrict__ st_out) {
  const ModelDev md = models[m];
  const GeomDev g = geoms[md.geom];
  double *tab = gauss + md.gauss_off;
  const double inc = p.inc[m];
  const double si = sin(inc), ci = cos(inc);
  const double si2 = si * si, ci2 = ci * ci;
  const double ml = p.mass_scale[m];
  const double mbh = p.m_bh[m];
  const double G = grav_const();
  const double s = g.s_pc;
  int bad_dep = !(si > 0.0) || !isfinite(inc);
  int bad_phys = !(ml >= 0.0) || !(mbh >= 0.0) || !isfinite(ml) || !isfinite(mbh);
  const int K = g.K, J = g.J1 - 1;
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    const double qo = g.lum_q[k], sig = g.lum_sigma[k];
    const double I0 = p.lum_I0 ? p.lum_I0[md.lum_off + k] : g.lum_I0[k];
    const double beta = p.beta[md.lum_off + k];
    if (!(qo * qo > ci2)) bad_dep = 1;
    if (!(beta < 1.0) || !(I0 >= 0.0) || !isfinite(I0)) bad_phys = 1;
    const double q = sqrt(fmax(qo * qo - ci2, 0.0)) / si;
    const double alpha = 0.5 / (sig * sig);
    tab[k] = alpha;
    tab[K + k] = alpha / (q * q);
    tab[2 * K + k] = qo * I0 / (sqrt(2.0 * kPi) * sig * q);
    tab[3 * K + k] = 1.0 / (1.0 - beta);
  }
  double *mt = tab + 4 * K;
  for (int j = threadIdx.x; j < J + 1; j += blockDim.x) {
    double r, e2, Kp;
    if (j < J) {
      const double qo = g.mass_q[j], sig = g.mass_sigma[j];
      const double S0 = p.mass_S0 ? p.mass_S0[md.mass_off + j] : g.mass_S0[j];
      if (!(qo * qo > ci2)) bad_dep = 1;
      if (!(S0 >= 0.0) || !isfinite(S0)) bad_phys = 1;
      const double q = sqrt(fmax(qo * qo - ci2, 0.0)) / si;
      const double M = ml * 2.0 * kPi * S0 * (s * sig) * (s * sig) * qo;
      r = 0.5 / (sig * sig);
      e2 = 1.0 - q * q;
      Kp = sqrt(2.0 / kPi) * G * M / (s * sig);
    } else {
      r = 0.5 / (g.bh_sigma * g.bh_sigma);
      e2 = 0.0;
      Kp = sqrt(2.0 / kPi) * G * mbh / (s * g.bh_sigma);
    }
    mt[j] = r;
    mt[g.J1 + j] = e2;
    mt[2 * g.J1 + j] = Kp;
  }
  if (threadIdx.x == 0) {
    mt[3 * g.J1] = si2;
    mt[3 * g.J1 + 1] = ci2;
  }
  const int any_dep = __syncthreads_or(bad_dep);
  const int any_phys = __syncthreads_or(bad_phys);
  if (threadIdx.x == 0) {
    const int code = any_dep ? 2 : (any_phys ? 3 : 0);
    st_ws[m] = code;
    if (st_out) st_out[m] = code;
  }
}

__global__ void __launch_bounds__(64) k_setup(const GeomDev *__restrict__ geoms,
                                              const ModelDev *__restrict__ models, int n,
                                              ParamsDev p, double *__restrict__ gauss,
                                              int *__restrict__ st_ws, int32_t *__restrict__ st_out,
                                              int *__restrict__ queues) {
  // Work-queue counters of the kernels that follow on the stream.
  if (queues && blockIdx.x == 0 && threadIdx.x < 2) queues[threadIdx.x] = 0;
  for (int m = blockIdx.x; m < n; m += gridDim.x)
    setup_item(geoms, models, m, p, gauss, st_ws, st_out);
}

constexpr int kSbChunk = 256 / kSbRows;   // Gaussians a block's threads form row factors of

// Row factors exp(-y^2 / 2 sigma'^2 q'^2) of the Gaussians k0 .. k0 + kSbChunk on
// a tile's rows, one a thread, and 1 / 2 sigma'^2 (block call).  They are the same
// in every column: an exponential per row in each wave was nine tenths of a
// tile's exponentials.  Measured (4096 models of 10 Gaussians on 19 x 19 pixels /
// 3476 of 9 on 76 x 76): k_prologue<false> 85 / 443 us with them, 45 / 277 here;
// k_sb_adj of the latter 406, here 194.
__device__ __forceinline__ void sb_row_factors(const GeomDev &g, int y0, int k0,
                                               double (*rf)[kSbRows + 1]) {
  const int kk = threadIdx.x / kSbRows, r = threadIdx.x % kSbRows, k = k0 + kk;
  __syncthreads();                 // the previous factors have been read
  if (k < g.K) {
    const double sig = g.lum_sigma[k], qo = g.lum_q[k];
    const double a = 1.0 / (2.0 * sig * sig);
    const double ay = a / (qo * qo), y = y0 + r < g.n_uy ? g.ys[y0 + r] : 0.0;
    rf[kk][r] = exp(-ay * (y * y));
    if (r == 0) rf[kk][kSbRows] = a;
  }
  __syncthreads();
}

// Surface-brightness adjoint: the derivative of sum_p lambda_I[p] I[p] with
// respect to I0_k, per tile of kSbRows rows x 64 columns (the forward's
// items): lane = column, waves split the Gaussians; FP64, wave sums; the
// per-tile partials are summed by the gradient kernels in tile order.
__global__ void __launch_bounds__(256) k_sb_adj(const GeomDev *__restrict__ geoms,
                                                const ModelDev *__restrict__ models,
                                                const Item *__restrict__ items, int n_it,
                                                const int *__restrict__ st_ws,
                                                const double *__restrict__ pix,
                                                double *__restrict__ sbp) {
  __shared__ double rf[kSbChunk][kSbRows + 1];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;
    const int y0 = it.a * kSbRows;
    const int ix = it.b * 64 + lane;
    const bool vx = ix < g.n_ux;
    const double x = vx ? g.xs[ix] : 0.0;
    const double *lamI = pix + md.pix_off + 3 * (int64_t)g.n_pix;
    double lam[kSbRows];
#pragma unroll
    for (int r = 0; r < kSbRows; ++r) {
      const bool v = vx && y0 + r < g.n_uy;
      lam[r] = v ? lamI[(int64_t)(y0 + r) * g.n_ux + ix] : 0.0;
    }
    const int tile = it.a * ((g.n_ux + 63) / 64) + it.b;
    const int n_tiles = sb_tiles(g.n_ux, g.n_uy);
    for (int k0 = 0; k0 < g.K; k0 += kSbChunk) {
      sb_row_factors(g, y0, k0, rf);
      for (int k = k0 + wave; k < min(g.K, k0 + kSbChunk); k += 4) {
        const double a = rf[k - k0][kSbRows];
        double acc = 0.0;
#pragma unroll
        for (int r = 0; r < kSbRows; ++r) acc += lam[r] * rf[k - k0][r];
        acc = wave_sum(acc * exp(-a * x * x));
        if (lane == 0) sbp[md.sbp_off + (int64_t)k * n_tiles + tile] = acc;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Term table: FP64 coefficients of every (k, j, n) term, stored as FP32
// (-c1 log2e, -gamma log2e, C0, C1).  Term t = (k * J1 + j) * n_u + n.
// ---------------------------------------------------------------------------
__device__ inline void term_coeffs(double alpha, double alphaq, double nu0, double b, double r,
                                   double e2, double Kp, double si2, double ci2, double u,
                                   double wq, double &c1, double &gam, double &C0, double &C1) {
  const double u2 = u * u;
  const double h = fma(-e2, u2, 1.0);
  const double ru2 = r * u2;
  c1 = alpha + ru2;
  const double rsh = rsq64(h), rh = rsh * rsh;
  const double A = fma(ru2, rh, alphaq);
  const double a = fma(c1, si2, A * ci2);
  const double rsa = rsq64(a);
  gam = c1 * A * rsa * rsa;
  const double base = nu0 * Kp * ru2;
  const double gg = base * rcp64(A) * rh * rsh;
  const double ww = 2.0 * base * rsh;
  const double P = (ci2 + b * si2) * gg;
  const double Q = si2 * (ww - 2.0 * c1 * b * gg);
  const double f = wq * kSqrtPi * rsa;
  C0 = f * P;
  C1 = f * Q;
}

// Term t = (k * J1 + j) * n_u + n of a model from its Gaussian table (the
// set-up's output), as the term table stores it.
__device__ inline float4 term_at(const GeomDev &g, const double *__restrict__ tab, int k, int j,
                                 int n) {
  const double *mt = tab + 4 * g.K;
  double c1, gam, C0, C1;
  term_coeffs(tab[k], tab[g.K + k], tab[2 * g.K + k], tab[3 * g.K + k], mt[j], mt[g.J1 + j],
              mt[2 * g.J1 + j], mt[3 * g.J1], mt[3 * g.J1 + 1], load_global(g.u + n),
              load_global(g.w + n), c1, gam, C0, C1);
  return make_float4((float)(-c1 * kLog2e), (float)(-gam * kLog2e), (float)C0, (float)C1);
}
__device__ inline float4 term_of(const GeomDev &g, const double *__restrict__ tab, int t) {
  const int n = t % g.n_u, kj = t / g.n_u;
  return term_at(g, tab, kj / g.J1, kj % g.J1, n);
}

// The per-(k, j) quantities of the set-up straight from the parameters (its
// formulas and operation order), for kernels that run beside the set-up:
// v = (alpha, alphaq, nu0, b, r, e2, Kp, si2, ci2).
__device__ inline void pair_from_params(const GeomDev &g, const ModelDev &md, int m,
                                        const ParamsDev &p, int k, int j, double *v) {
  const double inc = p.inc[m];
  const double si = sin(inc), ci = cos(inc);
  const double si2 = si * si, ci2 = ci * ci;
  const double qo = g.lum_q[k], sig = g.lum_sigma[k];
  const double I0 = p.lum_I0 ? p.lum_I0[md.lum_off + k] : g.lum_I0[k];
  const double q = sqrt(fmax(qo * qo - ci2, 0.0)) / si;
  const double alpha = 0.5 / (sig * sig);
  v[0] = alpha;
  v[1] = alpha / (q * q);
  v[2] = qo * I0 / (sqrt(2.0 * kPi) * sig * q);
  v[3] = 1.0 / (1.0 - p.beta[md.lum_off + k]);
  const double G = grav_const(), sp = g.s_pc;
  if (j < g.J1 - 1) {
    const double qoj = g.mass_q[j], sj = g.mass_sigma[j];
    const double S0 = p.mass_S0 ? p.mass_S0[md.mass_off + j] : g.mass_S0[j];
    const double qj = sqrt(fmax(qoj * qoj - ci2, 0.0)) / si;
    const double M = p.mass_scale[m] * 2.0 * kPi * S0 * (sp * sj) * (sp * sj) * qoj;
    v[4] = 0.5 / (sj * sj);
    v[5] = 1.0 - qj * qj;
    v[6] = sqrt(2.0 / kPi) * G * M / (sp * sj);
  } else {
    v[4] = 0.5 / (g.bh_sigma * g.bh_sigma);
    v[5] = 0.0;
    v[6] = sqrt(2.0 / kPi) * G * p.m_bh[m] / (sp * g.bh_sigma);
  }
  v[7] = si2;
  v[8] = ci2;
}

// ---------------------------------------------------------------------------
// Surface brightness, eq. (sb_mge_2D), FP64, on the unique-pixel map, using
// its separability: I(x, y) = sum_k I0_k exp(-x^2/2s_k^2) exp(-y^2/2s_k^2q_k^2).
// Item (m, block of 8 rows, block of 64 columns): the row factors are
// computed once per workgroup, the column factor once per thread and k.
// pix region per model: [N | I | lambda_N | lambda_I], n_pix doubles each.
// ---------------------------------------------------------------------------

// Item (m, block of 8 rows, block of 64 columns); lane = column, wave w takes
// luminous Gaussians k = w, w + 4, ...; the four partial sums are combined in
// a fixed order.
// One surface-brightness tile; every thread of the block calls it.
__device__ void sb_item(const Item &it, const ModelDev &md, const GeomDev &g, const ParamsDev &p,
                        double *__restrict__ pix, double (*red)[kSbRows][64],
                        double (*rf)[kSbRows + 1]) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int y0 = it.a * kSbRows;
  const int ix = it.b * 64 + lane;
  const bool vx = ix < g.n_ux;
  const double x = vx ? g.xs[ix] : 0.0;
  double acc[kSbRows];
#pragma unroll
  for (int r = 0; r < kSbRows; ++r) acc[r] = 0.0;
  for (int k0 = 0; k0 < g.K; k0 += kSbChunk) {
    sb_row_factors(g, y0, k0, rf);
    for (int k = k0 + wave; k < min(g.K, k0 + kSbChunk); k += 4) {
      const double I0 = p.lum_I0 ? p.lum_I0[md.lum_off + k] : g.lum_I0[k];
      const double a = rf[k - k0][kSbRows];
      const double fx = I0 * exp(-a * x * x);
#pragma unroll
      for (int r = 0; r < kSbRows; ++r) acc[r] += fx * rf[k - k0][r];
    }
  }
  if (wave > 0)
#pragma unroll
    for (int r = 0; r < kSbRows; ++r) red[wave - 1][r][lane] = acc[r];
  __syncthreads();
  if (wave == 0 && vx) {
#pragma unroll
    for (int r = 0; r < kSbRows; ++r)
      if (y0 + r < g.n_uy)
        pix[md.pix_off + g.n_pix + (int64_t)(y0 + r) * g.n_ux + ix] =
            ((acc[r] + red[0][r][lane]) + red[1][r][lane]) + red[2][r][lane];
  }
  __syncthreads();
}

__global__ void __launch_bounds__(256) k_sb(const GeomDev *__restrict__ geoms,
                                            const ModelDev *__restrict__ models,
                                            const Item *__restrict__ items, int n_it, ParamsDev p,
                                            double *__restrict__ pix) {
  __shared__ double red[3][kSbRows][64];
  __shared__ double rf[kSbChunk][kSbRows + 1];
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    sb_item(it, md, g, p, pix, red, rf);
  }
}

// Prologue of the cylindrical model: items of four kinds (Item::c): 0 set-up
// of model m (status, Gaussian table); 1 a block of 256 FP32 terms computed
// straight from the parameters, so it needs nothing from set-up items running
// in the same launch (a model with a bad status gets meaningless terms, which
// every later kernel skips); 2 a surface-brightness tile; 3 a block of terms
// from the Gaussian table of a set-up that ran in an earlier launch (zero
// terms for a bad status).  One launch of kinds 0, 1, 2 suits a few large
// models; many small ones run the set-up first and then kinds 2 and 3, which
// avoids recomputing each (k, j) pair's set-up in every term block.
template <bool kFused>
__global__ void __launch_bounds__(256) k_prologue(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  ParamsDev p, double *__restrict__ gauss,
                                                  int *__restrict__ st_ws,
                                                  int32_t *__restrict__ st_out,
                                                  int *__restrict__ queues,
                                                  float4 *__restrict__ terms,
                                                  double *__restrict__ pix) {
  __shared__ double red[3][kSbRows][64];
  __shared__ double rf[kSbChunk][kSbRows + 1];
  // per-(k, j) quantities of a term block (kind 1 only)
  __shared__ double pv[kFused ? 258 : 1][9];
  if (queues && blockIdx.x == 0 && threadIdx.x < 2) queues[threadIdx.x] = 0;
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (kFused && it.c == 0) {       // uniform per block
      setup_item(geoms, models, it.m, p, gauss, st_ws, st_out);
      continue;
    }
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (it.c == 2) {
      sb_item(it, md, g, p, pix, red, rf);
      continue;
    }
    if (!kFused) {                   // kind 3
      const int t = it.a * 256 + threadIdx.x;
      if (t < g.T)
        terms[md.term_off + t] = st_ws[it.m] == 0 ? term_of(g, gauss + md.gauss_off, t)
                                                  : make_float4(0.f, 0.f, 0.f, 0.f);
      else if (t < padded_terms(g.T))
        terms[md.term_off + t] = make_float4(0.f, 0.f, 0.f, 0.f);
      continue;
    }
    // kind 1: the (k, j) pairs of this block's 256 terms, once each, then
    // the terms
    const int t0 = it.a * 256;
    const int kj0 = t0 / g.n_u, kj1 = (min(t0 + 256, g.T) - 1) / g.n_u;
    for (int q = threadIdx.x; q <= kj1 - kj0; q += 256)
      pair_from_params(g, md, it.m, p, (kj0 + q) / g.J1, (kj0 + q) % g.J1, pv[q]);
    __syncthreads();
    const int t = t0 + threadIdx.x;
    if (t < g.T) {
      const int n = t % g.n_u;
      const double *v = pv[t / g.n_u - kj0];
      double c1, gam, C0, C1;
      term_coeffs(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], g.u[n], g.w[n], c1, gam,
                  C0, C1);
      terms[md.term_off + t] =
          make_float4((float)(-c1 * kLog2e), (float)(-gam * kLog2e), (float)C0, (float)C1);
    } else if (t < padded_terms(g.T)) {
      terms[md.term_off + t] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Per-pixel VALU quadrature.  Item (m, block of 256 unique pixels, slice of
// (k, j) pairs); thread = pixel.  The slice's terms are staged through LDS
// in runs of whole (k, j) pairs (at most kPixStage terms), read back as
// broadcasts (the same address in every lane); per pair the integrand is
// summed over the u-nodes in FP32 and folded into an FP64 accumulator.
// ---------------------------------------------------------------------------
constexpr int kPixStage = 1024;

__device__ __forceinline__ void num_pix_item(const Item it, const GeomDev *__restrict__ geoms,
    const ModelDev *__restrict__ models, const float4 *__restrict__ terms, const int *__restrict__ st_ws, double *__restrict__ part, float4 *stage) {
  const ModelDev md = models[it.m];
  const GeomDev g = geoms[md.geom];
  const int q = it.a * 256 + threadIdx.x;
  const bool valid = q < g.n_pix;
  float x2 = 0.f, y2 = 0.f;
  if (valid) {
    const double x = g.xs[q % g.n_ux], y = g.ys[q / g.n_ux];
    x2 = (float)(x * x);
    y2 = (float)(y * y);
  }
  const int n_pairs = g.K * g.J1;
  const int per = (n_pairs + md.n_slices - 1) / md.n_slices;
  const int p0 = it.b * per;
  const int p1 = min(n_pairs, p0 + per);
  const int nu = __builtin_amdgcn_readfirstlane(g.n_u);
  const int run = max(1, kPixStage / nu);   // pairs per LDS run
  double acc = 0.0;
  if (st_ws[it.m] == 0) {
    const float4 *tb = terms + md.term_off;
    for (int r0 = p0; r0 < p1; r0 += run) {
      const int r1 = min(p1, r0 + run);
      const int nt = (r1 - r0) * nu;
      __syncthreads();                 // the previous run's reads are done
      for (int e = threadIdx.x; e < nt; e += 256) stage[e] = tb[(int64_t)r0 * nu + e];
      __syncthreads();
      for (int pr = 0; pr < r1 - r0; ++pr) {
        const float4 *tp = stage + pr * nu;
        float s = 0.f;
        int n = 0;
        for (; n + 4 <= nu; n += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float4 c = tp[n + u];
            const float e = fast_exp2(fmaf(c.x, x2, c.y * y2));
            s = fmaf(e, fmaf(c.w, x2, c.z), s);
          }
        }
        for (; n < nu; ++n) {
          const float4 c = tp[n];
          const float e = fast_exp2(fmaf(c.x, x2, c.y * y2));
          s = fmaf(e, fmaf(c.w, x2, c.z), s);
        }
        acc += (double)s;
      }
    }
  }
  if (valid) part[md.part_off + it.b * part_slice_size(md) + part_index(md, g, q)] = acc;
}


// ---------------------------------------------------------------------------
// Separable matrix-core form.  On the unique-pixel map
//   N[x, y] = sum_t A[x, t] B[y, t],
//   A[x, t] = 2^(cx_t x^2) (C0_t + C1_t x^2),   B[y, t] = 2^(cy_t y^2),
// an exact factorisation of the same sum, evaluated as a dense FP32
// contraction over terms with v_mfma_f32_32x32x2f32.  Each 32x32 output
// block accumulates a chunk of 64 terms in FP32 and folds it into FP64.
//
// Operand layout of v_mfma_f32_32x32x2f32 (lane l): A[l % 32][l / 32],
// B[l / 32][l % 32]; accumulator r of lane l is D[i][j] with
// i = (r % 4) + 4 (l / 32) + 8 (r / 4), j = l % 32.
// ---------------------------------------------------------------------------
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ inline int mfma_row(int r, int lane) { return (r & 3) + 4 * (lane >> 5) + 8 * (r >> 2); }

constexpr int KC2 = 64;  // terms per chunk of the matrix-core numerator


// Term range of one slice, in whole chunks of `unit` terms.
__device__ inline void slice_range(int T, int n_slices, int slice, int &t0, int &t1,
                                   int unit) {
  const int chunks = (T + unit - 1) / unit;
  const int per = (chunks + n_slices - 1) / n_slices;
  t0 = min(T, slice * per * unit);
  t1 = min(T, t0 + per * unit);
}

// One workgroup, one item: an output tile of BX x BY blocks of 32x32 unique
// pixels (BX along x, BY along y) over one slice of the terms; the four
// waves take contiguous quarters of the slice in chunks of 64 terms.  Lane l
// generates the operands of its row / column l % 32 of every block for the
// term of its half-wave (A for BX rows, B for BY columns), so each generated
// value feeds BY (resp. BX) MFMAs.  A chunk's coefficients go through the
// wave's private 64-entry LDS slot (one vector load per lane, prefetched a
// chunk ahead); each chunk is summed into fresh FP32 blocks that are then
// folded into FP64 accumulators.  The four FP64 tiles are summed through LDS
// in a fixed order and wave 0 writes the slice's partial tile.
// Item (m, tile origin in 32-blocks x | y << 16, slice, variant 2..5 for
// (BX, BY) = (1,1), (2,1), (1,2), (2,2)); slices are whole 64-term chunks.
// With kGen (variant 6, maps of one 32x32 block, whose terms feed a single
// tile) each lane computes its term of the next chunk from the model's
// Gaussian table instead of loading it from the term table.
template <int BX, int BY, bool kGen>
__device__ __forceinline__ void num_tile_item(const Item it, const GeomDev *__restrict__ geoms,
                                              const ModelDev *__restrict__ models,
                                              const float4 *__restrict__ terms,
                                              const double *__restrict__ gauss,
                                              const int *__restrict__ st_ws,
                                              double *__restrict__ part,
                                              double *__restrict__ pix, float4 *cs, int wave,
                                              double *red) {
  const int lane = threadIdx.x & 63;
  const ModelDev md = models[it.m];
  const GeomDev g = geoms[md.geom];
  const int x0 = (it.a & 0xffff) * 32, y0 = (it.a >> 16) * 32;
  const int c32 = lane & 31, kh = lane >> 5;
  // Rows/columns outside the map get an exponent offset of -inf (and x^2 = 0),
  // so their operands are exactly 0 without a per-element select; inside the
  // map the offset is 0 and fma(c, x^2, 0) rounds exactly like c * x^2.
  float x2[BX], xoff[BX], y2[BY], yoff[BY];
#pragma unroll
  for (int bx = 0; bx < BX; ++bx) {
    const int xi = x0 + 32 * bx + c32;
    x2[bx] = 0.f;
    xoff[bx] = -__builtin_inff();
    if (xi < g.n_ux) { const double x = g.xs[xi]; x2[bx] = (float)(x * x); xoff[bx] = 0.f; }
  }
#pragma unroll
  for (int by = 0; by < BY; ++by) {
    const int yi = y0 + 32 * by + c32;
    y2[by] = 0.f;
    yoff[by] = -__builtin_inff();
    if (yi < g.n_uy) { const double y = g.ys[yi]; y2[by] = (float)(y * y); yoff[by] = 0.f; }
  }
  int ts, te;
  slice_range(g.T, md.n_slices, it.b, ts, te, KC2);
  // this wave's quarter of the slice, in whole chunks
  const int n_all = (st_ws[it.m] == 0) ? (te - ts + KC2 - 1) / KC2 : 0;
  const int qn = (n_all + 3) / 4;
  const int cb = min(n_all, wave * qn), ce = min(n_all, cb + qn);
  const int n_ch = ce - cb;
  const int t0 = ts + cb * KC2, t1 = min(te, ts + ce * KC2);
  const float4 *tb = terms + md.term_off;
  const double *gt = gauss + md.gauss_off;
  auto term = [&](int t) { return kGen ? term_of(g, gt, t) : tb[t]; };
  double acc[BX][BY][16];
#pragma unroll
  for (int bx = 0; bx < BX; ++bx)
#pragma unroll
    for (int by = 0; by < BY; ++by)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[bx][by][r] = 0.0;
  float4 cnext = make_float4(0.f, 0.f, 0.f, 0.f);
  if (n_ch > 0) cnext = term(min(t0 + lane, t1 - 1));
  const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int ch = 0; ch < n_ch; ++ch) {
    const int tc = t0 + ch * KC2;
    cs[lane] = cnext;
    __builtin_amdgcn_wave_barrier();
    if (ch + 1 < n_ch) cnext = term(min(tc + KC2 + lane, t1 - 1));
    v16f d[BX][BY];
#pragma unroll
    for (int bx = 0; bx < BX; ++bx)
#pragma unroll
      for (int by = 0; by < BY; ++by) d[bx][by] = zero;
    if (tc + KC2 <= t1) {          // whole chunk (wave-uniform), fully unrolled
#pragma unroll
      for (int s2 = 0; s2 < KC2 / 2; ++s2) {
        const float4 c = cs[2 * s2 + kh];
        float a[BX], b[BY];
#pragma unroll
        for (int bx = 0; bx < BX; ++bx)
          a[bx] = fast_exp2(fmaf(c.x, x2[bx], xoff[bx])) * fmaf(c.w, x2[bx], c.z);
#pragma unroll
        for (int by = 0; by < BY; ++by) b[by] = fast_exp2(fmaf(c.y, y2[by], yoff[by]));
#pragma unroll
        for (int bx = 0; bx < BX; ++bx)
#pragma unroll
          for (int by = 0; by < BY; ++by)
            d[bx][by] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[bx], b[by], d[bx][by], 0, 0, 0);
      }
    } else {                      // last, partial chunk of the slice
      for (int s2 = 0; s2 < KC2 / 2; ++s2) {
        const int k = 2 * s2 + kh;
        const float4 c = cs[k];
        const bool vt = tc + k < t1;
        float a[BX], b[BY];
#pragma unroll
        for (int bx = 0; bx < BX; ++bx) {
          const float v = fast_exp2(fmaf(c.x, x2[bx], xoff[bx])) * fmaf(c.w, x2[bx], c.z);
          a[bx] = vt ? v : 0.f;
        }
#pragma unroll
        for (int by = 0; by < BY; ++by) {
          const float v = fast_exp2(fmaf(c.y, y2[by], yoff[by]));
          b[by] = vt ? v : 0.f;
        }
#pragma unroll
        for (int bx = 0; bx < BX; ++bx)
#pragma unroll
          for (int by = 0; by < BY; ++by)
            d[bx][by] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[bx], b[by], d[bx][by], 0, 0, 0);
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int bx = 0; bx < BX; ++bx)
#pragma unroll
      for (int by = 0; by < BY; ++by)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[bx][by][r] += (double)d[bx][by][r];
  }
  // fixed-order sum of the four waves' tiles: wave 0 adds those of waves
  // 3, 2 and 1 in turn through one LDS tile
  for (int src = 3; src >= 1; --src) {
    __syncthreads();
    if (wave == src) {
#pragma unroll
      for (int bx = 0; bx < BX; ++bx)
#pragma unroll
        for (int by = 0; by < BY; ++by)
#pragma unroll
          for (int r = 0; r < 16; ++r) red[((bx * BY + by) * 16 + r) * 64 + lane] = acc[bx][by][r];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int bx = 0; bx < BX; ++bx)
#pragma unroll
        for (int by = 0; by < BY; ++by)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[bx][by][r] += red[((bx * BY + by) * 16 + r) * 64 + lane];
    }
  }
  if (wave != 0) return;
  if (md.n_slices == 1) {
    // the whole sum: straight into the N map (3476 models of 76 x 76 pixels: a
    // partial map and k_reduce took 412 us beside the 1130 us of this)
    double *o = pix + md.pix_off;
#pragma unroll
    for (int by = 0; by < BY; ++by) {
      const int y = y0 + 32 * by + c32;
#pragma unroll
      for (int bx = 0; bx < BX; ++bx)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int x = x0 + 32 * bx + 4 * kh + (r & 3) + 8 * (r >> 2);
          if (x < g.n_ux && y < g.n_uy) o[(int64_t)y * g.n_ux + x] = acc[bx][by][r];
        }
    }
    return;
  }
  // padded, transposed partial map: every row and column of the tile exists,
  // so the stores need no bounds checks; lanes store consecutive y
  const int ldh = 32 * md.n_yt;
  double *out = part + md.part_off + it.b * part_slice_size(md) +
                (int64_t)(x0 + 4 * kh) * ldh + y0 + c32;
#pragma unroll
  for (int bx = 0; bx < BX; ++bx)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      double *o = out + (int64_t)(32 * bx + (r & 3) + 8 * (r >> 2)) * ldh;
#pragma unroll
      for (int by = 0; by < BY; ++by) o[32 * by] = acc[bx][by][r];
    }
}

// Small maps (at most 4 TX x 4 TY unique pixels), terms computed in place:
// the map in 4 x 4 tiles by v_mfma_f32_4x4x1, whose sixteen blocks take
// sixteen terms, each block into its own sums.  Lane l generates the rows
// 4 i + l % 4 of A and the columns 4 j + l % 4 of B for term l / 4 of the
// sixteen, so no operand and few tiles are padding: a 19 x 19 map takes 25
// tiles of 4 x 4, where one 32 x 32 block is 2.8 times its pixels.  A block's
// FP32 sums run over kSmallFold chunks' share (64 terms) and are then added
// over the sixteen blocks in FP64, through LDS (16 registers at a time, rows
// of 68 floats so that the sixteen registers' reads fall on different banks).
// Waves, slices and the stored tile are those of num_tile_item.
// Matrix and vector issue bound it about equally (25 x 8 cycles, and ten
// exponentials and twenty multiply-adds per sixteen terms).  Measured, 4096
// models of 10 x 13 x 100 terms on 19 x 19 pixels: the 32 x 32 block 1509 us,
// this 930 us.
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kSmallFold = 16;   // chunks
constexpr int kSmallRed = 9 * 64;   // doubles of a wave's sums, and of its staging (16 x 68 floats)

template <int TX, int TY, bool kTab>
__device__ __forceinline__ void num_small_item(const Item it, const GeomDev *__restrict__ geoms,
                                               const ModelDev *__restrict__ models,
                                               const float4 *__restrict__ terms,
                                               const double *__restrict__ gauss,
                                               const int *__restrict__ st_ws,
                                               double *__restrict__ part,
                                               double *__restrict__ pix, float4 *cs, int wave,
                                               double *red) {
  constexpr int kTiles = TX * TY, NG = (4 * kTiles + 15) / 16, kRow = 68;
  static_assert(16 * kRow <= 2 * kSmallRed && NG * 64 <= kSmallRed,
                "the staging and the waves' sums fit red");
  const int lane = threadIdx.x & 63, r4 = lane & 3, blk = lane >> 2;
  const ModelDev md = models[it.m];
  const GeomDev &g = geoms[md.geom];
  const int x0 = kTab ? it.a & 0xffff : 0, y0 = kTab ? it.a >> 16 : 0;
  float x2[TX], y2[TY];
#pragma unroll
  for (int i = 0; i < TX; ++i) {
    const int xi = x0 + 4 * i + r4;
    const double x = xi < g.n_ux ? g.xs[xi] : 0.0;
    x2[i] = (float)(x * x);
  }
#pragma unroll
  for (int j = 0; j < TY; ++j) {
    const int yi = y0 + 4 * j + r4;
    const double y = yi < g.n_uy ? g.ys[yi] : 0.0;
    y2[j] = (float)(y * y);
  }
  int ts, te;
  slice_range(g.T, md.n_slices, it.b, ts, te, KC2);
  const int n_all = (st_ws[it.m] == 0) ? (te - ts + KC2 - 1) / KC2 : 0;
  const int qn = (n_all + 3) / 4;
  const int cb = min(n_all, wave * qn), ce = min(n_all, cb + qn);
  const int n_ch = ce - cb;
  const int t0 = ts + cb * KC2, t1 = min(te, ts + ce * KC2);
  const double *gt = gauss + md.gauss_off;
  __syncthreads();                 // the previous item's reads of red
  // the lane's next term, 64 on from the one before (stepped, not divided);
  // past the range a zero amplitude
  const int nu = g.n_u, J1 = g.J1;
  const float4 *tb = terms + md.term_off;
  int t = t0 + lane, n = t % nu, j = (t / nu) % J1, k = t / nu / J1;
  auto term = [&]() {
    if constexpr (kTab) {
      const float4 c = t < t1 ? tb[t] : make_float4(0.f, 0.f, 0.f, 0.f);
      t += KC2;
      return c;
    }
    const float4 c = t < t1 ? term_at(g, gt, k, j, n) : make_float4(0.f, 0.f, 0.f, 0.f);
    t += KC2;
    n += KC2;
    while (n >= nu) {
      n -= nu;
      if (++j == J1) {
        j = 0;
        ++k;
      }
    }
    return c;
  };
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f acc[TX][TY];
#pragma unroll
  for (int i = 0; i < TX; ++i)
#pragma unroll
    for (int j = 0; j < TY; ++j) acc[i][j] = zero;
  double tot[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) tot[q] = 0.0;
  float *st = reinterpret_cast<float *>(red) + wave * (16 * kRow);
  float4 cnext = make_float4(0.f, 0.f, 0.f, 0.f);
  if (n_ch > 0) cnext = term();
  for (int c0 = 0; c0 < n_ch; c0 += kSmallFold) {
    const int c1 = min(n_ch, c0 + kSmallFold);
    for (int ch = c0; ch < c1; ++ch) {
      cs[lane] = cnext;
      __builtin_amdgcn_wave_barrier();
      if (ch + 1 < n_ch) cnext = term();
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float4 c = cs[16 * s + blk];
        float a[TX], b[TY];
#pragma unroll
        for (int i = 0; i < TX; ++i) a[i] = fast_exp2(c.x * x2[i]) * fmaf(c.w, x2[i], c.z);
#pragma unroll
        for (int j = 0; j < TY; ++j) b[j] = fast_exp2(c.y * y2[j]);
#pragma unroll
        for (int i = 0; i < TX; ++i)
#pragma unroll
          for (int j = 0; j < TY; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();
    }
    // register 4 tile + r of lane 4 blk + c: pixel (4 i + r, 4 j + c) of block blk
#pragma unroll
    for (int q = 0; q < NG; ++q) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int tile = (16 * q + e) / 4;
        if (tile < kTiles) st[e * kRow + lane] = acc[tile / TY][tile % TY][e % 4];
      }
      __builtin_amdgcn_wave_barrier();
      double v = 0.0;
#pragma unroll
      for (int b = 0; b < 16; ++b) v += (double)st[blk * kRow + 4 * b + r4];
      tot[q] += v;
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int i = 0; i < TX; ++i)
#pragma unroll
      for (int j = 0; j < TY; ++j) acc[i][j] = zero;
  }
  // fixed-order sum of the four waves
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NG; ++q) red[(wave * NG + q) * 64 + lane] = tot[q];
  __syncthreads();
  const int ldh = 32 * md.n_yt;
  double *out = part + md.part_off + it.b * part_slice_size(md);
  for (int e = threadIdx.x; e < 16 * kTiles; e += 256) {
    // pixel (4 i + r, 4 j + c): tile 4 x 4 register r, column c
    const int tile = e / 16;
    const int x = x0 + 4 * (tile / TY) + (e / 4) % 4, y = y0 + 4 * (tile % TY) + e % 4;
    const double v = ((red[e] + red[NG * 64 + e]) + red[2 * NG * 64 + e]) + red[3 * NG * 64 + e];
    if (x >= g.n_ux || y >= g.n_uy) continue;
    if (md.n_slices > 1)
      out[(int64_t)x * ldh + y] = v;
    else                                     // the whole sum: straight into the N map
      pix[md.pix_off + (int64_t)y * g.n_ux + x] = v;
  }
}

// Numerator, per-pixel VALU form, over a work list of items (m, 256-pixel
// block, slice).  With a queue, every workgroup pulls the next item from a
// device counter (a persistent grid; items are ordered largest first);
// without one, workgroups stride over the list.
__global__ void __launch_bounds__(256) k_num_pix(const GeomDev *__restrict__ geoms,
                                                 const ModelDev *__restrict__ models,
                                                 const Item *__restrict__ items, int n_it,
                                                 const float4 *__restrict__ terms,
                                                 const int *__restrict__ st_ws,
                                                 double *__restrict__ part, int *queue) {
  __shared__ float4 stage[kPixStage];
  __shared__ int next;
  int i = blockIdx.x;
  for (;;) {
    if (queue) {
      if (threadIdx.x == 0) next = atomicAdd(queue, 1);
      __syncthreads();
      i = next;
      __syncthreads();
    }
    if (i >= n_it) break;
    num_pix_item(items[i], geoms, models, terms, st_ws, part, stage);
    if (!queue) i += gridDim.x;
  }
}

// Numerator, matrix-core form, over a work list of workgroup items.  With a
// queue, every workgroup pulls the next item (largest first) from a device
// counter (a persistent grid); without one, workgroups stride over the list.
// Variants of different tile shapes share one launch; the register budget is
// that of the 2x2 tile (two waves per SIMD, with the MFMA accumulators in
// ordinary VGPRs).
__global__ void __launch_bounds__(256, 2) k_num_mfma(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  const float4 *__restrict__ terms,
                                                  const double *__restrict__ gauss,
                                                  const int *__restrict__ st_ws,
                                                  double *__restrict__ part,
                                                  double *__restrict__ pix, int *queue) {
  __shared__ __attribute__((aligned(16))) float4 cs[4][KC2];
  __shared__ double red[4 * 16 * 64];
  __shared__ int next;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int i = blockIdx.x;
  for (;;) {
    if (queue) {
      if (threadIdx.x == 0) next = atomicAdd(queue, 1);
      __syncthreads();
      i = next;
      __syncthreads();
    }
    if (i >= n_it) break;
    const Item it = items[i];
    switch (it.c) {
      case 2: num_tile_item<1, 1, false>(it, geoms, models, terms, gauss, st_ws, part, pix, cs[wave], wave, red); break;
      case 3: num_tile_item<2, 1, false>(it, geoms, models, terms, gauss, st_ws, part, pix, cs[wave], wave, red); break;
      case 4: num_tile_item<1, 2, false>(it, geoms, models, terms, gauss, st_ws, part, pix, cs[wave], wave, red); break;
      case 6: num_tile_item<1, 1, true>(it, geoms, models, terms, gauss, st_ws, part, pix, cs[wave], wave, red); break;
      default: num_tile_item<2, 2, false>(it, geoms, models, terms, gauss, st_ws, part, pix, cs[wave], wave, red); break;
    }
    if (!queue) i += gridDim.x;
  }
}

// (A kernel per tiling: in one kernel with a switch the compiler spills.)
template <int TX, int TY, bool kTab>
__global__ void __launch_bounds__(256, 2) k_num_small(const GeomDev *__restrict__ geoms,
                                                   const ModelDev *__restrict__ models,
                                                   const Item *__restrict__ items, int n_it,
                                                   const float4 *__restrict__ terms,
                                                   const double *__restrict__ gauss,
                                                   const int *__restrict__ st_ws,
                                                   double *__restrict__ part,
                                                   double *__restrict__ pix) {
  __shared__ __attribute__((aligned(16))) float4 cs[4][KC2];
  __shared__ double red[4 * kSmallRed];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x)
    num_small_item<TX, TY, kTab>(items[i], geoms, models, terms, gauss, st_ws, part, pix, cs[wave], wave, red);
}

// Sum the split-term partials in a fixed order into the N map.  Item
// (m, block of 64 pixels in the partial maps' order, y fastest); the four
// waves take every fourth slice and their sums are combined in a fixed order.
__global__ void __launch_bounds__(256) k_reduce(const GeomDev *__restrict__ geoms,
                                                const ModelDev *__restrict__ models,
                                                const Item *__restrict__ items, int n_it,
                                                const double *__restrict__ part,
                                                double *__restrict__ pix) {
  __shared__ double red[3][64];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    // u walks the map with y fastest, as the partial maps are laid out
    const int u = it.a * 64 + lane;
    const int x = u / g.n_uy, y = u % g.n_uy;
    double acc = 0.0;
    if (u < g.n_pix) {
      const int64_t off = (int64_t)x * (32 * md.n_yt) + y;
      const int64_t stride = part_slice_size(md);
      // eight slices' loads in flight, added in slice order
      const double *pp = part + md.part_off + off;
      for (int s0 = wave; s0 < md.n_slices; s0 += 32) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int s = s0 + 4 * k;
          v[k] = s < md.n_slices ? pp[s * stride] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) acc += v[k];
      }
    }
    if (wave > 0) red[wave - 1][lane] = acc;
    __syncthreads();
    if (wave == 0 && u < g.n_pix)
      pix[md.pix_off + (int64_t)y * g.n_ux + x] = ((acc + red[0][lane]) + red[1][lane]) + red[2][lane];
    __syncthreads();
  }
}

// A thread's weighted sums of N and I over the entries e, e + stride, .. below
// e1: four accumulators, four gathers in flight, the remainder predicated: a
// loop over it waits for each of its up to three gathers in turn.  Measured:
// 4096 models x 20 bins 66 -> 53 us, one model of 60 bins of 6700 13.4 -> 10.9.
template <int kStride>
__device__ __forceinline__ void bin_sums(const GeomDev &g, const double *__restrict__ Nm,
                                         const double *__restrict__ Im, int e, int e1, bool want_n,
                                         double (&an)[4], double (&ai)[4]) {
  for (; e < e1; e += 4 * kStride) {
    double wv[4], nv[4], iv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int at = min(e + u * kStride, e1 - 1), q = g.bin_pix[at];
      wv[u] = g.bin_w[at];
      nv[u] = want_n ? Nm[q] : 0.0;
      iv[u] = Im[q];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool on = e + u * kStride < e1;
      an[u] = on ? fma(wv[u], nv[u], an[u]) : an[u];
      ai[u] = on ? fma(wv[u], iv[u], ai[u]) : ai[u];
    }
  }
}

// ---------------------------------------------------------------------------
// Bins: sums of the PSF-weighted maps per bin and their FP64 ratio.
// Item (m, bin, 0), launched with 1024 threads: the 16 waves of the block
// share one bin; item (m, first bin, 1), launched with 256 threads: each wave
// takes one of 4 consecutive bins (geometries whose bins all have few
// weights).  binws per model: [Nb | Ib], n_bins doubles each.
// ---------------------------------------------------------------------------
template <int BS>
__global__ void __launch_bounds__(BS) k_bins(const GeomDev *__restrict__ geoms,
                                              const ModelDev *__restrict__ models,
                                              const Item *__restrict__ items, int n_it,
                                              const double *__restrict__ pix,
                                              const int *__restrict__ st_ws,
                                              double *__restrict__ vrms2,
                                              double *__restrict__ binws) {
  __shared__ double sh[2 * (BS / 64)];
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    const double *Nm = pix + md.pix_off;
    const double *Im = Nm + g.n_pix;
    const bool want_n = vrms2 != nullptr;
    if (it.c == 1) {   // uniform per block: bins it.a + wave, one per wave
      const int lane = threadIdx.x & 63;
      const int b = it.a + (threadIdx.x >> 6);
      if (b >= g.n_bins) continue;   // uniform per wave; no barrier in this variant
      double an[4] = {0.0, 0.0, 0.0, 0.0}, ai[4] = {0.0, 0.0, 0.0, 0.0};
      bin_sums<64>(g, Nm, Im, g.bin_ptr[b] + lane, g.bin_ptr[b + 1], want_n, an, ai);
      double sn = wave_sum((an[0] + an[1]) + (an[2] + an[3]));
      const double si = wave_sum((ai[0] + ai[1]) + (ai[2] + ai[3]));
      if (!want_n) sn = 0.0;
      if (lane == 0) {
        const bool ok = st_ws[it.m] == 0;
        if (binws) {
          binws[md.bin_off + b] = sn;
          binws[md.bin_off + g.n_bins + b] = si;
        }
        if (want_n) vrms2[md.out_off + b] = ok ? sn / si : __builtin_nan("");
      }
      continue;
    }
    const int b = it.a;
    // four independent accumulators keep four gathers in flight per thread
    double an[4] = {0.0, 0.0, 0.0, 0.0}, ai[4] = {0.0, 0.0, 0.0, 0.0};
    bin_sums<BS>(g, Nm, Im, g.bin_ptr[b] + threadIdx.x, g.bin_ptr[b + 1], want_n, an, ai);
    // deterministic two-level sums: wave butterflies, then the wave partials
    // in a fixed order
    const double an_w = wave_sum((an[0] + an[1]) + (an[2] + an[3]));
    const double ai_w = wave_sum((ai[0] + ai[1]) + (ai[2] + ai[3]));
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
      sh[wv] = an_w;
      sh[BS / 64 + wv] = ai_w;
    }
    __syncthreads();
    double sn = 0.0, si = 0.0;
    if (threadIdx.x == 0)
      for (int w = 0; w < BS / 64; ++w) {
        sn += sh[w];
        si += sh[BS / 64 + w];
      }
    if (!want_n) sn = 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
      const bool ok = st_ws[it.m] == 0;
      if (binws) {
        binws[md.bin_off + b] = sn;
        binws[md.bin_off + g.n_bins + b] = si;
      }
      if (want_n) vrms2[md.out_off + b] = ok ? sn / si : __builtin_nan("");
    }
  }
}

// Expand the unique-pixel maps to the padded sub-pixel grid.  Item (m, row).
__global__ void __launch_bounds__(256) k_maps(const GeomDev *__restrict__ geoms,
                                              const ModelDev *__restrict__ models,
                                              const Item *__restrict__ items, int n_it,
                                              const double *__restrict__ pix,
                                              const int *__restrict__ st_ws,
                                              double *__restrict__ N_map,
                                              double *__restrict__ I_map) {
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    const int row = it.a;
    const int iy = g.uy[row];
    const bool ok = st_ws[it.m] == 0;
    for (int c = threadIdx.x; c < g.nxp; c += 256) {
      const int q = iy * g.n_ux + g.ux[c];
      const int64_t o = md.map_off + (int64_t)row * g.nxp + c;
      N_map[o] = ok ? pix[md.pix_off + q] : __builtin_nan("");
      I_map[o] = pix[md.pix_off + g.n_pix + q];
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint of the bin ratio and of the PSF/bin sums:
//   lambda_N[p] = sum_b W[b,p] cot_b / Ib_b,
//   lambda_I[p] = -sum_b W[b,p] cot_b V_b / Ib_b.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_bins_adjoint(const GeomDev *__restrict__ geoms,
                                                      const ModelDev *__restrict__ models,
                                                      const Item *__restrict__ items, int n_it,
                                                      const double *__restrict__ vrms2,
                                                      const double *__restrict__ cot,
                                                      const double *__restrict__ binws,
                                                      const int *__restrict__ st_ws,
                                                      double *__restrict__ pix) {
  // the bins' cot / I and V once per block (the first kAdjBins bins): per entry of
  // a pixel two gathers and a division, 27.3 us for 1024 small models, 19.3 here
  constexpr int kAdjBins = 256;
  __shared__ double cb[kAdjBins], vb[kAdjBins];
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    const int q = it.a * 256 + threadIdx.x;
    const double *Ib = binws + md.bin_off + g.n_bins;
    const bool good = st_ws[it.m] == 0;
    __syncthreads();                 // the previous item's reads
    for (int b = threadIdx.x; good && b < min(g.n_bins, kAdjBins); b += 256) {
      cb[b] = cot[md.out_off + b] / Ib[b];
      vb[b] = vrms2[md.out_off + b];
    }
    __syncthreads();
    if (q >= g.n_pix) continue;
    double ln = 0.0, li = 0.0;
    if (good) {
      const int e1 = g.pix_ptr[q + 1];
      for (int e = g.pix_ptr[q]; e < e1; ++e) {
        const int b = g.pix_bin[e];
        const double wv = g.pix_w[e];
        const double c = b < kAdjBins ? cb[b] : cot[md.out_off + b] / Ib[b];
        const double V = b < kAdjBins ? vb[b] : vrms2[md.out_off + b];
        ln += wv * c;
        li -= wv * c * V;
      }
    }
    pix[md.pix_off + 2 * (int64_t)g.n_pix + q] = ln;
    pix[md.pix_off + 3 * (int64_t)g.n_pix + q] = li;
  }
}

// ---------------------------------------------------------------------------
// Per-term adjoint sensitivities, per-pixel VALU form.  Lanes are terms; the
// unique pixels (x^2, y^2, lambda_N) are staged through LDS 256 at a time.
//   S0 = sum_p lambda E F,  S1 = sum_p lambda x^2 E F,
//   Sg = sum_p lambda y^2 E F (C0 + C1 x^2),
// with E F = exp(-c1 x^2 - gamma y^2).  Item (m, 256-term block).
// sens per model: [S0 | S1 | Sg], T doubles each.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void sens_pix_item(const Item it, const GeomDev *__restrict__ geoms,
    const ModelDev *__restrict__ models, const float4 *__restrict__ terms, const double *__restrict__ pix, const int *__restrict__ st_ws, double *__restrict__ sens, char *smem) {
  float *sx = reinterpret_cast<float *>(smem), *sy = sx + 256, *sl = sy + 256;

  const ModelDev md = models[it.m];
  const GeomDev g = geoms[md.geom];
  if (st_ws[it.m] != 0) return;   // uniform per block
  const int t = it.a * 256 + threadIdx.x;
  const bool valid = t < g.T;
  const float4 c = valid ? terms[md.term_off + t] : make_float4(0.f, 0.f, 0.f, 0.f);
  const double *lam = pix + md.pix_off + 2 * (int64_t)g.n_pix;
  double a0 = 0.0, a1 = 0.0, ag = 0.0;
  for (int base = 0; base < g.n_pix; base += 256) {
    const int q = base + threadIdx.x;
    __syncthreads();
    if (q < g.n_pix) {
      const double x = g.xs[q % g.n_ux], y = g.ys[q / g.n_ux];
      sx[threadIdx.x] = (float)(x * x);
      sy[threadIdx.x] = (float)(y * y);
      sl[threadIdx.x] = (float)lam[q];
    } else {
      sx[threadIdx.x] = 0.f;
      sy[threadIdx.x] = 0.f;
      sl[threadIdx.x] = 0.f;
    }
    __syncthreads();
    const int cnt = min(256, g.n_pix - base);
    float s0 = 0.f, s1 = 0.f, sg = 0.f;
    for (int e = 0; e < cnt; ++e) {
      const float x2 = sx[e], y2 = sy[e];
      const float le = sl[e] * fast_exp2(fmaf(c.x, x2, c.y * y2));
      s0 += le;
      s1 = fmaf(le, x2, s1);
      sg = fmaf(le * y2, fmaf(c.w, x2, c.z), sg);
    }
    a0 += s0;
    a1 += s1;
    ag += sg;
  }
  if (valid) {
    double *S = sens + md.sens_off;
    S[t] = a0;
    S[g.T + t] = a1;
    S[2 * (int64_t)g.T + t] = ag;
  }
}


// ---------------------------------------------------------------------------
// Per-term adjoint sensitivities, matrix-core form.  With E_t(x) = 2^(cx x^2)
// and F_t(y) = 2^(cy y^2) on the unique-pixel map,
//   G[x, t] = sum_y lambda[x, y] F_t(y),   H[x, t] = sum_y lambda[x, y] y^2 F_t(y)
// are two FP32 contractions over y sharing the lambda operand, and
//   S0_t = sum_x E G,  S1_t = sum_x x^2 E G,  Sg_t = sum_x E (C0 + C1 x^2) H.
// Item (m, 32-row x tile, tile of kSensTerms terms); wave w owns a quarter
// of the tile's terms and takes them as 32-term column blocks one after the
// other (lane l: term l % 32, y pair l / 32).  lambda is staged through LDS
// 256 rows of y at a time (once per item when the map has at most 256
// distinct |y|).  G and H are summed in FP32 over up to 128 y values; each
// such partial goes straight through the x epilogue (each lane's 16 rows in
// FP32) and the partial S0, S1, Sg are added in FP64, so no per-row FP64
// accumulators are live.  Output: per x tile, [S0 | S1 | Sg] (T doubles
// each).
// ---------------------------------------------------------------------------
constexpr int YC = 256;
constexpr int kSensWave = kSensTerms / 4;   // terms per wave of an item

__device__ __forceinline__ void sens_mfma_item(const Item it, const GeomDev *__restrict__ geoms,
                                               const ModelDev *__restrict__ models,
                                               const float4 *__restrict__ terms,
                                               const double *__restrict__ pix,
                                               const int *__restrict__ st_ws,
                                               double *__restrict__ sens, char *smem) {
  // lambda[x][y] staged x-major with the y values of each half-wave kh
  // (y = 2 s + kh) consecutive, so one 16-byte read gives a lane four steps'
  // operands; rows padded by 4 floats
  float (*lam)[YC + 4] = reinterpret_cast<float (*)[YC + 4]>(smem);
  float *ysq = reinterpret_cast<float *>(smem + 32 * (YC + 4) * sizeof(float));
  float *xsq = ysq + YC;                   // x^2 of the tile's rows (0 past the map)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c32 = lane & 31, kh = lane >> 5;
  const ModelDev md = models[it.m];
  const GeomDev g = geoms[md.geom];
  if (st_ws[it.m] != 0) return;   // uniform per block
  const int x0 = it.a * 32;
  const double *lamN = pix + md.pix_off + 2 * (int64_t)g.n_pix;
  const int n_yb = (g.n_uy + YC - 1) / YC;
  const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int h = 0; h < kSensWave / 32; ++h) {
    // this block's terms: it.b*kSensTerms + w*kSensWave + h*32 + (0..31)
    const int t = it.b * kSensTerms + wave * kSensWave + h * 32 + c32;
    const bool vt = t < g.T;
    const float4 c = vt ? terms[md.term_off + t] : make_float4(0.f, 0.f, 0.f, 0.f);
    double s0 = 0.0, s1 = 0.0, sg = 0.0;
    for (int ybi = 0; ybi < n_yb; ++ybi) {
      const int yb = ybi * YC;
      const int ny = min(YC, g.n_uy - yb);
      if (h == 0 || n_yb > 1) {         // uniform per block
        __syncthreads();
        // the rows the steps read: ny rounded up to whole blocks of 8 y
        const int rows = min(YC, (ny + 7) & ~7);
        for (int e = threadIdx.x; e < rows * 32; e += 256) {
          const int yy = e >> 5, xx = e & 31;
          float v = 0.f;
          if (yy < ny && x0 + xx < g.n_ux) v = (float)lamN[(int64_t)(yb + yy) * g.n_ux + x0 + xx];
          lam[xx][(yy & 1) * (YC / 2) + (yy >> 1)] = v;
        }
        for (int e = threadIdx.x; e < rows; e += 256) {
          float v = 0.f;
          if (e < ny) { const double y = g.ys[yb + e]; v = (float)(y * y); }
          ysq[(e & 1) * (YC / 2) + (e >> 1)] = v;
        }
        if (threadIdx.x < 32) {
          const int xr = x0 + threadIdx.x;
          float v = 0.f;
          if (xr < g.n_ux) { const double xv = g.xs[xr]; v = (float)(xv * xv); }
          xsq[threadIdx.x] = v;
        }
        __syncthreads();
      }
      for (int y0 = 0; y0 < ny; y0 += 128) {
        // operands lambda[x0 + c32][y0 + 2 s + kh] and y^2 for up to 128 y
        // values, four steps (8 y) per 16-byte read (rows past ny hold zero
        // lambda; y0 + 127 < YC)
        v16f dg = zero, dh = zero;
        const int nb = min(16, (ny - y0 + 7) / 8);   // uniform per block
        const float *lrow = &lam[c32][kh * (YC / 2) + y0 / 2];
        const float *yrow = ysq + kh * (YC / 2) + y0 / 2;
        // blocks alternate between two register buffers: the next block's
        // operands read and its exponentials taken behind the current MFMAs
        // (a read one block past the last stays inside the padded row and is
        // not used)
        float ra[2][4], ry[2][4], bb[2][4], by[2][4];
        auto load = [&](int u, int qb) {
          const float4 a4 = *reinterpret_cast<const float4 *>(lrow + 4 * qb);
          const float4 y4 = *reinterpret_cast<const float4 *>(yrow + 4 * qb);
          ra[u][0] = a4.x; ra[u][1] = a4.y; ra[u][2] = a4.z; ra[u][3] = a4.w;
          ry[u][0] = y4.x; ry[u][1] = y4.y; ry[u][2] = y4.z; ry[u][3] = y4.w;
        };
        auto expo = [&](int u) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            bb[u][j] = fast_exp2(c.y * ry[u][j]);
            by[u][j] = bb[u][j] * ry[u][j];
          }
        };
        auto mfma4 = [&](int u) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            dg = __builtin_amdgcn_mfma_f32_32x32x2f32(ra[u][j], bb[u][j], dg, 0, 0, 0);
            dh = __builtin_amdgcn_mfma_f32_32x32x2f32(ra[u][j], by[u][j], dh, 0, 0, 0);
          }
        };
        load(0, 0);
        expo(0);
        for (int qb = 0; qb < nb; qb += 2) {
          load(1, qb + 1);
          __builtin_amdgcn_sched_barrier(0);
          mfma4(0);
          expo(1);
          // taken here, not sunk into the branch below
          asm volatile("" ::"v"(bb[1][0]), "v"(bb[1][1]), "v"(bb[1][2]), "v"(bb[1][3]),
                       "v"(by[1][0]), "v"(by[1][1]), "v"(by[1][2]), "v"(by[1][3]));
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (qb + 1 < nb) {                 // uniform
            load(0, qb + 2);
            __builtin_amdgcn_sched_barrier(0);
            mfma4(1);
            expo(0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        // rows past the map have zero lambda, so zero sums; each lane's 16
        // rows in FP32, the y blocks and the lanes in FP64
        float f0 = 0.f, f1 = 0.f, fg = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float x2 = xsq[mfma_row(r, lane)];
          const float e = fast_exp2(c.x * x2);
          const float ed = e * dg[r];
          f0 += ed;
          f1 = fmaf(x2, ed, f1);
          fg = fmaf(e * fmaf(c.w, x2, c.z), dh[r], fg);
        }
        s0 += (double)f0;
        s1 += (double)f1;
        sg += (double)fg;
      }
    }
    s0 += __shfl_xor(s0, 32, 64);
    s1 += __shfl_xor(s1, 32, 64);
    sg += __shfl_xor(sg, 32, 64);
    if (kh == 0 && vt) {
      double *S = sens + md.sens_off + (int64_t)it.a * 3 * g.T;
      S[t] = s0;
      S[g.T + t] = s1;
      S[2 * (int64_t)g.T + t] = sg;
    }
  }
}

constexpr int kSensSmem = (32 * (YC + 4) + YC + 32) * (int)sizeof(float);
static_assert(kSensSmem >= 3 * 256 * (int)sizeof(float), "per-pixel sensitivity LDS");

// Adjoint sensitivities over a work list, variant in Item::c (0 per-pixel
// VALU, items (m, 256-term block); 1 MFMA, items (m, x tile, 256-term tile));
// queue-driven or strided as k_num.
__global__ void __launch_bounds__(256) k_sens(const GeomDev *__restrict__ geoms,
                                              const ModelDev *__restrict__ models,
                                              const Item *__restrict__ items, int n_it,
                                              const float4 *__restrict__ terms,
                                              const double *__restrict__ pix,
                                              const int *__restrict__ st_ws,
                                              double *__restrict__ sens, int *queue) {
  __shared__ __attribute__((aligned(16))) char smem[kSensSmem];
  __shared__ int next;
  int i = blockIdx.x;
  for (;;) {
    if (queue) {
      if (threadIdx.x == 0) next = atomicAdd(queue, 1);
      __syncthreads();
      i = next;
      __syncthreads();
    }
    if (i >= n_it) break;
    const Item it = items[i];
    if (it.c == 0)
      sens_pix_item(it, geoms, models, terms, pix, st_ws, sens, smem);
    else
      sens_mfma_item(it, geoms, models, terms, pix, st_ws, sens, smem);
    __syncthreads();
    if (!queue) i += gridDim.x;
  }
}

// ---------------------------------------------------------------------------
// Per-term adjoint sensitivities, wide matrix-core form: the contractions of
// sens_mfma_item for a part of XT <= 4 consecutive 32-row x tiles at once, so
// that each generated F_t(y) and y^2 F_t(y) feeds 2 XT MFMAs.  lambda_N of
// the part's rows is staged in LDS for up to 256 y at a time (once per item
// when the map has at most 256 distinct |y|) in the layout the MFMA steps
// read: row x holds, for each half kh of the wave, the values at y = 2s + kh
// for consecutive steps s, so one 16-byte read gives a lane four steps'
// operands (a quarter of the LDS instructions; rows are padded by 4 floats
// against bank conflicts).  Per term group the FP32 matrix-core sums run over
// all y (no FP64 fold: the 2 XT accumulator blocks take 128 registers at
// XT = 4), the next four steps' operands read and their exponentials taken
// behind the current MFMAs.  Item (m, part p | XT << 16 covering x tiles 4p ..
// 4p + XT - 1, first 32-term group, end group); eight waves, two per SIMD,
// so that one wave's LDS reads, waits and dependent epilogue pass behind the
// other's instructions (matrix and vector issue of a SIMD add up); wave w takes the item's groups w, w + 8, ...; output per part,
// [S0 | S1 | Sg] (T doubles each), as sens_mfma_item's per x tile.
// ---------------------------------------------------------------------------
constexpr int kWideTiles = 4;
constexpr int kWideLd = YC + 4;   // floats per staged x row: 2 halves x YC/2 steps + pad

struct SensWideLds {
  float lam[32 * kWideTiles][kWideLd];
  float ysq[YC];                   // [kh][s] = y^2 at y = 2s + kh
  float xsq[32 * kWideTiles];      // x^2 of the part's rows (0 past the map)
};

template <int XT>
__device__ __forceinline__ void sens_wide_item(const Item it, const ModelDev &md, const GeomDev &g,
                                               const float4 *__restrict__ terms,
                                               const double *__restrict__ pix,
                                               double *__restrict__ sens, SensWideLds &L,
                                               int wave) {
  const int lane = threadIdx.x & 63, c32 = lane & 31, kh = lane >> 5;
  const int part = it.a & 0xffff;
  const int x0 = 32 * kWideTiles * part;
  const double *lamN = pix + md.pix_off + 2 * (int64_t)g.n_pix;
  const int n_uy = __builtin_amdgcn_readfirstlane(g.n_uy);
  const int n_yb = (n_uy + YC - 1) / YC;
  const int g0 = it.b, g1 = it.c;
  const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bool staged = false;
  constexpr int NT = 64 * kWideWaves;
  if (threadIdx.x < 32 * XT) {
    const int xr = x0 + threadIdx.x;
    float v = 0.f;
    if (xr < g.n_ux) { const double xv = g.xs[xr]; v = (float)(xv * xv); }
    L.xsq[threadIdx.x] = v;          // read after the first staging barrier
  }
  // the group's term coefficients, loaded one group ahead
  auto coef = [&](int gr) {
    const int t = gr * 32 + c32;
    return (gr < g1 && t < g.T) ? terms[md.term_off + t] : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  float4 cnext = coef(g0 + wave);
  for (int gr = g0 + wave; gr - wave < g1; gr += kWideWaves) {   // same trip count in every wave
    const int t = gr * 32 + c32;
    const bool vt = gr < g1 && t < g.T;
    const float4 c = cnext;
    cnext = coef(gr + kWideWaves);
    v16f dg[XT], dh[XT];
#pragma unroll
    for (int bt = 0; bt < XT; ++bt) dg[bt] = dh[bt] = zero;
    for (int ybi = 0; ybi < n_yb; ++ybi) {
      const int yb = ybi * YC;
      const int ny = min(YC, n_uy - yb);
      if (!staged || n_yb > 1) {        // uniform per block
        __syncthreads();
        for (int e = threadIdx.x; e < YC * 32 * XT; e += NT) {
          const int yy = e / (32 * XT), xx = e % (32 * XT);
          float v = 0.f;
          if (yy < ny && x0 + xx < g.n_ux) v = (float)lamN[(int64_t)(yb + yy) * g.n_ux + x0 + xx];
          L.lam[xx][(yy & 1) * (YC / 2) + (yy >> 1)] = v;
        }
        for (int e = threadIdx.x; e < YC; e += NT) {
          float v = 0.f;
          if (e < ny) { const double y = g.ys[yb + e]; v = (float)(y * y); }
          L.ysq[(e & 1) * (YC / 2) + (e >> 1)] = v;
        }
        __syncthreads();
        staged = true;
      }
      // four y pairs per block of steps (rows past ny hold zero lambda);
      // blocks alternate between two operand buffers, the next block's
      // operands read and its exponentials taken behind the current MFMAs
      const int blocks = (((ny + 1) >> 1) + 3) >> 2;
      const float *yrow = L.ysq + kh * (YC / 2);
      float4 a4[2][XT], y4[2];
      float bx[2][4], bxy[2][4];
      auto load = [&](int buf, int q) {
        q = min(q, YC / 8 - 1);                  // past the last block: a harmless re-read
#pragma unroll
        for (int bt = 0; bt < XT; ++bt)
          a4[buf][bt] = *reinterpret_cast<const float4 *>(&L.lam[32 * bt + c32][kh * (YC / 2) + 4 * q]);
        y4[buf] = *reinterpret_cast<const float4 *>(yrow + 4 * q);
      };
      auto expo = [&](int buf) {
        const float ys[4] = {y4[buf].x, y4[buf].y, y4[buf].z, y4[buf].w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          bx[buf][u] = fast_exp2(c.y * ys[u]);
          bxy[buf][u] = bx[buf][u] * ys[u];
        }
      };
      auto mfma4 = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int bt = 0; bt < XT; ++bt) {
            const float4 &av4 = a4[buf][bt];
            const float av = u == 0 ? av4.x : (u == 1 ? av4.y : (u == 2 ? av4.z : av4.w));
            dg[bt] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bx[buf][u], dg[bt], 0, 0, 0);
            dh[bt] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, bxy[buf][u], dh[bt], 0, 0, 0);
          }
      };
      load(0, 0);
      expo(0);
      for (int q = 0; q < blocks; q += 2) {
        load(1, q + 1);
        __builtin_amdgcn_sched_barrier(0);
        mfma4(0);
        expo(1);
        // taken here, not sunk into the branch below
        asm volatile("" ::"v"(bx[1][0]), "v"(bx[1][1]), "v"(bx[1][2]), "v"(bx[1][3]),
                     "v"(bxy[1][0]), "v"(bxy[1][1]), "v"(bxy[1][2]), "v"(bxy[1][3]));
        // half the MFMAs go out before the exponentials wait for their reads
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * XT, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * XT, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (q + 1 < blocks) {                  // uniform
          load(0, q + 2);
          __builtin_amdgcn_sched_barrier(0);
          mfma4(1);
          expo(0);
          __builtin_amdgcn_sched_group_barrier(0x008, 4 * XT, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 4 * XT, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    // rows past the map have zero lambda, so zero g and h.  Each lane's 16
    // rows of a tile are summed in FP32 (beside the FP32 matrix-core sums over
    // y, a relative error of the same order), the tiles in FP64.
    double s0 = 0.0, s1 = 0.0, sg = 0.0;
#pragma unroll
    for (int bt = 0; bt < XT; ++bt) {
      float f0 = 0.f, f1 = 0.f, fg = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float x2 = L.xsq[32 * bt + mfma_row(r, lane)];
        const float e = fast_exp2(c.x * x2);
        const float ed = e * dg[bt][r];
        f0 += ed;
        f1 = fmaf(x2, ed, f1);
        fg = fmaf(e * fmaf(c.w, x2, c.z), dh[bt][r], fg);
      }
      s0 += (double)f0;
      s1 += (double)f1;
      sg += (double)fg;
    }
    s0 += __shfl_xor(s0, 32, 64);
    s1 += __shfl_xor(s1, 32, 64);
    sg += __shfl_xor(sg, 32, 64);
    if (kh == 0 && vt) {
      double *S = sens + md.sens_off + (int64_t)part * 3 * g.T;
      S[t] = s0;
      S[g.T + t] = s1;
      S[2 * (int64_t)g.T + t] = sg;
    }
  }
}

// Wide adjoint sensitivities over a work list (one workgroup of eight waves
// per CU: the staged lambda takes 135 KB of LDS); queue-driven or strided as
// k_sens.
__global__ void __launch_bounds__(64 * kWideWaves, 1) k_sens_wide(const GeomDev *__restrict__ geoms,
                                                      const ModelDev *__restrict__ models,
                                                      const Item *__restrict__ items, int n_it,
                                                      const float4 *__restrict__ terms,
                                                      const double *__restrict__ pix,
                                                      const int *__restrict__ st_ws,
                                                      double *__restrict__ sens, int *queue) {
  __shared__ __attribute__((aligned(16))) SensWideLds L;
  __shared__ int next;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int i = blockIdx.x;
  for (;;) {
    if (queue) {
      if (threadIdx.x == 0) next = atomicAdd(queue, 1);
      __syncthreads();
      i = next;
      __syncthreads();
    }
    if (i >= n_it) break;
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] == 0) {            // uniform per block
      switch (it.a >> 16) {
        case 1: sens_wide_item<1>(it, md, g, terms, pix, sens, L, wave); break;
        case 2: sens_wide_item<2>(it, md, g, terms, pix, sens, L, wave); break;
        case 3: sens_wide_item<3>(it, md, g, terms, pix, sens, L, wave); break;
        default: sens_wide_item<4>(it, md, g, terms, pix, sens, L, wave); break;
      }
    }
    __syncthreads();
    if (!queue) i += gridDim.x;
  }
}

// ---------------------------------------------------------------------------
// FP64 chain from per-term sensitivities to the parameters.  Forward-mode
// dual numbers carry d/d(inclination) through the deprojection and the term
// coefficients.  Items (m, k, jb): wave w of the workgroup takes mass
// Gaussian j = 4 jb + w (BH last) and its lanes the u-nodes.  Chain rows per
// model (doubles, after the sensitivity blocks): [K][J1][3] = (d/di, d/db_k,
// H_kj) for the terms of (k, j), with H_kj = sum_n (S0 c0 + S1 c1) the
// derivative with respect to the amplitude product I0_k M_j.  The
// surface-brightness path of I0_k is k_sb_adj's.
// ---------------------------------------------------------------------------
struct dual {
  double v, d;
};
__device__ inline dual operator+(dual a, dual b) { return {a.v + b.v, a.d + b.d}; }
__device__ inline dual operator-(dual a, dual b) { return {a.v - b.v, a.d - b.d}; }
__device__ inline dual operator*(dual a, dual b) { return {a.v * b.v, a.d * b.v + a.v * b.d}; }
__device__ inline dual operator/(dual a, dual b) {
  const double r = a.v / b.v;
  return {r, (a.d - r * b.d) / b.v};
}
__device__ inline dual operator*(double s, dual a) { return {s * a.v, s * a.d}; }
__device__ inline dual operator-(double s, dual a) { return {s - a.v, -a.d}; }
__device__ inline dual operator/(double s, dual a) {
  const double r = s / a.v;
  return {r, -r * a.d / a.v};
}
__device__ inline dual dsqrt(dual a) {
  const double r = sqrt(a.v);
  return {r, 0.5 * a.d / r};
}
__device__ inline dual dconst(double v) { return {v, 0.0}; }

__device__ inline double *chain_rows(double *sens, const ModelDev &md, const GeomDev &g) {
  return sens + md.sens_off + 3 * (int64_t)md.n_sens_parts * g.T;
}

__global__ void __launch_bounds__(256) k_chain(const GeomDev *__restrict__ geoms,
                                               const ModelDev *__restrict__ models,
                                               const Item *__restrict__ items, int n_it,
                                               ParamsDev p, double *__restrict__ sens,
                                               const int *__restrict__ st_ws) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;   // uniform per block; k_grads writes NaN
    const int k = it.a;
    const int J1 = g.J1, J = J1 - 1;
    double *rows = chain_rows(sens, md, g);
    const double qok = g.lum_q[k], sk = g.lum_sigma[k];
    const int j = it.b * 4 + wave;
    if (j >= J1) continue;            // uniform per wave; no block barrier follows
    const double inc = p.inc[it.m];
    const dual s = {sin(inc), cos(inc)};
    const dual c = {cos(inc), -sin(inc)};
    const dual si2 = s * s, ci2 = c * c;
    const double G = grav_const();
    const double sp = g.s_pc;
    const double I0 = p.lum_I0 ? p.lum_I0[md.lum_off + k] : g.lum_I0[k];
    const double b = 1.0 / (1.0 - p.beta[md.lum_off + k]);
    const dual qk = dsqrt(qok * qok - ci2) / s;
    const double alpha = 0.5 / (sk * sk);
    const dual alphaq = dconst(alpha) / (qk * qk);
    const dual nu1 = dconst(qok / (sqrt(2.0 * kPi) * sk)) / qk;   // nu0 / I0
    dual e2;
    double r, Kt, Mj;
    if (j < J) {
      const double qo = g.mass_q[j], sj = g.mass_sigma[j];
      const double S0 = p.mass_S0 ? p.mass_S0[md.mass_off + j] : g.mass_S0[j];
      const dual qj = dsqrt(qo * qo - ci2) / s;
      e2 = 1.0 - qj * qj;
      r = 0.5 / (sj * sj);
      Kt = sqrt(2.0 / kPi) * G / (sp * sj);
      Mj = p.mass_scale[it.m] * 2.0 * kPi * S0 * (sp * sj) * (sp * sj) * qo;
    } else {
      e2 = dconst(0.0);
      r = 0.5 / (g.bh_sigma * g.bh_sigma);
      Kt = sqrt(2.0 / kPi) * G / (sp * g.bh_sigma);
      Mj = p.m_bh[it.m];
    }
    const double amp = I0 * Mj;
    const double *S0a = sens + md.sens_off;
    const int np_ = md.n_sens_parts;
    double acc_i = 0.0, acc_b = 0.0, hj = 0.0;
    for (int n = lane; n < g.n_u; n += 64) {
      const int64_t t = ((int64_t)k * J1 + j) * g.n_u + n;
      // partial sensitivities of the x-row blocks, summed in block order;
      // eight blocks' loads are issued before their adds
      double S0 = 0.0, S1 = 0.0, Sg = 0.0;
      for (int q0 = 0; q0 < np_; q0 += 8) {
        double v0[8], v1[8], v2[8];
#pragma unroll
        for (int qq = 0; qq < 8; ++qq) {
          v0[qq] = v1[qq] = v2[qq] = 0.0;
          if (q0 + qq < np_) {
            const double *blk = S0a + (int64_t)(q0 + qq) * 3 * g.T;
            v0[qq] = blk[t];
            v1[qq] = blk[g.T + t];
            v2[qq] = blk[2 * (int64_t)g.T + t];
          }
        }
#pragma unroll
        for (int qq = 0; qq < 8; ++qq) {
          S0 += v0[qq];
          S1 += v1[qq];
          Sg += v2[qq];
        }
      }
      const double u = g.u[n], wq = g.w[n];
      const double u2 = u * u;
      const dual h = 1.0 - u2 * e2;
      const double c1 = alpha + r * u2;
      const dual A = alphaq + (r * u2) * (dconst(1.0) / h);
      const dual a = c1 * si2 + A * ci2;
      const dual gam = c1 * A / a;
      const dual sh_ = dsqrt(h);
      const dual base = (Kt * r * u2) * nu1;                    // per unit I0 M
      const dual gg = base / (A * h * sh_);
      const dual ww = 2.0 * base / sh_;
      const dual P = (ci2 + b * si2) * gg;
      const dual Q = si2 * (ww - (2.0 * c1 * b) * gg);
      const dual f = wq * dsqrt(kPi / a);
      const dual c0 = f * P, c1u = f * Q;                       // C = I0 M c
      acc_i += amp * (S0 * c0.d + S1 * c1u.d) - Sg * gam.d;
      // dC0/db = f si2 g, dC1/db = -2 f si2 c1 g
      acc_b += amp * f.v * si2.v * gg.v * (S0 - 2.0 * c1 * S1);
      hj += S0 * c0.v + S1 * c1u.v;
    }
    acc_i = wave_sum(acc_i);
    acc_b = wave_sum(acc_b);
    hj = wave_sum(hj);
    if (lane == 0) {
      double *o = rows + ((int64_t)k * J1 + j) * 3;
      o[0] = acc_i;
      o[1] = acc_b;
      o[2] = hj;
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint of a small-map model (its unique-pixel map fits one 32x32 block):
// the per-term sensitivities and the FP64 chain in one pass, lane = term.
// Each term's coefficients are computed in place as FP64 dual numbers
// carrying d/di (the set-up and term formulas of the forward), rounded to
// FP32 for the sums
//   S0 = sum_p lambda E F,  S1 = sum_p lambda x^2 E F,
//   Sg = sum_p lambda y^2 E F (C0 + C1 x^2),   E F = exp(-c1 x^2 - gamma y^2):
// F(y) and y^2 F(y) for every y in registers, then per x the FP32 sums
// g = sum_y lambda F and h = sum_y lambda y^2 F on the matrix cores and the
// x-sums in FP32, converted to FP64; the y loops are unrolled for the map's
// number of y quads.  Matrix and vector issue bound it.  Measured, 1024 models
// of 13000 terms on 19 x 19 pixels: lambda broadcast from LDS to every lane's
// own multiply-adds 637 us (the reads as long as the sums), this 478 us.
// The term's chain values (those of k_chain) go through LDS and every (k, j)
// row is summed over its u-nodes by one wave in a fixed order.  Item (m, k0 |
// k1 << 16, r0 | r1 << 16): of the tracers k0 <= k < k1 (at most
// kSmallAdjTracers) the (k, j) rows r0 .. r1 - 1; lambda_N, the squared coordinates, every mass
// Gaussian's and every tracer's set-up values are staged in LDS once per
// item, and the item's (k, j) rows, tracer-major, are taken in windows of
// whole rows with at most kAdjTerms terms, so that the passes of 256 terms
// run across tracers.  Writes the chain rows of k_chain (the model has no
// partial sensitivity blocks).
// ---------------------------------------------------------------------------
constexpr int kSmallMap = 32;
constexpr int kAdjTerms = kSmallAdjTerms;
constexpr int kSmallLam = kSmallMap + 4;   // the four rows of a read on different banks

// The three FP32 map sums of one term (lane) over NYQ quads of y (past the
// map y^2 = 0 and lambda = 0, so the padding adds nothing) and nxq quads of x:
// F(y) and y^2 F(y) in registers; per quad of x the sums g and h over y by
// v_mfma_f32_4x4x1 with lambda(4 i + l % 4, y) as A in lane l and F as B: block
// l / 4, column l % 4 is lane l's own term and register r its sum at x = 4 i +
// r, so nothing moves between lanes.  lambda is read four y at a time.
template <int NYQ>
__device__ __forceinline__ void small_sums(float cx, float cy, float C0, float C1,
                                           const float (*lam)[kSmallLam], const float *xsq,
                                           const float *ysq, int nxq, float &s0, float &s1,
                                           float &sg) {
  float F[4 * NYQ], Fy[4 * NYQ];
#pragma unroll
  for (int yy = 0; yy < 4 * NYQ; ++yy) {
    const float y2 = ysq[yy];
    F[yy] = fast_exp2(cy * y2);
    Fy[yy] = F[yy] * y2;
  }
  // an offset the compiler cannot prove loop-invariant, so that the lambda
  // reads are not hoisted out of the caller's term loop into registers
  int zoff;
  asm volatile("s_mov_b32 %0, 0" : "=s"(zoff));
  const int r4 = threadIdx.x & 3;
  s0 = 0.f;
  s1 = 0.f;
  sg = 0.f;
  // NX quads at a time: with two, four independent sums cover the matrix
  // instructions' latency
  auto quads = [&](int xq, auto nxt) {
    constexpr int NX = decltype(nxt)::value;
    v4f gs[NX], hs[NX];
#pragma unroll
    for (int q = 0; q < NX; ++q) gs[q] = hs[q] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int yq = 0; yq < NYQ; ++yq) {
      float4 l[NX];
#pragma unroll
      for (int q = 0; q < NX; ++q)
        l[q] = (reinterpret_cast<const float4 *>(lam[4 * (xq + q) + r4]) + zoff)[yq];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < NX; ++q) {
          const float a = c == 0 ? l[q].x : (c == 1 ? l[q].y : (c == 2 ? l[q].z : l[q].w));
          gs[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, F[4 * yq + c], gs[q], 0, 0, 0);
          hs[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(a, Fy[4 * yq + c], hs[q], 0, 0, 0);
        }
    }
#pragma unroll
    for (int q = 0; q < NX; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float x2 = xsq[4 * (xq + q) + r];
        const float E = fast_exp2(cx * x2);
        const float Eg = E * gs[q][r];
        s0 += Eg;
        s1 = fmaf(Eg, x2, s1);
        sg = fmaf(E * hs[q][r], fmaf(C1, x2, C0), sg);
      }
  };
  int xq = 0;
  for (; xq + 1 < nxq; xq += 2) quads(xq, std::integral_constant<int, 2>());
  if (xq < nxq) quads(xq, std::integral_constant<int, 1>());
}

// (A kernel per number of y quads: in one kernel all take the largest one's
// registers.)
template <int NYQ>
__global__ void __launch_bounds__(256, NYQ <= 5 ? 3 : 2) k_adj_small(const GeomDev *__restrict__ geoms,
                                                   const ModelDev *__restrict__ models,
                                                   const Item *__restrict__ items, int n_it,
                                                   ParamsDev p, const double *__restrict__ pix,
                                                   const int *__restrict__ st_ws,
                                                   double *__restrict__ sens) {
  __shared__ __attribute__((aligned(16))) float lam[kSmallMap][kSmallLam];   // [x][y]
  __shared__ float xsq[kSmallMap], ysq[kSmallMap];
  // per mass Gaussian: e2, de2/di, r, K_j / M_j, M_j
  __shared__ double jv[kSmallAdjMass][5];
  // per tracer: alpha, alphaq and d/di, nu0 / I0 and d/di, cos^2 i + b sin^2 i
  // and d/di, b, I0
  __shared__ double tv[kSmallAdjTracers][9];
  __shared__ double vals[kAdjTerms][3];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;   // uniform per block; k_grads writes NaN
    // block-uniform bounds in scalar registers, so the unrolled loops'
    // guards are scalar branches
    const int k0 = __builtin_amdgcn_readfirstlane(it.a & 0xffff);
    const int k1 = __builtin_amdgcn_readfirstlane(it.a >> 16);
    const int nx = __builtin_amdgcn_readfirstlane(g.n_ux);
    const int ny = __builtin_amdgcn_readfirstlane(g.n_uy);
    const int nu = __builtin_amdgcn_readfirstlane(g.n_u);
    const int J1 = __builtin_amdgcn_readfirstlane(g.J1), J = J1 - 1;
    __syncthreads();                  // the previous item's LDS reads are done
    const double *lamN = pix + md.pix_off + 2 * (int64_t)g.n_pix;
    for (int e = threadIdx.x; e < kSmallMap * kSmallMap; e += 256) {
      const int xx = e / kSmallMap, yy = e % kSmallMap;
      lam[xx][yy] = (yy < ny && xx < nx) ? (float)lamN[yy * nx + xx] : 0.f;
    }
    if (threadIdx.x < kSmallMap) {
      const int q = threadIdx.x;
      xsq[q] = q < nx ? (float)(g.xs[q] * g.xs[q]) : 0.f;
      ysq[q] = q < ny ? (float)(g.ys[q] * g.ys[q]) : 0.f;
    }
    const double inc = p.inc[it.m];
    const dual sn = {sin(inc), cos(inc)};
    const dual cs = {cos(inc), -sin(inc)};
    const dual si2 = sn * sn, ci2 = cs * cs;
    const double G = grav_const(), sp = g.s_pc;
    for (int j = threadIdx.x; j < J1; j += 256) {
      double *v = jv[j];
      if (j < J) {
        const double qo = g.mass_q[j], sj = g.mass_sigma[j];
        const double S0 = p.mass_S0 ? p.mass_S0[md.mass_off + j] : g.mass_S0[j];
        const dual qj = dsqrt(qo * qo - ci2) / sn;
        const dual e2 = 1.0 - qj * qj;
        v[0] = e2.v;
        v[1] = e2.d;
        v[2] = 0.5 / (sj * sj);
        v[3] = sqrt(2.0 / kPi) * G / (sp * sj);
        v[4] = p.mass_scale[it.m] * 2.0 * kPi * S0 * (sp * sj) * (sp * sj) * qo;
      } else {
        v[0] = 0.0;
        v[1] = 0.0;
        v[2] = 0.5 / (g.bh_sigma * g.bh_sigma);
        v[3] = sqrt(2.0 / kPi) * G / (sp * g.bh_sigma);
        v[4] = p.m_bh[it.m];
      }
    }
    if (threadIdx.x < k1 - k0) {
      // tracer k: deprojection (App. A) with its inclination derivative
      const int k = k0 + threadIdx.x;
      const double qok = g.lum_q[k], sk = g.lum_sigma[k];
      const double b = 1.0 / (1.0 - p.beta[md.lum_off + k]);
      const dual qk = dsqrt(qok * qok - ci2) / sn;
      const double alpha = 0.5 / (sk * sk);
      const dual alphaq = dconst(alpha) / (qk * qk);
      const dual nu1 = dconst(qok / (sqrt(2.0 * kPi) * sk)) / qk;   // nu0 / I0
      const dual pf = ci2 + b * si2;
      double *v = tv[threadIdx.x];
      v[0] = alpha;
      v[1] = alphaq.v;
      v[2] = alphaq.d;
      v[3] = nu1.v;
      v[4] = nu1.d;
      v[5] = pf.v;
      v[6] = pf.d;
      v[7] = b;
      v[8] = p.lum_I0 ? p.lum_I0[md.lum_off + k] : g.lum_I0[k];
    }
    double *rows = chain_rows(sens, md, g);
    const int row0 = __builtin_amdgcn_readfirstlane(it.b & 0xffff);
    const int row1 = __builtin_amdgcn_readfirstlane(it.b >> 16);
    const int per_win = max(1, kAdjTerms / nu);   // whole rows per window
    const float rnu = 1.f / nu, rJ1 = 1.f / J1;
    for (int r0 = row0; r0 < row1; r0 += per_win) {
      const int nr = min(per_win, row1 - r0);
      const int n_terms = nr * nu;
      __syncthreads();                // staging done; earlier readers of vals done
      for (int base = 0; base < n_terms; base += 256) {
        // lanes past the window repeat its last term: the matrix instructions
        // take the whole wave
        const int tq = base + threadIdx.x, tl = min(tq, n_terms - 1);
        // (exact: at most 2^14 rows, FP32 quotients of half-integers)
        const int rr = (int)((tl + 0.5f) * rnu), n = tl - rr * nu;
        const int row = r0 + rr, kk = (int)((row + 0.5f) * rJ1), jj = row - kk * J1;
        const double *tk = tv[kk];
        const double *v = jv[jj];
        const double alpha = tk[0], b = tk[7];
        const dual alphaq = {tk[1], tk[2]}, nu1 = {tk[3], tk[4]}, pf = {tk[5], tk[6]};
        const double r = v[2], Mj = v[4];
        const double u = load_global(g.u + n), wq = load_global(g.w + n), u2 = u * u;
        const dual h = {fma(-v[0], u2, 1.0), -u2 * v[1]};
        const double c1 = alpha + r * u2;
        const double rshv = rsq64(h.v), rhv = rshv * rshv;
        const dual rh = {rhv, -rhv * rhv * h.d};
        const dual A = alphaq + (r * u2) * rh;
        const dual a = c1 * si2 + A * ci2;
        const double rsav = rsq64(a.v), rav = rsav * rsav;
        const dual gam = c1 * A * dual{rav, -rav * rav * a.d};
        const dual rsh = {rshv, -0.5 * rshv * rhv * h.d};
        const dual bse = (v[3] * r * u2) * nu1;               // per unit I0 M
        const double rAv = rcp64(A.v);
        const dual gg = bse * dual{rAv, -rAv * rAv * A.d} * rh * rsh;
        const dual ww = 2.0 * bse * rsh;
        const dual P = pf * gg;
        const dual Q = si2 * (ww - (2.0 * c1 * b) * gg);
        const double fv = wq * kSqrtPi * rsav;
        const dual f = {fv, -0.5 * fv * rav * a.d};
        const dual c0 = f * P, c1u = f * Q;                   // C = I0 M c
        const double amp = tk[8] * Mj;
        const float cx = (float)(-c1 * kLog2e), cy = (float)(-gam.v * kLog2e);
        const float C0 = (float)(amp * c0.v), C1 = (float)(amp * c1u.v);
        float s0, s1, sg;
        const int nxq = (nx + 3) >> 2;
        small_sums<NYQ>(cx, cy, C0, C1, lam, xsq, ysq, nxq, s0, s1, sg);
        const double S0 = s0, S1 = s1, Sg = sg;
        if (tq < n_terms) {
          vals[tl][0] = amp * (S0 * c0.d + S1 * c1u.d) - Sg * gam.d;
          // dC0/db = f si2 g, dC1/db = -2 f si2 c1 g
          vals[tl][1] = amp * f.v * si2.v * gg.v * (S0 - 2.0 * c1 * S1);
          vals[tl][2] = S0 * c0.v + S1 * c1u.v;
        }
      }
      __syncthreads();
      // (k, j) rows: one wave per row, lanes over the u-nodes in order, then
      // a butterfly
      for (int rr = wave; rr < nr; rr += 4) {
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        for (int n = lane; n < nu; n += 64) {
          const double *v = vals[rr * nu + n];
          a0 += v[0];
          a1 += v[1];
          a2 += v[2];
        }
        a0 = wave_sum(a0);
        a1 = wave_sum(a1);
        a2 = wave_sum(a2);
        if (lane == 0) {
          double *o = rows + ((int64_t)k0 * J1 + r0 + rr) * 3;
          o[0] = a0;
          o[1] = a1;
          o[2] = a2;
        }
      }
    }
  }
}

// Final per-model gradients from the chain rows.  One block of kW waves per
// model: each wave reduces one luminous Gaussian's row at a time over the
// mass Gaussians (lanes), then the waves reduce the mass derivatives over
// the luminous Gaussians; partial sums are combined in a fixed order.
template <int kW>
__global__ void __launch_bounds__(64 * kW) k_grads(const GeomDev *__restrict__ geoms,
                                               const ModelDev *__restrict__ models, int n,
                                               ParamsDev p, double *__restrict__ sens,
                                               const double *__restrict__ sbp,
                                               const int *__restrict__ st_ws, GradsDev out) {
  __shared__ double part[kW];
  __shared__ double mpart[kW][64];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  for (int m = blockIdx.x; m < n; m += gridDim.x) {
    const ModelDev md = models[m];
    const GeomDev g = geoms[md.geom];
    const int K = g.K, J1 = g.J1, J = J1 - 1;
    const double *rows = chain_rows(sens, md, g);
    const bool ok = st_ws[m] == 0;
    const double nan = __builtin_nan("");
    const double sp = g.s_pc;
    const double ml = p.mass_scale[m];
    auto mass = [&](int j) {
      if (j == J) return p.m_bh[m];
      const double S0 = p.mass_S0 ? p.mass_S0[md.mass_off + j] : g.mass_S0[j];
      return ml * 2.0 * kPi * S0 * (sp * g.mass_sigma[j]) * (sp * g.mass_sigma[j]) * g.mass_q[j];
    };
    // d/di, d/dbeta_k, d/dI0_k
    double di = 0.0;
    for (int k = wave; k < K; k += kW) {
      double a = 0.0, db = 0.0, dI = 0.0;
      for (int j = lane; j < J1; j += 64) {
        const double *o = rows + ((int64_t)k * J1 + j) * 3;
        a += o[0];
        db += o[1];
        dI += mass(j) * o[2];
      }
      // surface-brightness path of I0_k: the tile partials, in tile order
      double sb = 0.0;
      const int n_tiles = sb_tiles(g.n_ux, g.n_uy);
      if (ok)
        for (int tl = lane; tl < n_tiles; tl += 64) sb += sbp[md.sbp_off + (int64_t)k * n_tiles + tl];
      a = wave_sum(a);
      db = wave_sum(db);
      dI = wave_sum(dI);
      sb = wave_sum(sb);
      di += a;
      if (lane == 0) {
        const double b = 1.0 / (1.0 - p.beta[md.lum_off + k]);
        if (out.beta) out.beta[md.lum_off + k] = ok ? db * b * b : nan;   // db/dbeta = b^2
        if (out.lum_I0) out.lum_I0[md.lum_off + k] = ok ? dI + sb : nan;
      }
    }
    // d/dM_j = sum_k I0_k H_kj; then the mass scale, Sigma0_j and the BH
    double dml = 0.0;
    for (int j0 = 0; j0 < J1; j0 += 64) {
      const int j = j0 + lane;
      double dM = 0.0;
      if (j < J1) {
        // loads of eight tracers are issued before their (ordered) adds
        for (int k0 = wave; k0 < K; k0 += 8 * kW) {
          double iv[8], hv[8];
#pragma unroll
          for (int kk = 0; kk < 8; ++kk) {
            const int k = k0 + kW * kk;
            iv[kk] = 0.0;
            hv[kk] = 0.0;
            if (k < K) {
              iv[kk] = p.lum_I0 ? p.lum_I0[md.lum_off + k] : g.lum_I0[k];
              hv[kk] = rows[((int64_t)k * J1 + j) * 3 + 2];
            }
          }
#pragma unroll
          for (int kk = 0; kk < 8; ++kk) dM += iv[kk] * hv[kk];
        }
      }
      __syncthreads();
      mpart[wave][lane] = dM;
      __syncthreads();
      if (wave == 0 && j < J1) {
        dM = 0.0;
        for (int w = 0; w < kW; ++w) dM += mpart[w][lane];
        if (j < J) {
          const double qo = g.mass_q[j], sj = g.mass_sigma[j];
          const double S0 = p.mass_S0 ? p.mass_S0[md.mass_off + j] : g.mass_S0[j];
          const double unit = 2.0 * kPi * (sp * sj) * (sp * sj) * qo;   // dM/d(ml S0)
          if (out.mass_S0) out.mass_S0[md.mass_off + j] = ok ? dM * ml * unit : nan;
          dml += dM * S0 * unit;
        } else {
          if (out.m_bh) out.m_bh[m] = ok ? dM : nan;
        }
      }
    }
    if (wave == 0) dml = wave_sum(dml);
    if (lane == 0) part[wave] = di;
    __syncthreads();
    if (threadIdx.x == 0) {
      double dsum = 0.0;
      for (int w = 0; w < kW; ++w) dsum += part[w];
      if (out.inc) out.inc[m] = ok ? dsum : nan;
      if (out.mass_scale) out.mass_scale[m] = ok ? dml : nan;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Goodness of fit, eq. (chi2_dyn): chi^2 = r^T P r with r_b = v_obs,b -
// sqrt(V_b) (eq. (Vrms)) and P the inverse covariance of the measured v_rms.
// One workgroup per model: r in LDS; s = P r by rows, one row per wave at a
// time with the lanes along the row and a fixed-order wave sum; chi^2 = r.s
// summed in a fixed order.  dV (optional) receives cot_m * d chi^2 / dV_b =
// -cot_m s_b / sqrt(V_b).  All FP64; NaN for a model whose status is not OK
// or with any V_b <= 0 (v_rms undefined).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_chi2(const GeomDev *__restrict__ geoms,
                                              const ModelDev *__restrict__ models, int n,
                                              const KinDev *__restrict__ kin,
                                              const double *__restrict__ V,
                                              const int *__restrict__ st_ws,
                                              double *__restrict__ chi2,
                                              const double *__restrict__ cot,
                                              double *__restrict__ dV) {
  __shared__ double r[kChi2MaxBins];
  __shared__ double part[4];
  __shared__ int bad;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double nan = __builtin_nan("");
  for (int m = blockIdx.x; m < n; m += gridDim.x) {
    const ModelDev md = models[m];
    const int nb = geoms[md.geom].n_bins;
    const KinDev kd = kin[md.geom];
    const double *Vm = V + md.out_off;
    if (tid == 0) bad = (st_ws && st_ws[m] != 0) ? 1 : 0;
    __syncthreads();
    for (int b = tid; b < nb; b += 256) {
      const double v = Vm[b];
      if (!(v > 0.0)) bad = 1;       // every writer stores the same value
      r[b] = kd.vobs[b] - sqrt(v);
    }
    __syncthreads();
    const bool ok = bad == 0;
    const double scale = cot ? cot[m] : 1.0;
    double acc = 0.0;
    for (int b = wave; b < nb; b += 4) {
      const double *row = kd.prec + (int64_t)b * nb;
      double sb = 0.0;
      for (int c = lane; c < nb; c += 64) sb = fma(row[c], r[c], sb);
      sb = wave_sum(sb);
      acc = fma(r[b], sb, acc);
      if (dV && lane == 0) dV[md.out_off + b] = ok ? -scale * sb / sqrt(Vm[b]) : nan;
    }
    if (lane == 0) part[wave] = acc;
    __syncthreads();
    if (tid == 0 && chi2) chi2[m] = ok ? ((part[0] + part[1]) + part[2]) + part[3] : nan;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// One-dimensional MGE of radial profiles (Sect. 3.2, eq. integral_transfer
// and the Euler approximation after it).  A profile F(R) = sum_c a_c
// (R^2 + c_c^2)^(-p_c) is expanded as F(R) ~ sum_n A_n exp(-R^2/(2 sigma_n^2))
// with A_n = scale_n sum_k eta_k Re F(sigma_n chi_k), chi_k^2 = 2 beta_k, so
// F is needed at R^2 = 2 sigma_n^2 beta_k, where Re(R^2) > 0 and the
// principal logarithm of R^2 + c^2 is analytic.  FP64 throughout.
// ---------------------------------------------------------------------------
struct cplx {
  double re, im;
};
__device__ inline cplx c_log(cplx z) { return {log(hypot(z.re, z.im)), atan2(z.im, z.re)}; }
__device__ inline cplx c_exp(cplx z) {
  double sn, cs;
  sincos(z.im, &sn, &cs);
  const double e = exp(z.re);
  return {e * cs, e * sn};
}
__device__ inline cplx c_mul(cplx a, cplx b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ inline cplx c_div(cplx a, cplx b) {
  const double d = b.re * b.re + b.im * b.im;
  return {(a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d};
}

// Nodes R^2 = 2 sigma_n^2 beta_k and weights, staged in LDS.
struct MgeTables {
  double s2[kMgeMaxSigma], scale[kMgeMaxSigma], eta[kMgeMaxTerms], bim[kMgeMaxTerms];
};
__device__ inline void mge_stage(const MgeConst &kc, MgeTables &t) {
  const int e = threadIdx.x;
  if (e < kc.n_sigma) {
    t.s2[e] = 2.0 * kc.sigma2[e];
    t.scale[e] = kc.scale[e];
  }
  if (e < kc.n_terms) {
    t.eta[e] = kc.eta[e];
    t.bim[e] = kc.beta_im[e];
  }
  __syncthreads();
}
constexpr int kMgeBlocks = 1 << 16;

// 32 lanes per (profile, Gaussian n), the terms k over the lanes, added in a
// fixed order.  The complex logarithms and exponentials (some 400 FP64
// operations each) bound both kernels; with a thread per output 512 profiles
// kept 168 waves busy here and 16 below: 34 and 301 us, now 13 and 11.
__global__ void __launch_bounds__(256) k_mge1d(int n_prof, int n_comp,
                                               const double *__restrict__ comp, MgeConst kc,
                                               double *__restrict__ amp) {
  __shared__ MgeTables t;
  mge_stage(kc, t);
  const int lane = threadIdx.x & 31;
  for (int64_t id = (int64_t)blockIdx.x * (blockDim.x / 32) + threadIdx.x / 32;
       id < (int64_t)n_prof * kc.n_sigma; id += (int64_t)gridDim.x * (blockDim.x / 32)) {
    const int prof = (int)(id / kc.n_sigma), n = (int)(id % kc.n_sigma);
    const double *cp = comp + (int64_t)prof * n_comp * 3;
    double f = 0.0;
    for (int k = lane; k < kc.n_terms; k += 32) {
      const cplx r2 = {t.s2[n] * kc.beta_re, t.s2[n] * t.bim[k]};
      double fr = 0.0;   // Re F(R)
      for (int c = 0; c < n_comp; ++c) {
        const double a = cp[3 * c], cc = cp[3 * c + 1], p = cp[3 * c + 2];
        const cplx L = c_log({r2.re + cc * cc, r2.im});
        fr += a * c_exp({-p * L.re, -p * L.im}).re;
      }
      f += t.eta[k] * fr;
    }
    for (int o = 16; o > 0; o >>= 1) f += __shfl_xor(f, o, 32);
    if (lane == 0) amp[id] = t.scale[n] * f;
  }
}

// A wave per (profile, component): its three derivatives summed over the
// Gaussians n (weighted by the cotangent) and the terms k, (n, k) pairs over
// the lanes, in a fixed order.
__global__ void __launch_bounds__(256) k_mge1d_vjp(int n_prof, int n_comp,
                                                   const double *__restrict__ comp, MgeConst kc,
                                                   const double *__restrict__ cot,
                                                   double *__restrict__ grad) {
  __shared__ MgeTables t;
  mge_stage(kc, t);
  const int lane = threadIdx.x & 63;
  for (int64_t id = (int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
       id < (int64_t)n_prof * n_comp; id += (int64_t)gridDim.x * (blockDim.x / 64)) {
    const int prof = (int)(id / n_comp);
    const double *cp = comp + id * 3;
    const double a = cp[0], cc = cp[1], p = cp[2];
    double ga = 0.0, gc = 0.0, gp = 0.0;
    for (int e = lane; e < kc.n_sigma * kc.n_terms; e += 64) {
      const int n = e / kc.n_terms, k = e % kc.n_terms;
      const cplx w = {t.s2[n] * kc.beta_re + cc * cc, t.s2[n] * t.bim[k]};
      const cplx L = c_log(w);
      const cplx E = c_exp({-p * L.re, -p * L.im});          // w^-p
      const cplx Ew = c_div(E, w);                            // w^-(p+1)
      const double s = t.scale[n] * cot[(int64_t)prof * kc.n_sigma + n] * t.eta[k];
      ga += s * E.re;
      gc += s * (-2.0 * p * cc * a) * Ew.re;
      gp += s * (-a) * c_mul(L, E).re;
    }
    ga = wave_sum(ga);
    gc = wave_sum(gc);
    gp = wave_sum(gp);
    if (lane == 0) {
      grad[id * 3] = ga;
      grad[id * 3 + 1] = gc;
      grad[id * 3 + 2] = gp;
    }
  }
}

// ---------------------------------------------------------------------------
// Spherically aligned model (eqs. J1, J2).  For tracer Gaussian k with
// constant beta the Jeans equations integrate along the characteristics
// r^(1-beta) sin(theta) = const:
//   P_k = nu v_r^2 = r^(-2 beta) int_r^inf r'^(2 beta) nu (d_z Phi) / cos(theta') dr',
//   d_theta P_k = r^(1 - 3 beta) cos(theta) I_D,
//   I_D = int_r^inf r'^(3 beta + 1) R' nu [G_theta + G (1/q^2 - 1) / sigma^2] dr',
//   nu v_phi^2 = (1 - beta) P + (1 - beta) sin(theta) r^(1 - 3 beta) I_D - nu R^2 G_phi,
// with G = (d_z Phi) / z, G_theta and G_phi u-integrals over the mass
// Gaussians (each term w K exp(-r_j u^2 (R^2 + z^2 / h)) times a polynomial
// in u).  The moments summed over the tracers, A_r = sum P_k, A_theta =
// sum (1 - beta_k) P_k and A_phi = sum nu v_phi^2_k, are tabulated on a polar
// grid and interpolated along the line of sight.
// ---------------------------------------------------------------------------
constexpr int kSphChunk = 1024;   // (j, u) terms staged in LDS at a time

__device__ inline SphAdj sph_adj_of(double *sens, const ModelDev &md, const GeomDev &g) {
  return sph_adj_layout(sens + md.sens_off, g.K, g.n_pix, sph_terms_padded(g.J1, g.n_u),
                        md.n_sens_parts);
}

// FP32 coefficients of the (j, u) terms of G, G_theta and G_phi, once per
// model: (-r_j u^2 log2e, -r_j u^2 / h log2e, gP, gT) and gF, zero-padded to
// a whole number of 64-term groups (a zero term adds exactly nothing); for the
// adjoint the same in FP64, with T_theta's weights gT r_j u^2 (1 / h - 1); and the
// potential grid's scales (first item).  Item (m, block of 256 terms); thread =
// term.
__global__ void __launch_bounds__(256) k_sph_terms(const GeomDev *__restrict__ geoms,
                                                   const ModelDev *__restrict__ models,
                                                   const Item *__restrict__ items, int n_it,
                                                   const double *__restrict__ gauss,
                                                   const int *__restrict__ st_ws,
                                                   float4 *__restrict__ terms,
                                                   double *__restrict__ terms64,
                                                   double *__restrict__ pol) {
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    const int nu_n = g.n_u, T = g.J1 * nu_n, Tp = sph_terms_padded(g.J1, nu_n);
    const int t = it.a * 256 + threadIdx.x;
    const bool grid = md.sgrid_slices > 0;
    if (grid && it.a == 0 && threadIdx.x < 64) {
      const double *tab = gauss + md.gauss_off, *e2 = tab + 4 * g.K + g.J1;
      // smallest h = 1 - e_j^2 u^2 over the nodes, max sigma_k^2
      double s0 = 1.0, sk2 = 0.0;
      const double um = g.u[g.n_u - 1];
      for (int j = threadIdx.x; j < g.J1; j += 64) s0 = fmin(s0, fma(-e2[j], um * um, 1.0));
      for (int k = threadIdx.x; k < g.K; k += 64) sk2 = fmax(sk2, 0.5 / tab[k]);
      for (int o = 32; o > 0; o >>= 1) {
        s0 = fmin(s0, __shfl_xor(s0, o, 64));
        sk2 = fmax(sk2, __shfl_xor(sk2, o, 64));
      }
      const double span = (kSphNR - 1) * g.sph_dlnr, rhi = exp(g.sph_lnr0 + span);
      if (threadIdx.x == 0) {
        double *p = pol + md.pol_off;
        p[0] = (kPolN - 6) / (span + 0.5 * log1p(50.0 * sk2 / (rhi * rhi)));   // iX
        p[1] = s0;
        p[2] = (kPolC - 8) / log1p(1.0 / s0);                                  // iC
      }
    }
    if (t >= Tp) continue;
    float4 *tc = terms + md.term_off;
    float *tf = (float *)(tc + Tp);
    SphTerm *t64 = terms64 ? reinterpret_cast<SphTerm *>(terms64 + md.term64_off) : nullptr;
    if (t >= T || st_ws[it.m] != 0) {
      tc[t] = make_float4(0.f, 0.f, 0.f, 0.f);
      tf[t] = 0.f;
      if (t64) t64[t] = SphTerm{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      continue;
    }
    const double *mt = gauss + md.gauss_off + 4 * g.K;
    const int j = t / nu_n, n = t % nu_n;
    const double rj = mt[j], e2 = mt[g.J1 + j], Kp = mt[2 * g.J1 + j];
    const double u = g.u[n], u2 = u * u, wK = g.w[n] * Kp;
    const double hh = 1.0 - e2 * u2, h15 = hh * sqrt(hh);
    const double gT = wK * e2 * 4.0 * rj * rj * u2 * u2 * u2 / (h15 * hh);
    const SphTerm c{-rj * u2 * kLog2e, -rj * u2 / hh * kLog2e, wK * 2.0 * rj * u2 / h15, gT,
                    wK * e2 * 2.0 * rj * u2 * u2 / h15, gT * rj * u2 * (e2 * u2 / hh)};
    tc[t] = make_float4((float)c.cx, (float)c.cy, (float)c.gP, (float)c.gT);
    tf[t] = (float)c.gF;
    if (t64) t64[t] = c;
  }
}

// Item (m, group of four table points): wave w computes point 4 q + w (one
// table point per wave, so no block-wide reductions), taking the tracers two
// per round (each coefficient read from LDS feeds both); lane l is node l of
// the composite Gauss-Legendre rule in tau = ln(r'/r) on [0, ln(r_max / r)],
// r_max^2 = r^2 + 50 sigma_k^2.  The per-model term coefficients go through LDS
// in chunks shared by the four waves; each group of 64 terms is summed in
// FP32 (fully unrolled, the coefficient reads are wave-wide broadcasts) and
// folded into FP64; everything else is FP64; all sums run in a fixed order.
__global__ void __launch_bounds__(256) k_sph_moments(const GeomDev *__restrict__ geoms,
                                                     const ModelDev *__restrict__ models,
                                                     const Item *__restrict__ items, int n_it,
                                                     const double *__restrict__ gauss,
                                                     const float4 *__restrict__ terms,
                                                     const int *__restrict__ st_ws,
                                                     double *__restrict__ table) {
  __shared__ float4 tc[kSphChunk];   // (-c log2e, -d log2e, gP, gT)
  __shared__ float tf[kSphChunk];    // gF
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    const int cell = 4 * it.a + wave;
    double *out = table + md.sph_off + (int64_t)cell * 3;
    if (st_ws[it.m] != 0) {                 // uniform per block
      if (lane < 3) out[lane] = 0.0;
      continue;
    }
    const int K = g.K, Tp = sph_terms_padded(g.J1, g.n_u);
    const float4 *gtc = terms + md.term_off;
    const float *gtf = (const float *)(gtc + Tp);
    const double *tab = gauss + md.gauss_off;
    const int ir = cell / kSphNT, ith = cell % kSphNT;
    const double lnr = g.sph_lnr0 + ir * g.sph_dlnr, r = exp(lnr);
    const double th = ith * (0.5 * kPi / (kSphNT - 1));
    const double sth = sin(th), cth = cos(th);
    const double Rp0 = r * sth, zp0 = r * cth;
    const float R20 = (float)(Rp0 * Rp0), Z20 = (float)(zp0 * zp0);
    const int seg = lane >> 3, gi = lane & 7;
    // the rule's node and weight of this lane, read from global memory (a
    // lane-dependent index into the by-value descriptor would go to scratch)
    const double glx = geoms[md.geom].gl8_x[gi], glw = geoms[md.geom].gl8_w[gi];
    double Ar = 0.0, At = 0.0, Ap = 0.0;   // the point's moments (lane 0)
    double accF = 0.0;                      // this lane's share of G_phi
    constexpr int kTr = 2;                  // tracers per round
    const int rounds = (K + kTr - 1) / kTr; // the same in every wave
    for (int q = 0; q < rounds; ++q) {
      double alpha[kTr], alphaq[kTr], beta[kTr], wn[kTr], nuv[kTr], rp[kTr], Rp[kTr], Zp[kTr];
      double rbe[kTr], rpb[kTr];             // r^beta, r'^beta (the powers are their products)
      float R2[kTr], Z2[kTr];
      bool on[kTr];
#pragma unroll
      for (int u = 0; u < kTr; ++u) {
        const int k = kTr * q + u;
        on[u] = k < K;                      // uniform
        alpha[u] = 1.0; alphaq[u] = 1.0; beta[u] = 0.0; wn[u] = 0.0; nuv[u] = 0.0;
        rp[u] = r; rbe[u] = 1.0; rpb[u] = 1.0; Rp[u] = 0.0; Zp[u] = 0.0; R2[u] = 0.f; Z2[u] = 0.f;
        if (on[u]) {
          alpha[u] = tab[k];
          alphaq[u] = tab[K + k];
          beta[u] = 1.0 - 1.0 / tab[3 * K + k];
          const double tmax = 0.5 * log1p(50.0 * (0.5 / alpha[u]) / (r * r));
          const double hs = tmax / kSphSeg;
          const double tau = (seg + 0.5 + 0.5 * glx) * hs;
          rp[u] = exp(lnr + tau);
          // (r'/r)^beta; sin theta' = sin theta (r / r')^(1 - beta)
          const double rbt = exp(beta[u] * tau);
          rbe[u] = exp(beta[u] * lnr);
          rpb[u] = rbe[u] * rbt;
          const double st = fmin(1.0, sth * (r / rp[u]) * rbt);
          const double ct = sqrt(fmax(0.0, 1.0 - st * st));
          Rp[u] = rp[u] * st;
          const double zp = rp[u] * ct;
          Zp[u] = zp;
          R2[u] = (float)(Rp[u] * Rp[u]);
          Z2[u] = (float)(zp * zp);
          wn[u] = 0.5 * glw * hs * rp[u];
          nuv[u] = tab[2 * K + k] * exp(-(alpha[u] * Rp[u] * Rp[u] + alphaq[u] * zp * zp));
        }
      }
      double accG[kTr], accT[kTr];
#pragma unroll
      for (int u = 0; u < kTr; ++u) { accG[u] = 0.0; accT[u] = 0.0; }
      // the terms: the node sums and, in the first round, G_phi at the table
      // point
      for (int c0 = 0; c0 < Tp; c0 += kSphChunk) {
        const int cn = min(kSphChunk, Tp - c0);
        __syncthreads();
        for (int t = threadIdx.x; t < cn; t += 256) {
          tc[t] = gtc[c0 + t];
          tf[t] = gtf[c0 + t];
        }
        __syncthreads();
        for (int t0 = 0; t0 < cn; t0 += 64) {
          float sg0 = 0.f, sd0 = 0.f, sg1 = 0.f, sd1 = 0.f;
#pragma unroll
          for (int t = 0; t < 64; ++t) {
            const float4 c = tc[t0 + t];
            const float e0 = fast_exp2(fmaf(c.x, R2[0], c.y * Z2[0]));
            const float e1 = fast_exp2(fmaf(c.x, R2[1], c.y * Z2[1]));
            sg0 = fmaf(c.z, e0, sg0);
            sd0 = fmaf(c.w, e0, sd0);
            sg1 = fmaf(c.z, e1, sg1);
            sd1 = fmaf(c.w, e1, sd1);
          }
          accG[0] += (double)sg0;
          accT[0] += (double)sd0;
          accG[1] += (double)sg1;
          accT[1] += (double)sd1;
        }
        if (q == 0) {
          for (int t = lane; t < cn; t += 64) {
            const float4 c = tc[t];
            accF += (double)(tf[t] * fast_exp2(fmaf(c.x, R20, c.y * Z20)));
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kTr; ++u) {
        if (!on[u]) continue;
        const double sk2 = 0.5 / alpha[u], qk2 = alpha[u] / alphaq[u];
        // r'^(2 beta + 1) and r'^(3 beta + 1)
        const double p2 = rp[u] * rpb[u] * rpb[u], p3 = p2 * rpb[u];
        double fP = wn[u] * p2 * nuv[u] * accG[u];
        double fD = wn[u] * p3 * Rp[u] * nuv[u] * (accT[u] + accG[u] * (1.0 / qk2 - 1.0) / sk2);
        fP = wave_sum(fP);
        fD = wave_sum(fD);
        // r^(-2 beta) and r^(1 - 3 beta)
        const double rb2 = rbe[u] * rbe[u];
        const double P = fP / rb2;
        Ar += P;
        At += (1.0 - beta[u]) * P;
        Ap += (1.0 - beta[u]) * P + (1.0 - beta[u]) * sth * (r / (rb2 * rbe[u])) * fD;
      }
    }
    // G_phi and the tracer density at the point, lane sums in a fixed order
    const double Gphi = wave_sum(accF);
    double nus = 0.0;
    for (int k = lane; k < K; k += 64)
      nus += tab[2 * K + k] * exp(-(tab[k] * Rp0 * Rp0 + tab[K + k] * zp0 * zp0));
    nus = wave_sum(nus);
    if (lane == 0) {
      out[0] = Ar;
      out[1] = At;
      out[2] = Ap - nus * Rp0 * Rp0 * Gphi;
    }
  }
}

// ---------------------------------------------------------------------------
// Adjoint of the spherically aligned model.  With lambda_N per unique pixel
// (bin adjoint) the chain runs back through the line-of-sight rule (to the
// table and, at fixed table, to i and the node scale a), through the
// characteristic integrals (to beta_k, alphaq_k, nu0_k per table cell and
// tracer, and to the (j, u) term coefficients by term-major sums over all
// (cell, tracer, node) points), through the term coefficients (to e_j^2 and
// K_j), and through the set-up to the parameters.  FP64 except the FP32
// exponentials and their sums over 64 or 256 points, as in the forward.
// ---------------------------------------------------------------------------

// Radial interpolation of the moment table: Catmull-Rom (cubic convolution,
// a = -1/2) in ln r over the radii xi - 1 .. xi + 2 around the cell [xi,
// xi + 1] holding fraction fx; at the ends of the range the missing radius is
// the linear extrapolation of the two nearest, folded into the weights.
// ew: weights of radii xi - 1 + a (0 where out of range); dew: d ew / d fx.
__device__ inline void sph_radial_weights(int xi, double fx, double *ew, double *dew) {
  const double f2 = fx * fx, f3 = f2 * fx;
  ew[0] = 0.5 * (-f3 + 2.0 * f2 - fx);
  ew[1] = 0.5 * (3.0 * f3 - 5.0 * f2 + 2.0);
  ew[2] = 0.5 * (-3.0 * f3 + 4.0 * f2 + fx);
  ew[3] = 0.5 * (f3 - f2);
  dew[0] = 0.5 * (-3.0 * f2 + 4.0 * fx - 1.0);
  dew[1] = 0.5 * (9.0 * f2 - 10.0 * fx);
  dew[2] = 0.5 * (-9.0 * f2 + 8.0 * fx + 1.0);
  dew[3] = 0.5 * (3.0 * f2 - 2.0 * fx);
  if (xi == 0) {                  // radius -1 = 2 r_0 - r_1
    ew[1] += 2.0 * ew[0];
    ew[2] -= ew[0];
    ew[0] = 0.0;
    dew[1] += 2.0 * dew[0];
    dew[2] -= dew[0];
    dew[0] = 0.0;
  }
  if (xi + 2 > kSphNR - 1) {      // radius NR = 2 r_(NR-1) - r_(NR-2)
    ew[2] += 2.0 * ew[3];
    ew[1] -= ew[3];
    ew[3] = 0.0;
    dew[2] += 2.0 * dew[3];
    dew[1] -= dew[3];
    dew[3] = 0.0;
  }
}

// Angular weights, Catmull-Rom in theta over the angles yi - 1 .. yi + 2.
__device__ inline void sph_angular_weights(double fy, double *ew, double *dew) {
  const double f2 = fy * fy, f3 = f2 * fy;
  ew[0] = 0.5 * (-f3 + 2.0 * f2 - fy);
  ew[1] = 0.5 * (3.0 * f3 - 5.0 * f2 + 2.0);
  ew[2] = 0.5 * (-3.0 * f3 + 4.0 * f2 + fy);
  ew[3] = 0.5 * (f3 - f2);
  dew[0] = 0.5 * (-3.0 * f2 + 4.0 * fy - 1.0);
  dew[1] = 0.5 * (9.0 * f2 - 10.0 * fy);
  dew[2] = 0.5 * (-9.0 * f2 + 8.0 * fy + 1.0);
  dew[3] = 0.5 * (3.0 * f2 - 2.0 * fy);
}

// ---------------------------------------------------------------------------
// Line of sight.  The table of a model fits the LDS (80 KB), with a mirrored
// column on either side (the moments are even about theta = 0 and pi / 2; slot
// s holds angle s - 1), so that a stencil row is twelve contiguous doubles.
// A block takes a contiguous range of the 64-pixel items, loading the table
// where the model changes; 16 lanes per pixel, four nodes each (the adjoint
// lays its lanes out otherwise).
// Node quantities that no pixel changes are computed once per model.
// ---------------------------------------------------------------------------
constexpr int kLosThreads = 1024, kLosAdjThreads = 512, kLosBlocks = 256;
constexpr int kLosCols = kSphNT + 2;

// Nodes z' = a sinh(w), w on [-W, W] by the composite rule, a = min_k sigma_k
// q_k / 4, a sinh(W) = 12 max_k sigma_k.
struct LosNode {
  double zp, wz;           // position, weight
  double dzp, dwz;         // their derivatives with respect to a (adjoint)
};
struct LosModel {
  double si, ci;
};
// One whole wave, lane = node.
__device__ inline void los_setup(const GeomDev &g, const double *tab, LosNode *nodes, LosModel &m) {
  const int K = g.K, lane = threadIdx.x & 63;
  const double *mt = tab + 4 * K;
  double smin = 1e300, smax = 0.0;
  for (int k = lane; k < K; k += 64) {
    const double sk = sqrt(0.5 / tab[k]), qk = sqrt(tab[k] / tab[K + k]);
    smin = fmin(smin, sk * qk);
    smax = fmax(smax, sk);
  }
  for (int o = 32; o > 0; o >>= 1) {
    smin = fmin(smin, __shfl_xor(smin, o, 64));
    smax = fmax(smax, __shfl_xor(smax, o, 64));
  }
  const double a = 0.25 * smin, cW = 12.0 * smax, W = asinh(cW / a);
  const double Wa = -(cW / (a * a)) / sqrt(1.0 + (cW / a) * (cW / a));   // dW/da
  const double hw = 2.0 * W / kSphSeg, glx = g.gl8_x[lane & 7], glw = g.gl8_w[lane & 7];
  const double om = -1.0 + ((lane >> 3) + 0.5 + 0.5 * glx) / 4.0;         // w = W om
  const double w = -W + ((lane >> 3) + 0.5 + 0.5 * glx) * hw;
  // sinh w, cosh w from one exponential (|w| > 0.004 W at every node)
  const double ex = exp(w), iex = 1.0 / ex, shw = 0.5 * (ex - iex), chw = 0.5 * (ex + iex);
  nodes[lane] = LosNode{a * shw, 0.5 * glw * hw * a * chw, shw + a * chw * om * Wa,
                        0.5 * glw * (2.0 / kSphSeg) *
                            (Wa * a * chw + W * chw + W * a * shw * om * Wa)};
  if (lane == 0) m = LosModel{sqrt(mt[3 * g.J1]), sqrt(mt[3 * g.J1 + 1])};
}
// The whole block: table with mirrored columns to LDS.
__device__ inline void los_table(const double *__restrict__ T, double *t) {
  for (int e = threadIdx.x; e < kSphNR * kLosCols * 3; e += blockDim.x) {
    const int row = e / (kLosCols * 3), q = e % (kLosCols * 3), s = q / 3, f = q % 3;
    const int c = s == 0 ? 1 : (s == kLosCols - 1 ? kSphNT - 2 : s - 1);
    t[e] = T[(row * kSphNT + c) * 3 + f];
  }
}
// A node of a pixel: where it falls in the table.
struct LosPoint {
  double X, Y, Z, iR, ir;  // position; 1 / R (zero on the axis), 1 / r
  double xf;               // radial index (fractional); fx, fy the cell fractions
  double fx, fy;
  int xi, yi;
};
__device__ __forceinline__ LosPoint los_point(const GeomDev &g, double x, double y, double zp,
                                              const LosModel &m, double idlnr, const LosMath &mt) {
  LosPoint p;
  p.X = x;
  p.Y = zp * m.si - y * m.ci;
  p.Z = y * m.si + zp * m.ci;
  const double R2 = fma(p.X, p.X, p.Y * p.Y), r2 = fma(p.Z, p.Z, R2);
  p.iR = R2 > 0.0 ? rsq64(fmax(R2, 1e-300)) : 0.0;
  p.ir = rsq64(r2);
  p.xf = fma(0.5, pol_log(r2, mt), -g.sph_lnr0) * idlnr;
  const double yf = los_atan(R2 * p.iR, fabs(p.Z), mt) * ((kSphNT - 1) / (0.5 * kPi));
  p.xi = min(max((int)floor(p.xf), 0), kSphNR - 2);
  p.yi = min((int)yf, kSphNT - 2);
  p.fx = fmin(fmax(p.xf - p.xi, 0.0), 1.0);
  p.fy = fmin(fmax(yf - p.yi, 0.0), 1.0);
  return p;
}

// Node of tracer k's characteristic through table point (r, theta): the same
// FP64 operations as the forward moment kernel.
struct SphNode {
  double rp, st, ct, Rp, zp, wn, en, tau, rbt;   // rbt = (r'/r)^beta
  bool clamped;
};
__device__ inline SphNode sph_node(double r, double lnr, double sth, double alpha, double alphaq,
                                   double beta, int seg, double glx, double glw) {
  SphNode o;
  const double tmax = 0.5 * log1p(50.0 * (0.5 / alpha) / (r * r));
  const double hs = tmax / kSphSeg;
  o.tau = (seg + 0.5 + 0.5 * glx) * hs;
  o.rp = exp(lnr + o.tau);
  o.rbt = exp(beta * o.tau);
  const double sraw = sth * (r / o.rp) * o.rbt;   // sin theta (r / r')^(1 - beta)
  o.clamped = !(sraw < 1.0);
  o.st = fmin(1.0, sraw);
  o.ct = sqrt(fmax(0.0, 1.0 - o.st * o.st));
  o.Rp = o.rp * o.st;
  o.zp = o.rp * o.ct;
  o.wn = 0.5 * glw * hs * o.rp;
  o.en = exp(-(alpha * o.Rp * o.Rp + alphaq * o.zp * o.zp));
  return o;
}

__device__ inline void sph_cell(const GeomDev &g, int cell, double &r, double &sth, double &cth) {
  const int ir = cell / kSphNT, ith = cell % kSphNT;
  r = exp(g.sph_lnr0 + ir * g.sph_dlnr);
  const double th = ith * (0.5 * kPi / (kSphNT - 1));
  sth = sin(th);
  cth = cos(th);
}


// Start of the line-of-sight adjoint, kZeroParts blocks per model: each clears
// its share of the table cotangent and sums |lambda_N| over its share of the
// pixels (into SphAdj::tchain, which the per-term chain writes later).
constexpr int kZeroParts = 32;
__global__ void __launch_bounds__(256) k_sph_zero(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models, int n,
                                                  const int *__restrict__ st_ws,
                                                  const double *__restrict__ pix,
                                                  double *__restrict__ sens) {
  __shared__ double sh[4];
  static_assert(3 * kSphCells % kZeroParts == 0, "equal shares");
  for (int i = blockIdx.x; i < n * kZeroParts; i += gridDim.x) {
    const int m = i / kZeroParts, part = i % kZeroParts;
    const ModelDev md = models[m];
    const GeomDev &g = geoms[md.geom];
    const SphAdj adj = sph_adj_of(sens, md, g);
    unsigned long long *d = reinterpret_cast<unsigned long long *>(adj.dtab);
    constexpr int kShare = 3 * kSphCells / kZeroParts;
    for (int e = threadIdx.x; e < kShare; e += 256) d[part * kShare + e] = 0ull;
    if (st_ws[m] != 0) continue;   // uniform per block
    const double *lam = pix + md.pix_off + 2 * (int64_t)g.n_pix;
    double s = 0.0;
    for (int q = part * 256 + threadIdx.x; q < g.n_pix; q += kZeroParts * 256) s += fabs(lam[q]);
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) adj.tchain[part] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
    __syncthreads();                 // sh read before the next item
  }
}

// The table cotangent's fixed-point scale, by one whole wave.  Every
// contribution is lambda_N w_z (n.e_f)^2 times interpolation weights, so the
// sum of their magnitudes over all pixels, nodes and cells is at most
// sum_p |lambda_N| x sum_nodes w_z (the node rule integrates a cosh(w) over
// [-W, W]: 2 a sinh W = 24 max sigma_k, taken as 25) x sum |radial weights|
// x sum |angular weights| (each below 2; sum_f (n.e_f)^2 = 1).  The scale is
// the power of two that maps that bound below 2^61 (at most 2^1000, for
// tiny bounds), so the 64-bit integer sums cannot overflow and do not depend
// on the order of the additions.  A non-finite bound gives NaN, which
// k_sph_dtab_fix turns into a NaN cotangent.
__device__ inline double sph_dtab_scale(const GeomDev &g, const double *tab, const SphAdj &adj) {
  const int lane = threadIdx.x & 63;
  const double s = wave_sum(lane < kZeroParts ? adj.tchain[lane] : 0.0);
  double smax = 0.0;
  for (int k = lane; k < g.K; k += 64) smax = fmax(smax, sqrt(0.5 / tab[k]));
  for (int o = 32; o > 0; o >>= 1) smax = fmax(smax, __shfl_xor(smax, o, 64));
  const double bound = s * 25.0 * smax * 4.0;
  if (bound == 0.0) return 1.0;
  if (!(bound < __builtin_inf())) return __builtin_nan("");
  return ldexp(1.0, min(1000, 60 - ilogb(bound)));
}

// The fixed-point table cotangent to FP64: kFixParts blocks per model.
constexpr int kFixParts = 9;
__global__ void __launch_bounds__(256) k_sph_dtab_fix(const GeomDev *__restrict__ geoms,
                                                      const ModelDev *__restrict__ models, int n,
                                                      const int *__restrict__ st_ws,
                                                      double *__restrict__ sens) {
  constexpr int kShare = 3 * kSphCells / kFixParts;
  static_assert(kShare * kFixParts == 3 * kSphCells, "equal shares");
  for (int i = blockIdx.x; i < n * kFixParts; i += gridDim.x) {
    const int m = i / kFixParts, e0 = (i % kFixParts) * kShare;
    if (st_ws[m] != 0) continue;
    const ModelDev md = models[m];
    const SphAdj adj = sph_adj_of(sens, md, geoms[md.geom]);
    const double scale = adj.dscale[0];
    long long *d = reinterpret_cast<long long *>(adj.dtab);
    for (int e = e0 + threadIdx.x; e < e0 + kShare; e += 256) {
      const long long v = d[e];
      adj.dtab[e] = scale == scale ? (double)v / scale : scale;
    }
  }
}

// v rounded to an integer, |v| < 2^62: two halves by adding 1.5 x 2^52 (the
// conversion instructions stop at 32 bits).
__device__ __forceinline__ long long los_round(double v) {
  constexpr double kM = 6755399441055744.0;
  const double t = fma(v, 0x1p-30, kM), u = fma(t - kM, -0x1p30, v) + kM;
  return (long long)__double2loint(t) * (1ll << 30) + (long long)__double2loint(u);
}

// Line-of-sight adjoint.  Item (m, a): the pixels a, a + n, a + 2 n, .. of the
// n = ceil(n_pix / 64) items, lane = pixel, the nodes over the waves: pixels
// spread over the map at the same node, so that the lanes of an atomic add meet
// few equal cells (neighbouring pixels, or the many nodes of one pixel that are
// near the plane of the sky, share theirs).  The table cotangent receives
// lambda_N w_z (n.e_f)^2 times the interpolation weights, each rounded to a
// 64-bit fixed-point integer at the model's scale, accumulated in a
// block-private LDS copy of the table (integer LDS atomics) and added to the
// model's table once per block and model (integer global atomics, non-zero
// entries only): integer sums, so the result does not depend on the order of
// the additions.  The derivatives of the node's integrand at fixed table with
// respect to i (line of sight and node position) and to the node scale a
// are summed per item in a fixed order (butterflies over each wave, then
// the waves in order).
// FP64 issue bounds it, half of it the 48 roundings and LDS atomics per node.
// Measured, 46,225 pixels: 256-thread blocks reading the table from global
// memory with library functions and all node quantities per pixel 303 us, this
// 205 us.
__global__ void __launch_bounds__(kLosAdjThreads) k_sph_num_adj(
    const GeomDev *__restrict__ geoms, const ModelDev *__restrict__ models,
    const Item *__restrict__ items, int n_it, const double *__restrict__ gauss,
    const int *__restrict__ st_ws, const double *__restrict__ table,
    const double *__restrict__ pix, double *__restrict__ sens) {
  __shared__ double T[kSphNR * kLosCols * 3];
  __shared__ unsigned long long ldt[3 * kSphCells];
  __shared__ LosNode nodes[64];
  __shared__ LosMath mt;
  __shared__ LosModel lm;
  __shared__ double wred[kLosAdjThreads / 64][2];
  __shared__ double scale_sh;
  constexpr int kLosNodes = kSphNodes * 64 / kLosAdjThreads;   // nodes per wave
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  los_math_fill(mt);
  const int i0 = (int)((int64_t)n_it * blockIdx.x / gridDim.x);
  const int i1 = (int)((int64_t)n_it * (blockIdx.x + 1) / gridDim.x);
  int cur = -1;                                  // the model whose table is loaded
  auto flush = [&](int m) {
    const ModelDev md = models[m];
    unsigned long long *dt =
        reinterpret_cast<unsigned long long *>(sph_adj_of(sens, md, geoms[md.geom]).dtab);
    for (int e = threadIdx.x; e < 3 * kSphCells; e += kLosAdjThreads) {
      const unsigned long long v = ldt[e];
      if (v != 0ull) atomicAdd(dt + e, v);
    }
  };
  for (int ii = i0; ii < i1; ++ii) {
    const Item it = items[ii];
    if (st_ws[it.m] != 0) continue;              // uniform per block
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const SphAdj adj = sph_adj_of(sens, md, g);
    if (it.m != cur) {
      __syncthreads();                           // the previous model's reads and sums
      if (cur >= 0) flush(cur);
      __syncthreads();
      for (int e = threadIdx.x; e < 3 * kSphCells; e += kLosAdjThreads) ldt[e] = 0ull;
      los_table(table + md.sph_off, T);
      const double *tab = gauss + md.gauss_off;
      if (threadIdx.x < 64) los_setup(g, tab, nodes, lm);
      if (threadIdx.x >= 64 && threadIdx.x < 128) {
        const double sc = sph_dtab_scale(g, tab, adj);
        if (threadIdx.x == 64) {
          scale_sh = sc;
          if (it.a == 0) adj.dscale[0] = sc;     // for k_sph_dtab_fix
        }
      }
      cur = it.m;
      __syncthreads();
    }
    const double scale = scale_sh;
    const bool fixed = scale == scale;           // NaN: non-finite cotangent
    const int q = it.a + lane * ((g.n_pix + 63) / 64);
    const bool on = q < g.n_pix;
    const double x = on ? g.xs[q % g.n_ux] : 0.0, y = on ? g.ys[q / g.n_ux] : 0.0;
    const double lamN = on ? pix[md.pix_off + 2 * (int64_t)g.n_pix + q] : 0.0;
    const double si = lm.si, ci = lm.ci, idlnr = 1.0 / g.sph_dlnr;
    constexpr double kIdth = (kSphNT - 1) / (0.5 * kPi);
    double acc_i = 0.0, acc_a = 0.0;
    for (int jn = 0; on && jn < kLosNodes; ++jn) {
      const LosNode nn = nodes[kLosNodes * wave + jn];
      const LosPoint p = los_point(g, x, y, nn.zp, lm, idlnr, mt);
      if (p.xf > kSphNR - 1) continue;
      const double ct = p.Z * p.ir, R2 = fma(p.X, p.X, p.Y * p.Y), R = R2 * p.iR, st = R * p.ir;
      const double sp = p.Y * p.iR, cp = p.X * p.iR;
      const double ner = si * st * sp + ci * ct, net = si * ct * sp - ci * st, nep = si * cp;
      const double nf[3] = {ner, net, nep};
      double ew[4], dew[4], tw[4], dtw[4];
      sph_radial_weights(p.xi, p.fx, ew, dew);
      sph_angular_weights(p.fy, tw, dtw);
      const bool xin = p.xf >= 0.0;        // below the first radius the table is constant
      double A[3] = {0.0, 0.0, 0.0}, AL[3] = {0.0, 0.0, 0.0}, AT[3] = {0.0, 0.0, 0.0};
      double base[3];
#pragma unroll
      for (int f = 0; f < 3; ++f) base[f] = lamN * nn.wz * nf[f] * nf[f] * scale;
      // columns of the unmirrored cotangent
      int lc[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int c = abs(p.yi - 1 + b);
        lc[b] = (c > kSphNT - 1 ? 2 * (kSphNT - 1) - c : c) * 3;
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int row = min(max(p.xi - 1 + a, 0), kSphNR - 1);   // out of range: zero weight
        const double *c = T + (row * kLosCols + p.yi) * 3;
        unsigned long long *d = ldt + row * (kSphNT * 3);
        double rt[3] = {0.0, 0.0, 0.0}, rd[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int f = 0; f < 3; ++f) {
            rt[f] = fma(tw[b], c[3 * b + f], rt[f]);
            rd[f] = fma(dtw[b], c[3 * b + f], rd[f]);
          }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
          A[f] = fma(ew[a], rt[f], A[f]);
          AL[f] = fma(dew[a], rt[f], AL[f]);
          AT[f] = fma(ew[a], rd[f], AT[f]);
        }
        if (fixed) {
#pragma unroll
          for (int f = 0; f < 3; ++f) {
            const double bf = base[f] * ew[a];
#pragma unroll
            for (int b = 0; b < 4; ++b)
              atomicAdd(d + lc[b] + f, (unsigned long long)los_round(bf * tw[b]));
          }
        }
      }
      // the weight derivatives are per unit of the table's index steps
#pragma unroll
      for (int f = 0; f < 3; ++f) {
        AL[f] = xin ? AL[f] * idlnr : 0.0;
        AT[f] *= kIdth;
      }
      // derivatives of ln r and theta = atan2(R, |Z|) with respect to Y and Z
      const double ir2 = p.ir * p.ir, sz = p.Z < 0.0 ? -1.0 : 1.0;
      const double lY = p.Y * ir2, lZ = p.Z * ir2;
      const double tY = fabs(p.Z) * sp * ir2, tZ = -R * sz * ir2;
      // line-of-sight components and their derivatives (Y, Z; explicit i);
      // on the axis (iR = 0) those of the angular components are left out
      double nY[3], nZ[3], ni[3];
      nY[0] = (si - ner * p.Y * p.ir) * p.ir;
      nZ[0] = (ci - ner * p.Z * p.ir) * p.ir;
      ni[0] = (ci * p.Y - si * p.Z) * p.ir;
      const double irR = p.ir * p.iR, rr = R2 > 0.0 ? fma(p.Z, p.Z, R2) * p.ir : 0.0;
      nY[1] = ((si * p.Z - 2.0 * ci * p.Y) - net * (p.Y * p.ir * R + rr * sp)) * irR;
      nZ[1] = (si * p.Y - net * ct * R) * irR;
      ni[1] = (ci * p.Z * p.Y + si * R2) * irR;
      nY[2] = -si * cp * sp * p.iR;
      nZ[2] = 0.0;
      ni[2] = ci * cp;
      double F = 0.0, FY = 0.0, FZ = 0.0, Fi = 0.0;
#pragma unroll
      for (int f = 0; f < 3; ++f) {
        const double dAY = AL[f] * lY + AT[f] * tY, dAZ = AL[f] * lZ + AT[f] * tZ;
        F += nf[f] * nf[f] * A[f];
        FY += 2.0 * nf[f] * nY[f] * A[f] + nf[f] * nf[f] * dAY;
        FZ += 2.0 * nf[f] * nZ[f] * A[f] + nf[f] * nf[f] * dAZ;
        Fi += 2.0 * nf[f] * ni[f] * A[f];
      }
      const double Yi = nn.zp * ci + y * si, Zi = y * ci - nn.zp * si;
      acc_i += lamN * nn.wz * (Fi + FY * Yi + FZ * Zi);
      acc_a += lamN * (nn.dwz * F + nn.wz * (FY * si + FZ * ci) * nn.dzp);
    }
    // fixed-order sums: each wave's 64 lanes by a butterfly, then the waves
    acc_i = wave_sum(acc_i);
    acc_a = wave_sum(acc_a);
    if ((threadIdx.x & 63) == 0) {
      wred[threadIdx.x >> 6][0] = acc_i;
      wred[threadIdx.x >> 6][1] = acc_a;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
      double v = 0.0;
      for (int w = 0; w < kLosAdjThreads / 64; ++w) v += wred[w][threadIdx.x];
      adj.losp[2 * it.a + threadIdx.x] = v;
    }
    __syncthreads();                             // wred read before the next item
  }
  __syncthreads();
  if (cur >= 0) flush(cur);
}

// Forward pass of the adjoint: the moment table (as k_sph_moments) with the
// node sums its adjoint needs.  Item (m, table cell), the forward's layout:
// wave w takes tracers 8 q + w and 8 q + 4 + w, lane = node.  Per node the
// term sums G, G_theta and their derivatives in R'^2 and z'^2; per (cell,
// tracer) the node sums of the characteristic integrals (fP, fD) and of
// their derivatives with respect to beta_k (bP, bD), alphaq_k (qP, qD) and
// nu0_k (eP, eD) go to SphAdj::jac, none of which depends on the table
// cotangent, and the cell's G_phi to SphAdj::gphi; k_sph_rows combines
// them with the cotangent once the line-of-sight adjoint has produced it.
__global__ void __launch_bounds__(256) k_sph_moments_jac(const GeomDev *__restrict__ geoms,
                                                         const ModelDev *__restrict__ models,
                                                         const Item *__restrict__ items, int n_it,
                                                         const double *__restrict__ gauss,
                                                         const float4 *__restrict__ terms,
                                                         const int *__restrict__ st_ws,
                                                         double *__restrict__ table,
                                                         double *__restrict__ sens) {
  __shared__ float4 tc[kSphChunk];
  __shared__ float4 tx[kSphChunk];   // (gP c_x, gP c_y, gT c_x, gT c_y)
  __shared__ float tf[kSphChunk];
  __shared__ double sh[256];
  __shared__ double wred[3][4];
  constexpr double kLn2 = 0.6931471805599453;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    double *out = table + md.sph_off + (int64_t)it.a * 3;
    if (st_ws[it.m] != 0) {                  // uniform per block
      if (threadIdx.x < 3) out[threadIdx.x] = 0.0;
      continue;
    }
    const SphAdj adj = sph_adj_of(sens, md, g);
    const int K = g.K, Tp = sph_terms_padded(g.J1, g.n_u);
    const float4 *gtc = terms + md.term_off;
    const float *gtf = (const float *)(gtc + Tp);
    const double *tab = gauss + md.gauss_off;
    const int cell = it.a;
    double r, sth, cth;
    sph_cell(g, cell, r, sth, cth);
    const double lnr = g.sph_lnr0 + (cell / kSphNT) * g.sph_dlnr;   // ln r (r = e^lnr)
    const double Rp0 = r * sth, zp0 = r * cth;
    const float R20 = (float)(Rp0 * Rp0), Z20 = (float)(zp0 * zp0);
    const int seg = lane >> 3, gi = lane & 7;
    const double glx = geoms[md.geom].gl8_x[gi], glw = geoms[md.geom].gl8_w[gi];
    double accF = 0.0;
    double Ar = 0.0, At = 0.0, Ap = 0.0;    // this wave's tracers (lane 0)
    constexpr int kTr = 2;                  // tracers per wave and round
    const int rounds = (K + 4 * kTr - 1) / (4 * kTr);
    for (int q = 0; q < rounds; ++q) {
      int kk[kTr];
      bool on[kTr];
      double alpha[kTr], alphaq[kTr], beta[kTr], nu0[kTr];
      SphNode nd[kTr];
      float R2[kTr], Z2[kTr];
#pragma unroll
      for (int u = 0; u < kTr; ++u) {
        kk[u] = 4 * (kTr * q + u) + wave;
        on[u] = kk[u] < K;                  // uniform per wave
        alpha[u] = 1.0; alphaq[u] = 1.0; beta[u] = 0.0; nu0[u] = 0.0;
        nd[u] = SphNode{};
        R2[u] = 0.f; Z2[u] = 0.f;
        if (on[u]) {
          const int k = kk[u];
          alpha[u] = tab[k];
          alphaq[u] = tab[K + k];
          nu0[u] = tab[2 * K + k];
          beta[u] = 1.0 - 1.0 / tab[3 * K + k];
          nd[u] = sph_node(r, lnr, sth, alpha[u], alphaq[u], beta[u], seg, glx, glw);
          R2[u] = (float)(nd[u].Rp * nd[u].Rp);
          Z2[u] = (float)(nd[u].zp * nd[u].zp);
        }
      }
      double aG[kTr], aT[kTr], aGR[kTr], aGZ[kTr], aTR[kTr], aTZ[kTr];
#pragma unroll
      for (int u = 0; u < kTr; ++u) aG[u] = aT[u] = aGR[u] = aGZ[u] = aTR[u] = aTZ[u] = 0.0;
      // the terms: the node sums and, in the first round, G_phi at the table
      // point
      for (int c0 = 0; c0 < Tp; c0 += kSphChunk) {
        const int cn = min(kSphChunk, Tp - c0);
        __syncthreads();
        for (int t = threadIdx.x; t < cn; t += 256) {
          const float4 c = gtc[c0 + t];
          tc[t] = c;
          tx[t] = make_float4(c.z * c.x, c.z * c.y, c.w * c.x, c.w * c.y);
          tf[t] = gtf[c0 + t];
        }
        __syncthreads();
        if (on[0]) {
          for (int t0 = 0; t0 < cn; t0 += 64) {
            float sG0 = 0.f, sT0 = 0.f, sGR0 = 0.f, sGZ0 = 0.f, sTR0 = 0.f, sTZ0 = 0.f;
            float sG1 = 0.f, sT1 = 0.f, sGR1 = 0.f, sGZ1 = 0.f, sTR1 = 0.f, sTZ1 = 0.f;
#pragma unroll 16
            for (int t = 0; t < 64; ++t) {
              const float4 c = tc[t0 + t], d = tx[t0 + t];
              const float e0 = fast_exp2(fmaf(c.x, R2[0], c.y * Z2[0]));
              const float e1 = fast_exp2(fmaf(c.x, R2[1], c.y * Z2[1]));
              sG0 = fmaf(c.z, e0, sG0);
              sT0 = fmaf(c.w, e0, sT0);
              sGR0 = fmaf(d.x, e0, sGR0);
              sGZ0 = fmaf(d.y, e0, sGZ0);
              sTR0 = fmaf(d.z, e0, sTR0);
              sTZ0 = fmaf(d.w, e0, sTZ0);
              sG1 = fmaf(c.z, e1, sG1);
              sT1 = fmaf(c.w, e1, sT1);
              sGR1 = fmaf(d.x, e1, sGR1);
              sGZ1 = fmaf(d.y, e1, sGZ1);
              sTR1 = fmaf(d.z, e1, sTR1);
              sTZ1 = fmaf(d.w, e1, sTZ1);
            }
            aG[0] += (double)sG0;
            aT[0] += (double)sT0;
            aGR[0] += (double)sGR0;
            aGZ[0] += (double)sGZ0;
            aTR[0] += (double)sTR0;
            aTZ[0] += (double)sTZ0;
            aG[1] += (double)sG1;
            aT[1] += (double)sT1;
            aGR[1] += (double)sGR1;
            aGZ[1] += (double)sGZ1;
            aTR[1] += (double)sTR1;
            aTZ[1] += (double)sTZ1;
          }
        }
        if (q == 0) {
          for (int t = threadIdx.x; t < cn; t += 256) {
            const float4 c = tc[t];
            accF += (double)(tf[t] * fast_exp2(fmaf(c.x, R20, c.y * Z20)));
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kTr; ++u) {
        if (!on[u]) continue;               // uniform per wave
        const SphNode &n = nd[u];
        const double be = beta[u];
        const double kap = 2.0 * (alphaq[u] - alpha[u]);
        const double nu = nu0[u] * n.en;
        const double H = aT[u] + kap * aG[u];
        // d/dbeta of the node: s' = s (r/r')^(1-beta) -> ds'/dbeta = s' tau
        const double ds = n.clamped ? 0.0 : n.st * n.tau;
        const double dc = n.ct > 0.0 ? -n.st * ds / n.ct : 0.0;
        const double dR = n.rp * ds, dz = n.rp * dc;
        const double dR2 = 2.0 * n.Rp * dR, dZ2 = 2.0 * n.zp * dz;
        const double dnu = -nu * (alpha[u] * dR2 + alphaq[u] * dZ2);
        // the term coefficients carry log2 e: dE/d(R'^2) = ln 2 c.x E
        const double dG = kLn2 * (aGR[u] * dR2 + aGZ[u] * dZ2);
        const double dH = kLn2 * (aTR[u] * dR2 + aTZ[u] * dZ2) + kap * dG;
        const double lrp = lnr + n.tau;     // ln r'
        // r'^beta = r^beta (r'/r)^beta; r'^(2 beta + 1), r'^(3 beta + 1)
        const double rbe = exp(be * lnr), rpb = rbe * n.rbt;
        const double pP = n.wn * n.rp * rpb * rpb;
        const double pD = pP * rpb;
        double fP = pP * nu * aG[u];
        double fD = pD * n.Rp * nu * H;
        double bP = pP * (2.0 * lrp * nu * aG[u] + dnu * aG[u] + nu * dG);
        double bD = pD * (3.0 * lrp * n.Rp * nu * H + dR * nu * H + n.Rp * dnu * H +
                          n.Rp * nu * dH);
        double qP = pP * aG[u] * (-n.zp * n.zp * nu);
        double qD = pD * n.Rp * (-n.zp * n.zp * nu * H + nu * 2.0 * aG[u]);
        double eP = pP * n.en * aG[u];
        double eD = pD * n.Rp * n.en * H;
        // the eight node sums; lanes 8 f .. 8 f + 7 hold sum f
        const double vs[8] = {fP, fD, bP, bD, qP, qD, eP, eD};
        const double ys = wave_sum8(vs, lane);
        if ((lane & 7) == 0)
          adj.jac[((int64_t)kk[u] * kSphCells + cell) * 8 + (lane >> 3)] = ys;
        fP = ys;                            // in lane 0
        fD = __shfl(ys, 8, 64);
        if (lane == 0) {
          const double rb2 = rbe * rbe;     // r^(-2 beta), r^(1 - 3 beta) below
          const double P = fP / rb2;
          Ar += P;
          At += (1.0 - be) * P;
          Ap += (1.0 - be) * P + (1.0 - be) * sth * (r / (rb2 * rbe)) * fD;
        }
      }
    }
    if (lane == 0) {
      wred[0][wave] = Ar;
      wred[1][wave] = At;
      wred[2][wave] = Ap;
    }
    const double Gphi = block_sum256(accF, sh);   // synchronises the block
    if (threadIdx.x == 0) {
      double nus = 0.0;
      for (int k = 0; k < K; ++k)
        nus += tab[2 * K + k] * exp(-(tab[k] * Rp0 * Rp0 + tab[K + k] * zp0 * zp0));
      out[0] = ((wred[0][0] + wred[0][1]) + wred[0][2]) + wred[0][3];
      out[1] = ((wred[1][0] + wred[1][1]) + wred[1][2]) + wred[1][3];
      out[2] = (((wred[2][0] + wred[2][1]) + wred[2][2]) + wred[2][3]) - nus * Rp0 * Rp0 * Gphi;
      adj.gphi[cell] = Gphi;
    }
    __syncthreads();
  }
}

// Rows of the characteristic integrals' adjoint: per (cell, tracer) the
// derivatives of the cell's L = lambda . (A_r, A_theta, A_phi) with respect
// to beta_k, alphaq_k and nu0_k from the node sums of k_sph_moments_jac and
// the table cotangent lambda; the A_phi term -nu R^2 G_phi adds its
// alphaq_k, nu0_k derivatives; summed over 64 cells.  Item (m, 64 cells),
// lane = cell, the four waves take the tracers in turn (a thread per tracer of one cell left most
// of a wave idle: 48 models of 10 tracers 136 us, now 25).
__global__ void __launch_bounds__(256) k_sph_rows(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  const double *__restrict__ gauss,
                                                  const int *__restrict__ st_ws,
                                                  double *__restrict__ sens) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    if (st_ws[it.m] != 0) continue;          // uniform per block
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const SphAdj adj = sph_adj_of(sens, md, g);
    const int K = g.K, cell = 64 * it.a + lane;
    const double *tab = gauss + md.gauss_off;
    double r, sth, cth;
    sph_cell(g, cell, r, sth, cth);
    const double R02 = (r * sth) * (r * sth), z02 = (r * cth) * (r * cth);
    const double lr = adj.dtab[3 * cell], lt = adj.dtab[3 * cell + 1], lp = adj.dtab[3 * cell + 2];
    const double Gphi = adj.gphi[cell];
    const double lnr = g.sph_lnr0 + (cell / kSphNT) * g.sph_dlnr;   // ln r (r = e^lnr)
    for (int k = wave; k < K; k += 4) {
      const double *jr = adj.jac + ((int64_t)k * kSphCells + cell) * 8;
      const double fP = jr[0], fD = jr[1], bP = jr[2], bD = jr[3];
      const double qP = jr[4], qD = jr[5], eP = jr[6], eD = jr[7];
      const double be = 1.0 - 1.0 / tab[3 * K + k];
      const double rbe = exp(be * lnr);   // r^beta: r^(-2 beta), r^(1 - 3 beta)
      const double rb = 1.0 / (rbe * rbe), rd = r * rb / rbe;
      const double P = rb * fP;
      const double muP = lr + (1.0 - be) * (lt + lp);
      const double muD = lp * (1.0 - be) * sth * rd;
      const double dbeta = muP * rb * bP + muD * bD - (lt + lp) * P - 2.0 * lnr * muP * P -
                           fD * lp * sth * rd * (1.0 + 3.0 * (1.0 - be) * lnr);
      const double e0 = exp(-(tab[k] * R02 + tab[K + k] * z02));
      const double s0 = wave_sum(dbeta);
      const double s1 =
          wave_sum((muP * rb * qP + muD * qD) + lp * R02 * Gphi * tab[2 * K + k] * e0 * z02);
      const double s2 = wave_sum((muP * rb * eP + muD * eD) + -lp * R02 * Gphi * e0);
      if (lane < 3)
        adj.rows[((int64_t)k * kSphRowParts + it.a) * 3 + lane] = lane == 0 ? s0 : (lane == 1 ? s1 : s2);
    }
  }
}

// Point p = (cell, tracer, node) of a model's characteristic integrals: the
// node (as in the forward, with the powers of r and r' written as
// exponentials of ln r and tau, r' = r e^tau) and the cotangents phi =
// dL/dG and psi = dL/dG_theta there, from the table cotangent in adj.dtab.
// sinth: sin of the table's polar angles; gp: the geometry (its 8-node rule
// is read from global memory: a lane-dependent index into a by-value
// descriptor would go to scratch).
__device__ inline void sph_point_cot(const GeomDev &g, const GeomDev *__restrict__ gp,
                                     const double *tab, const SphAdj &adj, const double *sinth,
                                     int64_t p, double &Rp, double &zp, double &phi,
                                     double &psi) {
  const int K = g.K;
  const int cell = (int)(p / ((int64_t)K * kSphNodes));
  const int k = (int)((p / kSphNodes) % K), node = (int)(p % kSphNodes);
  const int ir = cell / kSphNT, ith = cell % kSphNT;
  const double lnr = g.sph_lnr0 + ir * g.sph_dlnr, r = exp(lnr);
  const double sth = sinth[ith];
  const double lr = adj.dtab[3 * cell], lt = adj.dtab[3 * cell + 1];
  const double lp = adj.dtab[3 * cell + 2];
  const double alpha = tab[k], alphaq = tab[K + k], nu0 = tab[2 * K + k];
  const double beta = 1.0 - 1.0 / tab[3 * K + k];
  const int gi = node & 7;
  const double glx = gp->gl8_x[gi], glw = gp->gl8_w[gi];
  const double hs = 0.5 * log1p(50.0 * (0.5 / alpha) / (r * r)) / kSphSeg;
  const double tau = ((node >> 3) + 0.5 + 0.5 * glx) * hs;
  const double rp = exp(lnr + tau);
  const double rbt = exp(beta * tau);    // (r'/r)^beta
  const double st = fmin(1.0, sth * (r / rp) * rbt);
  const double ct = sqrt(fmax(0.0, 1.0 - st * st));
  Rp = rp * st;
  zp = rp * ct;
  const double wn = 0.5 * glw * hs * rp;
  const double nu = nu0 * exp(-(alpha * Rp * Rp + alphaq * zp * zp));
  const double muP = lr + (1.0 - beta) * (lt + lp);
  // r^beta, r'^beta; r^(1 - 3 beta), r'^(3 beta + 1) and r'^(2 beta + 1)
  // r^(-2 beta) = r' (r'/r)^(2 beta) as their products
  const double rbe = exp(beta * lnr), rpb = rbe * rbt;
  const double muD = lp * (1.0 - beta) * sth * (r / (rbe * rbe * rbe));
  const double dD = muD * wn * (rp * rpb * rpb * rpb) * Rp * nu;
  phi = muP * wn * (rp * rbt * rbt) * nu + dD * 2.0 * (alphaq - alpha);
  psi = dD;
}

// Term-major sensitivities.  Item (m, 256-term tile, point range); thread =
// term.  Each 256-point chunk of the range is regenerated (thread = point):
// node position and the cotangents phi = dL/dG, psi = dL/dG_theta at the
// node; then every term sums phi E, psi E and their z'^2 moments over the chunk in
// FP32, folded into FP64.
__global__ void __launch_bounds__(256) k_sph_sens(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  const double *__restrict__ gauss,
                                                  const float4 *__restrict__ terms,
                                                  const int *__restrict__ st_ws,
                                                  double *__restrict__ sens) {
  __shared__ float4 pa[256];   // (R'^2, z'^2, phi, psi)
  __shared__ float2 pb[256];   // (phi z'^2, psi z'^2)
  __shared__ double sc[2][kSphNT];   // sin, cos of the table's polar angles
  if (threadIdx.x < kSphNT) {
    const double th = threadIdx.x * (0.5 * kPi / (kSphNT - 1));
    sc[0][threadIdx.x] = sin(th);
    sc[1][threadIdx.x] = cos(th);
  }
  __syncthreads();
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;
    const SphAdj adj = sph_adj_of(sens, md, g);
    const int K = g.K, Tp = sph_terms_padded(g.J1, g.n_u);
    const double *tab = gauss + md.gauss_off;
    const int t = it.a * 256 + threadIdx.x;
    const bool tv = t < Tp;
    const float4 c = tv ? terms[md.term_off + t] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int64_t len = sph_range_len(K, md.n_sens_parts), P = sph_points(K);
    const int64_t p0 = (int64_t)it.b * len, p1 = min(P, p0 + len);
    double SP = 0.0, ST = 0.0, SyP = 0.0, SyT = 0.0;
    for (int64_t c0 = p0; c0 < p1; c0 += 256) {
      // regenerate this chunk's points
      const int64_t p = c0 + threadIdx.x;
      float4 va = make_float4(0.f, 0.f, 0.f, 0.f);
      float2 vb = make_float2(0.f, 0.f);
      if (p < p1) {
        double Rp, zp, phi, psi;
        sph_point_cot(g, geoms + md.geom, tab, adj, sc[0], p, Rp, zp, phi, psi);
        const float R2 = (float)(Rp * Rp), Z2 = (float)(zp * zp);
        const float fphi = (float)phi, fpsi = (float)psi;
        va = make_float4(R2, Z2, fphi, fpsi);
        vb = make_float2(fphi * Z2, fpsi * Z2);
      }
      __syncthreads();
      pa[threadIdx.x] = va;
      pb[threadIdx.x] = vb;
      __syncthreads();
      float sP = 0.f, sT = 0.f, syP = 0.f, syT = 0.f;
      if (tv) {
#pragma unroll 16
        for (int j = 0; j < 256; ++j) {   // points past the range are zero
          const float4 A = pa[j];
          const float2 B = pb[j];
          const float e = fast_exp2(fmaf(c.x, A.x, c.y * A.y));
          sP = fmaf(A.z, e, sP);
          sT = fmaf(A.w, e, sT);
          syP = fmaf(B.x, e, syP);
          syT = fmaf(B.y, e, syT);
        }
      }
      SP += (double)sP;
      ST += (double)sT;
      SyP += (double)syP;
      SyT += (double)syT;
    }
    if (tv) {
      double *o = adj.sparts + ((int64_t)it.b * Tp + t) * 4;
      o[0] = SP;
      o[1] = ST;
      o[2] = SyP;
      o[3] = SyT;
    }
    __syncthreads();
  }
}

// Term sensitivities of the table points' G_phi term (chi = -lambda_phi nu
// R0^2 per cell).  Item (m, 256-term tile) split in kSphCellParts parts of
// 256 cells; thread = term.  Each part's sums go to their own slot.  FP64 but for
// the exponential: the cells' signs differ, and FP32 sums over 256 of them left up
// to 2e-6 in a single model's inclination derivative.
__global__ void __launch_bounds__(256) k_sph_sens_cells(const GeomDev *__restrict__ geoms,
                                                        const ModelDev *__restrict__ models,
                                                        const Item *__restrict__ items, int n_it,
                                                        const double *__restrict__ gauss,
                                                        const double *__restrict__ terms64,
                                                        const int *__restrict__ st_ws,
                                                        double *__restrict__ sens) {
  __shared__ double2 px[256];   // R0^2, z0^2
  __shared__ double pc[256];    // chi
  for (int vi = blockIdx.x; vi < n_it * kSphCellParts; vi += gridDim.x) {
    const Item it = items[vi / kSphCellParts];
    const int part = vi % kSphCellParts;
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;
    const SphAdj adj = sph_adj_of(sens, md, g);
    const int K = g.K, Tp = sph_terms_padded(g.J1, g.n_u);
    const double *tab = gauss + md.gauss_off;
    const int t = it.a * 256 + threadIdx.x;
    const bool tv = t < Tp;
    const SphTerm *tc = reinterpret_cast<const SphTerm *>(terms64 + md.term64_off);
    const double cx = tv ? tc[t].cx : 0.0, cy = tv ? tc[t].cy : 0.0;
    double sF = 0.0, sy = 0.0;
    {
      const int cell = part * 256 + threadIdx.x;
      double r, sth, cth;
      sph_cell(g, cell, r, sth, cth);
      const double R0 = r * sth, z0 = r * cth;
      double nus = 0.0;
      for (int k = 0; k < K; ++k) nus += tab[2 * K + k] * exp(-(tab[k] * R0 * R0 + tab[K + k] * z0 * z0));
      __syncthreads();
      px[threadIdx.x] = make_double2(R0 * R0, z0 * z0);
      pc[threadIdx.x] = -adj.dtab[3 * cell + 2] * nus * R0 * R0;
      __syncthreads();
      if (tv) {
        for (int j = 0; j < 256; ++j) {
          const double2 x = px[j];
          const double e = pc[j] * (double)fast_exp2((float)fma(cx, x.x, cy * x.y));
          sF += e;
          sy = fma(x.y, e, sy);
        }
      }
    }
    if (tv) {
      double *o = adj.cparts + ((int64_t)part * Tp + t) * 2;
      o[0] = sF;
      o[1] = sy;
    }
    __syncthreads();
  }
}

// Per-term chain (FP64): the sensitivities summed over the point ranges in a
// fixed order, then through the coefficients' dependence on e_j^2 and K_j.
// Item (m, 256-term tile); thread = term.
__global__ void __launch_bounds__(256) k_sph_chain(const GeomDev *__restrict__ geoms,
                                                   const ModelDev *__restrict__ models,
                                                   const Item *__restrict__ items, int n_it,
                                                   const double *__restrict__ gauss,
                                                   const int *__restrict__ st_ws,
                                                   double *__restrict__ sens) {
  constexpr double kLn2 = 0.6931471805599453, kLog2e = 1.4426950408889634;
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;
    const SphAdj adj = sph_adj_of(sens, md, g);
    const int Tp = sph_terms_padded(g.J1, g.n_u), T = g.J1 * g.n_u;
    const int t = it.a * 256 + threadIdx.x;
    if (t >= T) continue;
    double S[4] = {0.0, 0.0, 0.0, 0.0};
    for (int rg = 0; rg < md.n_sens_parts; ++rg) {
      const double *o = adj.sparts + ((int64_t)rg * Tp + t) * 4;
#pragma unroll
      for (int c = 0; c < 4; ++c) S[c] += o[c];
    }
    // the cell parts in order
    double cp[2] = {0.0, 0.0};
    for (int pt = 0; pt < kSphCellParts; ++pt) {
      const double *o = adj.cparts + ((int64_t)pt * Tp + t) * 2;
#pragma unroll
      for (int c = 0; c < 2; ++c) cp[c] += o[c];
    }
    const double *mt = gauss + md.gauss_off + 4 * g.K;
    const int j = t / g.n_u, n = t % g.n_u;
    const double rj = mt[j], e2 = mt[g.J1 + j], Kp = mt[2 * g.J1 + j];
    const double u = g.u[n], u2 = u * u, w = g.w[n];
    const double h = 1.0 - e2 * u2, h15 = h * sqrt(h);
    // coefficients per unit K_j
    const double P1 = w * 2.0 * rj * u2 / h15;
    const double T1 = w * e2 * 4.0 * rj * rj * u2 * u2 * u2 / (h15 * h);
    const double F1 = w * e2 * 2.0 * rj * u2 * u2 / h15;
    const double cy = -rj * u2 / h * kLog2e;
    const double dcy = kLn2 * Kp * (P1 * S[2] + T1 * S[3] + F1 * cp[1]);   // dL/dc_y
    const double dP1 = P1 * 1.5 * u2 / h;
    const double dT1 = w * 4.0 * rj * rj * u2 * u2 * u2 * (1.0 / (h15 * h) + e2 * 2.5 * u2 / (h15 * h * h));
    const double dF1 = w * 2.0 * rj * u2 * u2 * (1.0 / h15 + e2 * 1.5 * u2 / (h15 * h));
    double *o = adj.tchain + (int64_t)t * 2;
    o[0] = Kp * (S[0] * dP1 + S[1] * dT1 + cp[0] * dF1) + dcy * cy * u2 / h;   // d/de2
    o[1] = S[0] * P1 + S[1] * T1 + cp[0] * F1;                                // d/dKp
  }
}

// Per-model gradients.  Block per model: sums over cells (rows), u-nodes
// (per-term chain) and pixel blocks (line-of-sight partials) in a fixed
// order, then the set-up's derivatives (App. A) to the parameters.
__global__ void __launch_bounds__(512) k_sph_grads(const GeomDev *__restrict__ geoms,
                                                   const ModelDev *__restrict__ models, int n,
                                                   ParamsDev p, const double *__restrict__ gauss,
                                                   const int *__restrict__ st_ws,
                                                   double *__restrict__ sens,
                                                   const double *__restrict__ sbp, GradsDev out) {
  constexpr int kW = 8;    // waves per block
  __shared__ double sh[4][kW];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  for (int m = blockIdx.x; m < n; m += gridDim.x) {
    const ModelDev md = models[m];
    const GeomDev g = geoms[md.geom];
    const bool ok = st_ws[m] == 0;
    const double nan = __builtin_nan("");
    const int K = g.K, J1 = g.J1, J = J1 - 1;
    const SphAdj adj = sph_adj_of(sens, md, g);
    const double *tab = gauss + md.gauss_off;
    const double *mt = tab + 4 * K;
    const double inc = p.inc[m];
    const double si = sin(inc), ci = cos(inc);
    // dq/di of a deprojected Gaussian of observed axis ratio qo
    auto dqdi = [&](double qo, double q) { return ci * (1.0 - qo * qo) / (q * si * si * si); };
    double di = 0.0;
    // tracers: the rows' sums over 64 cells each
    for (int k = wave; k < K; k += kW) {
      double b = 0.0, aq = 0.0, nv = 0.0;
      if (ok && lane < kSphRowParts) {
        const double *row = adj.rows + ((int64_t)k * kSphRowParts + lane) * 3;
        b = row[0];
        aq = row[1];
        nv = row[2];
      }
      double sb = 0.0;
      const int n_tiles = sb_tiles(g.n_ux, g.n_uy);
      if (ok)
        for (int tl = lane; tl < n_tiles; tl += 64) sb += sbp[md.sbp_off + (int64_t)k * n_tiles + tl];
      b = wave_sum(b);
      aq = wave_sum(aq);
      nv = wave_sum(nv);
      sb = wave_sum(sb);
      if (lane == 0) {
        const double qo = g.lum_q[k], sk = g.lum_sigma[k];
        const double alpha = tab[k], q = sqrt(alpha / tab[K + k]);
        const double dq = dqdi(qo, q);
        // alphaq = alpha / q^2, nu0 = qo I0 / (sqrt(2 pi) sigma q)
        di += aq * (-2.0 * alpha / (q * q * q)) * dq + nv * (-tab[2 * K + k] / q) * dq;
        if (out.beta) out.beta[md.lum_off + k] = ok ? b : nan;
        if (out.lum_I0)
          out.lum_I0[md.lum_off + k] =
              ok ? nv * qo / (sqrt(2.0 * kPi) * sk * q) + sb : nan;
      }
    }
    // mass Gaussians and the BH: per-term chain summed over u-nodes
    const double sp = g.s_pc, Gc = grav_const();
    const double ml = p.mass_scale[m];
    double dml = 0.0;
    for (int j = wave; j < J1; j += kW) {
      double de2 = 0.0, dK = 0.0;
      if (ok)
        for (int nn = lane; nn < g.n_u; nn += 64) {
          const double *o = adj.tchain + ((int64_t)j * g.n_u + nn) * 2;
          de2 += o[0];
          dK += o[1];
        }
      de2 = wave_sum(de2);
      dK = wave_sum(dK);
      if (lane != 0) continue;
      if (j < J) {
        const double qo = g.mass_q[j], sj = g.mass_sigma[j];
        const double q = sqrt(fmax(1.0 - mt[J1 + j], 0.0));
        di += de2 * (-2.0 * q) * dqdi(qo, q);
        const double S0 = p.mass_S0 ? p.mass_S0[md.mass_off + j] : g.mass_S0[j];
        // K_j = sqrt(2/pi) G M_j / (s sigma_j), M_j = ml 2 pi S0_j (s sigma'_j)^2 q'_j
        const double unit = sqrt(2.0 / kPi) * Gc * 2.0 * kPi * (sp * sj) * (sp * sj) * qo / (sp * sj);
        if (out.mass_S0) out.mass_S0[md.mass_off + j] = ok ? dK * ml * unit : nan;
        dml += dK * S0 * unit;
      } else if (out.m_bh) {
        out.m_bh[m] = ok ? dK * sqrt(2.0 / kPi) * Gc / (sp * g.bh_sigma) : nan;
      }
    }
    // line-of-sight partials: i at fixed node scale, and the node scale
    // a = min_k sigma_k q_k / 4 through its minimising tracer's q_k(i)
    double li = 0.0, la = 0.0;
    const int npb = (g.n_pix + 63) / 64;
    if (ok)
      for (int b = threadIdx.x; b < npb; b += 64 * kW) {
        li += adj.losp[2 * b];
        la += adj.losp[2 * b + 1];
      }
    // fixed-order block sums: wave butterflies, then the wave partials
    di = wave_sum(di);
    dml = wave_sum(dml);
    li = wave_sum(li);
    la = wave_sum(la);
    if (lane == 0) {
      sh[0][wave] = di;
      sh[1][wave] = dml;
      sh[2][wave] = li;
      sh[3][wave] = la;
    }
    __syncthreads();
    if (wave == 0) {
      // the first tracer of the smallest sigma_k q_k, over the lanes: one
      // thread through 40 tracers took half of a single model's 31 us
      double smin = 1e300, dadi = 0.0;
      int at = K;
      for (int k = lane; k < K; k += 64) {
        const double sk = sqrt(0.5 / tab[k]), q = sqrt(tab[k] / tab[K + k]);
        if (sk * q < smin) {
          smin = sk * q;
          at = k;
          dadi = 0.25 * sk * dqdi(g.lum_q[k], q);
        }
      }
      for (int o = 32; o > 0; o >>= 1) {
        const double s = __shfl_xor(smin, o, 64), d = __shfl_xor(dadi, o, 64);
        const int k = __shfl_xor(at, o, 64);
        if (s < smin || (s == smin && k < at)) {
          smin = s;
          at = k;
          dadi = d;
        }
      }
      if (lane == 0) {
        double dis = 0.0, dmls = 0.0, lis = 0.0, las = 0.0;
        for (int w = 0; w < kW; ++w) {
          dis += sh[0][w];
          dmls += sh[1][w];
          lis += sh[2][w];
          las += sh[3][w];
        }
        if (out.inc) out.inc[m] = ok ? dis + lis + las * dadi : nan;
        if (out.mass_scale) out.mass_scale[m] = ok ? dmls : nan;
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Radial anisotropy profile sampled per tracer Gaussian (Sect. 6):
// beta_k = beta_0 + (beta_inf - beta_0) / (1 + (r_a / sigma_k)^alpha).
// Block per model, thread per Gaussian; an invalid profile (r_a or alpha not
// positive and finite) gives NaN, which the forward's set-up reports.
// ---------------------------------------------------------------------------
__device__ inline bool logistic_ok(const double *pf) {
  return pf[2] > 0.0 && pf[3] > 0.0 && isfinite(pf[2]) && isfinite(pf[3]) && isfinite(pf[0]) &&
         isfinite(pf[1]);
}

__global__ void __launch_bounds__(256) k_beta_logistic(const GeomDev *__restrict__ geoms,
                                                       const ModelDev *__restrict__ models, int n,
                                                       const double *__restrict__ prof,
                                                       double *__restrict__ beta) {
  for (int m = blockIdx.x; m < n; m += gridDim.x) {
    const ModelDev md = models[m];
    const GeomDev g = geoms[md.geom];
    const double *pf = prof + 4 * (int64_t)m;
    const bool ok = logistic_ok(pf);
    for (int k = threadIdx.x; k < g.K; k += blockDim.x) {
      const double x = pow(pf[2] / g.lum_sigma[k], pf[3]);
      beta[md.lum_off + k] = ok ? pf[0] + (pf[1] - pf[0]) / (1.0 + x) : __builtin_nan("");
    }
  }
}

// grad[m][0..3] = sum_k cot_k d beta_k / d (beta_0, beta_inf, r_a, alpha); the
// sum over k runs in a fixed order (thread strides, then the block sum).
__global__ void __launch_bounds__(256) k_beta_logistic_vjp(const GeomDev *__restrict__ geoms,
                                                           const ModelDev *__restrict__ models,
                                                           int n, const double *__restrict__ prof,
                                                           const double *__restrict__ cot,
                                                           double *__restrict__ grad) {
  __shared__ double sh[256];
  for (int m = blockIdx.x; m < n; m += gridDim.x) {
    const ModelDev md = models[m];
    const GeomDev g = geoms[md.geom];
    const double *pf = prof + 4 * (int64_t)m;
    const bool ok = logistic_ok(pf);
    const double d = pf[1] - pf[0];
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = threadIdx.x; k < g.K; k += blockDim.x) {
      const double lr = log(pf[2] / g.lum_sigma[k]);
      const double x = exp(pf[3] * lr), f = 1.0 / (1.0 + x);
      const double c = cot[md.lum_off + k];
      const double dfx = -f * f * x;                  // x df/dx
      a[0] += c * (1.0 - f);
      a[1] += c * f;
      a[2] += c * d * dfx * pf[3] / pf[2];
      a[3] += c * d * dfx * lr;
    }
    for (int i = 0; i < 4; ++i) {
      const double s = block_sum256(a[i], sh);
      if (threadIdx.x == 0) grad[4 * (int64_t)m + i] = ok ? s : __builtin_nan("");
      __syncthreads();
    }
  }
}

// Line-of-sight integral of the projected moment table into the unique-pixel
// N map.  Items (m, 64-pixel block), a contiguous range of them per block;
// the table is interpolated bicubically (sph_radial_weights,
// sph_angular_weights), the first radius standing for smaller ones and zero
// beyond the last.  FP64, whose issue and the 24 scattered LDS reads per node
// bound it.  Measured, 46,225 pixels: 256-thread blocks reading the table from
// global memory with library functions and all node quantities per pixel 119
// us, this 55.
__global__ void __launch_bounds__(kLosThreads) k_sph_num(const GeomDev *__restrict__ geoms,
                                                         const ModelDev *__restrict__ models,
                                                         const Item *__restrict__ items, int n_it,
                                                         const double *__restrict__ gauss,
                                                         const int *__restrict__ st_ws,
                                                         const double *__restrict__ table,
                                                         double *__restrict__ pix) {
  __shared__ double T[kSphNR * kLosCols * 3];
  __shared__ LosNode nodes[64];
  __shared__ LosMath mt;
  __shared__ LosModel lm;
  constexpr int kLosLanes = kLosThreads / 64, kLosNodes = kSphNodes / kLosLanes;
  const int pl = threadIdx.x / kLosLanes, h = threadIdx.x % kLosLanes;
  los_math_fill(mt);
  const int i0 = (int)((int64_t)n_it * blockIdx.x / gridDim.x);
  const int i1 = (int)((int64_t)n_it * (blockIdx.x + 1) / gridDim.x);
  int cur = -1;                              // the model whose table is loaded
  for (int ii = i0; ii < i1; ++ii) {
    const Item it = items[ii];
    const ModelDev md = models[it.m];
    const GeomDev &g = geoms[md.geom];
    const int q = it.a * 64 + pl;
    const bool on = q < g.n_pix;
    double *Nout = pix + md.pix_off + q;
    if (st_ws[it.m] != 0) {                  // uniform per block
      if (on && h == 0) *Nout = 0.0;
      continue;
    }
    if (it.m != cur) {
      __syncthreads();                       // the previous model's reads
      los_table(table + md.sph_off, T);
      if (threadIdx.x < 64) los_setup(g, gauss + md.gauss_off, nodes, lm);
      cur = it.m;
      __syncthreads();
    }
    const double x = on ? g.xs[q % g.n_ux] : 0.0, y = on ? g.ys[q / g.n_ux] : 0.0;
    const double si = lm.si, ci = lm.ci, idlnr = 1.0 / g.sph_dlnr;
    double acc = 0.0;
    for (int jn = 0; on && jn < kLosNodes; ++jn) {
      const LosNode nn = nodes[kLosLanes * jn + h];
      const LosPoint p = los_point(g, x, y, nn.zp, lm, idlnr, mt);
      if (p.xf > kSphNR - 1) continue;
      double ew[4], dew[4], tw[4], dtw[4];
      sph_radial_weights(p.xi, p.fx, ew, dew);
      sph_angular_weights(p.fy, tw, dtw);
      double A[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const int row = min(max(p.xi - 1 + a, 0), kSphNR - 1);   // out of range: zero weight
        const double *c = T + (row * kLosCols + p.yi) * 3;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
          double v = tw[0] * c[f];
#pragma unroll
          for (int b = 1; b < 4; ++b) v = fma(tw[b], c[3 * b + f], v);
          A[f] = fma(ew[a], v, A[f]);
        }
      }
      const double ct = p.Z * p.ir, st = fma(p.X, p.X, p.Y * p.Y) * p.iR * p.ir;
      const double sp = p.Y * p.iR, cp = p.X * p.iR;
      const double ner = si * st * sp + ci * ct, net = si * ct * sp - ci * st, nep = si * cp;
      acc += nn.wz * (ner * ner * A[0] + net * net * A[1] + nep * nep * A[2]);
    }
    // over the pixel's lanes, in every lane
#pragma unroll
    for (int o = 1; o < kLosLanes; o <<= 1) acc += __shfl_xor(acc, o, 64);
    if (on && h == 0) *Nout = acc;
  }
}

inline int grid_of(int n_it) { return n_it < 1 ? 1 : n_it; }

}  // namespace

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
void launch_setup(const GeomDev *g, const ModelDev *m, int n, ParamsDev p, double *gauss,
                  int *st_ws, int32_t *st_out, int *queues, hipStream_t st) {
  hipLaunchKernelGGL(k_setup, dim3(grid_of(n)), dim3(64), 0, st, g, m, n, p, gauss, st_ws, st_out,
                     queues);
}
void launch_prologue(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, ParamsDev p,
                     double *gauss, int *st_ws, int32_t *st_out, int *queues, float4 *terms,
                     double *pix, bool fused, hipStream_t st) {
  if (fused)
    hipLaunchKernelGGL(k_prologue<true>, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, p,
                       gauss, st_ws, st_out, queues, terms, pix);
  else
    hipLaunchKernelGGL(k_prologue<false>, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, p,
                       gauss, st_ws, st_out, queues, terms, pix);
}
void launch_sb(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, ParamsDev p,
               double *pix, hipStream_t st) {
  hipLaunchKernelGGL(k_sb, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, p, pix);
}
void launch_num(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                const float4 *terms, const double *gauss, const int *st_ws, double *part, double *pix,
                int *queue, int grid, bool mfma, hipStream_t st) {
  if (mfma)
    hipLaunchKernelGGL(k_num_mfma, dim3(grid_of(grid)), dim3(256), 0, st, g, m, it, n_it, terms,
                       gauss, st_ws, part, pix, queue);
  else
    hipLaunchKernelGGL(k_num_pix, dim3(grid_of(grid)), dim3(256), 0, st, g, m, it, n_it, terms,
                       st_ws, part, queue);
}
template <int TX, int TY, bool kTab>
static void small_kernel(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                         const float4 *terms, const double *gauss, const int *st_ws, double *part,
                         double *pix, hipStream_t st) {
  hipLaunchKernelGGL((k_num_small<TX, TY, kTab>), dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it,
                     n_it, terms, gauss, st_ws, part, pix);
}
void launch_num_small(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, int tiling,
                      const float4 *terms, const double *gauss, const int *st_ws, double *part,
                      double *pix, hipStream_t st) {
  switch (tiling) {
#define JAM_TILING(n, tx, ty)                                                             \
  case n: small_kernel<tx, ty, false>(g, m, it, n_it, terms, gauss, st_ws, part, pix, st); break; \
  case 9 + n: small_kernel<tx, ty, true>(g, m, it, n_it, terms, gauss, st_ws, part, pix, st); break;
    JAM_TILING(0, 3, 3)
    JAM_TILING(1, 3, 5)
    JAM_TILING(2, 3, 6)
    JAM_TILING(3, 5, 3)
    JAM_TILING(4, 5, 5)
    JAM_TILING(5, 5, 6)
    JAM_TILING(6, 6, 3)
    JAM_TILING(7, 6, 5)
    JAM_TILING(8, 6, 6)
#undef JAM_TILING
  }
}
void launch_reduce(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                   const double *part, double *pix, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, part, pix);
}
void launch_bins(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, int n_wave,
                 const double *pix, const int *st_ws, double *vrms2, double *binws,
                 hipStream_t st) {
  if (n_wave > 0)
    hipLaunchKernelGGL(k_bins<256>, dim3(n_wave), dim3(256), 0, st, g, m, it, n_wave, pix,
                       st_ws, vrms2, binws);
  if (n_it > n_wave)
    hipLaunchKernelGGL(k_bins<1024>, dim3(n_it - n_wave), dim3(1024), 0, st, g, m, it + n_wave,
                       n_it - n_wave, pix, st_ws, vrms2, binws);
}
void launch_maps(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                 const double *pix, const int *st_ws, double *N_map, double *I_map,
                 hipStream_t st) {
  hipLaunchKernelGGL(k_maps, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, pix, st_ws,
                     N_map, I_map);
}
void launch_bins_adjoint(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                         const double *vrms2, const double *cot, const double *binws,
                         const int *st_ws, double *pix, hipStream_t st) {
  hipLaunchKernelGGL(k_bins_adjoint, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, vrms2,
                     cot, binws, st_ws, pix);
}
void launch_sens(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                 const float4 *terms, const double *pix, const int *st_ws, double *sens,
                 int *queue, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_sens, dim3(grid_of(grid)), dim3(256), 0, st, g, m, it, n_it, terms, pix,
                     st_ws, sens, queue);
}
void launch_sens_wide(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                      const float4 *terms, const double *pix, const int *st_ws, double *sens,
                      int *queue, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_sens_wide, dim3(grid_of(grid)), dim3(64 * kWideWaves), 0, st, g, m, it,
                     n_it, terms, pix, st_ws, sens, queue);
}
int occupancy_num(bool mfma) {
  int nb = 0;
  const hipError_t e = mfma ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_num_mfma, 256, 0)
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_num_pix, 256, 0);
  if (e != hipSuccess) nb = 1;
  return nb < 1 ? 1 : nb;
}
int occupancy_sens() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_sens, 256, 0) != hipSuccess) nb = 1;
  return nb < 1 ? 1 : nb;
}
template <int NYQ>
static void adj_small_kernel(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                             ParamsDev p, const double *pix, const int *st_ws, double *sens,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_adj_small<NYQ>, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, p,
                     pix, st_ws, sens);
}
void launch_adj_small(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, int y_quads,
                      ParamsDev p, const double *pix, const int *st_ws, double *sens,
                      hipStream_t st) {
  switch (y_quads) {
    case 1: adj_small_kernel<1>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
    case 2: adj_small_kernel<2>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
    case 3: adj_small_kernel<3>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
    case 4: adj_small_kernel<4>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
    case 5: adj_small_kernel<5>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
    case 6: adj_small_kernel<6>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
    case 7: adj_small_kernel<7>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
    default: adj_small_kernel<8>(g, m, it, n_it, p, pix, st_ws, sens, st); break;
  }
}
void launch_chain(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, ParamsDev p,
                  double *sens, const int *st_ws, hipStream_t st) {
  hipLaunchKernelGGL(k_chain, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, p, sens, st_ws);
}
constexpr int kGradsWide = 256;   // models
void launch_grads(const GeomDev *g, const ModelDev *m, int n, ParamsDev p, double *sens,
                  const double *sbp, const int *st_ws, GradsDev out, hipStream_t st) {
  // Sixteen waves a model for its latency while there is a CU for each; beyond
  // that four, most of sixteen waiting for the one with the longest rows.  16 / 4
  // waves: 512 models of 21 Gaussians 16.8 / 15.4 us, 1024 of 10 24.4 / 13.4, 3476
  // of 9 86 / 41, 1024 of 5 to 60 55 / 45.
  if (n > kGradsWide)
    hipLaunchKernelGGL(k_grads<4>, dim3(grid_of(n)), dim3(256), 0, st, g, m, n, p, sens, sbp, st_ws,
                     out);
  else
    hipLaunchKernelGGL(k_grads<16>, dim3(grid_of(n)), dim3(1024), 0, st, g, m, n, p, sens, sbp, st_ws,
                     out);
}
void launch_sb_adjoint(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                       const int *st_ws, const double *pix, double *sbp, hipStream_t st) {
  hipLaunchKernelGGL(k_sb_adj, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, st_ws, pix,
                     sbp);
}
void launch_sph_terms(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                      const double *gauss, const int *st_ws, float4 *terms, double *terms64,
                      double *pol, hipStream_t st) {
  hipLaunchKernelGGL(k_sph_terms, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, gauss,
                     st_ws, terms, terms64, pol);
}
void launch_sph_moments(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                        const double *gauss, const float4 *terms, const int *st_ws, double *table,
                        hipStream_t st) {
  hipLaunchKernelGGL(k_sph_moments, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, gauss,
                     terms, st_ws, table);
}
void launch_sph_moments_jac(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                            const double *gauss, const float4 *terms, const int *st_ws,
                            double *table, double *sens, hipStream_t st) {
  hipLaunchKernelGGL(k_sph_moments_jac, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it,
                     gauss, terms, st_ws, table, sens);
}
void launch_sph_num(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                    const double *gauss, const int *st_ws, const double *table, double *pix,
                    hipStream_t st) {
  hipLaunchKernelGGL(k_sph_num, dim3(grid_of(std::min(n_it, kLosBlocks))), dim3(kLosThreads), 0, st, g, m, it, n_it,
                     gauss, st_ws, table, pix);
}
void launch_sph_adjoint(const GeomDev *g, const ModelDev *m, int n, const Item *it_los, int n_los,
                        const Item *it_cell, int n_cell, const double *gauss, const int *st_ws,
                        const double *table, const double *pix, double *sens, hipStream_t st) {
  hipLaunchKernelGGL(k_sph_zero, dim3(grid_of(std::min(n, 65536) * kZeroParts)), dim3(256), 0, st,
                     g, m, n, st_ws, pix, sens);
  hipLaunchKernelGGL(k_sph_num_adj, dim3(grid_of(std::min(n_los, kLosBlocks))), dim3(kLosAdjThreads), 0, st, g, m, it_los, n_los,
                     gauss, st_ws, table, pix, sens);
  hipLaunchKernelGGL(k_sph_dtab_fix, dim3(grid_of(std::min(n, 65536) * kFixParts)), dim3(256), 0, st, g, m, n, st_ws, sens);
  hipLaunchKernelGGL(k_sph_rows, dim3(grid_of(n_cell)), dim3(256), 0, st, g, m, it_cell, n_cell,
                     gauss, st_ws, sens);
}
void launch_sph_sens(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                     const double *gauss, const float4 *terms, const int *st_ws, double *sens,
                     hipStream_t st) {
  hipLaunchKernelGGL(k_sph_sens, dim3(grid_of(n_it)), dim3(256), 0, st, g, m, it, n_it, gauss,
                     terms, st_ws, sens);
}
void launch_sph_chain(const GeomDev *g, const ModelDev *m, int n, const Item *it_tile, int n_tile,
                      ParamsDev p, const double *gauss, const double *terms64, const int *st_ws,
                      const double *sbp, double *sens, GradsDev out, hipStream_t st) {
  hipLaunchKernelGGL(k_sph_sens_cells, dim3(grid_of(n_tile * kSphCellParts)), dim3(256), 0, st, g,
                     m, it_tile, n_tile, gauss, terms64, st_ws, sens);
  hipLaunchKernelGGL(k_sph_chain, dim3(grid_of(n_tile)), dim3(256), 0, st, g, m, it_tile, n_tile,
                     gauss, st_ws, sens);
  hipLaunchKernelGGL(k_sph_grads, dim3(grid_of(n)), dim3(512), 0, st, g, m, n, p, gauss, st_ws,
                     sens, sbp, out);
}
void launch_beta_logistic(const GeomDev *g, const ModelDev *m, int n, const double *prof,
                          double *beta, hipStream_t st) {
  hipLaunchKernelGGL(k_beta_logistic, dim3(grid_of(n)), dim3(256), 0, st, g, m, n, prof, beta);
}
void launch_beta_logistic_vjp(const GeomDev *g, const ModelDev *m, int n, const double *prof,
                              const double *cot, double *grad, hipStream_t st) {
  hipLaunchKernelGGL(k_beta_logistic_vjp, dim3(grid_of(n)), dim3(256), 0, st, g, m, n, prof, cot,
                     grad);
}
void launch_mge1d(int n_prof, int n_comp, const double *comp, const MgeConst &k, double *amp,
                  hipStream_t st) {
  const int64_t n = (int64_t)n_prof * k.n_sigma;
  hipLaunchKernelGGL(k_mge1d, dim3((unsigned)std::min<int64_t>((n + 7) / 8, kMgeBlocks)), dim3(256), 0, st, n_prof, n_comp,
                     comp, k, amp);
}
void launch_mge1d_vjp(int n_prof, int n_comp, const double *comp, const MgeConst &k,
                      const double *cot, double *grad, hipStream_t st) {
  const int64_t n = (int64_t)n_prof * n_comp;
  hipLaunchKernelGGL(k_mge1d_vjp, dim3((unsigned)std::min<int64_t>((n + 3) / 4, kMgeBlocks)), dim3(256), 0, st, n_prof,
                     n_comp, comp, k, cot, grad);
}
void launch_chi2(const GeomDev *g, const ModelDev *m, int n, const KinDev *kin, const double *V,
                 const int *st_ws, double *chi2, const double *cot, double *dV, hipStream_t st) {
  hipLaunchKernelGGL(k_chi2, dim3(grid_of(std::min(n, 65536))), dim3(256), 0, st, g, m, n, kin, V,
                     st_ws, chi2, cot, dV);
}

}  // namespace jam
