// gfx950 kernels of the compressed cylindrical form (ModelDev::form 5), FP64.
//
// For one tracer k the sky numerator is a sum over the (j, n) terms of
//   E_k(x) G_k(y) exp(-v x^2 - d y^2) (C0 + C1 x^2),
//   E_k = exp(-alpha x^2), G_k = exp(-gamma0 y^2),  v = r u^2 >= 0,  d = gamma - gamma0 >= v,
// with gamma0 = alpha alphaq / (alpha sin^2 i + alphaq cos^2 i) the tracer's
// own projected exponent.  exp(-v x^2) is a smooth function of v alone, and
// exp(-d y^2) of d alone, so both are interpolated: v runs over panels (the
// first [0, 1 / M2), M2 the largest squared coordinate of the map, linear in
// v; the others a factor kChebR wide, in log v) with kChebP Chebyshev nodes
// each, d over the range that the panel's terms reach, with 16 nodes per
// decade or less.  A panel's terms, however many, then act on the map as
// kChebP x 16 node weights (per decade of d)
//   W_b[m][l] = sum_t C_b l_m(v_t) l_l(d_t)        (b = 0, 1),
// and N = sum_k E_k sum_(panel, m) e^(-v_m x^2) (H_0m(y) + x^2 H_1m(y)) with
// H_bm(y) = G_k(y) sum_l W_b[m][l] e^(-d_l y^2).  The interpolants converge
// geometrically (the functions are bounded for |Im log v| < pi / 2): the map's
// relative error is about 1e-10 where N does not change sign, two orders under
// the FP32 sums of the direct forms.  The tracer factor stays outside, so
// far-out pixels keep their relative accuracy.
//
// Why: the direct sum costs n_pix multiply-adds per term (46,225 on a 215 x
// 215 map); here a term costs 2 x 8 x 16 and the map a contraction over the
// nodes, of which about half reach the average pixel.  Measured, IFU-scale
// model (40 x 41 x 128 terms, 215 x 215 distinct pixels), FP32 direct sums
// before and this after: forward 233 -> 79 us, forward + adjoint 626 -> 225
// us; 135 x 101 distinct pixels, 42 x 96 x 128 terms: maps 228 -> 69 us.
//
// v is the same for every tracer and every proposal, so the terms sorted by
// panel, their Chebyshev variable, the node exponentials e^(-v_m x^2) and the
// tracer factors are tables of the geometry.
#include "jam_device.h"
#include "jam_internal.h"

#include <hip/hip_runtime.h>
#include <algorithm>

namespace jam {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4 (lane l): A[l % 16][l / 16], B[l / 16][l % 16],
// D register r = D[4 r + l / 16][l % 16].
__device__ __forceinline__ v4d mfma64(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4d zero4() { return v4d{0.0, 0.0, 0.0, 0.0}; }

// Orders a wave's own LDS writes before its later reads by other lanes (LDS
// operations of a wave execute in order; this keeps the compiler to it).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave stages 32 terms at a time: rows of 34 doubles (lanes of a 16-row
// operand read then fall on 16 different bank pairs).
constexpr int kStage = 34;
constexpr int kWaveLds = 32 * kStage;   // doubles of staging per wave

// cos(n pi / 32) at compile time.
constexpr double cos32(int n) {
  n %= 64;
  if (n > 32) n = 64 - n;
  const double sign = n > 16 ? -1.0 : 1.0;
  const double x = (n > 16 ? 32 - n : n) * (kPi / 32.0);
  double t = 1.0, s = 1.0;
  for (int k = 1; k < 14; ++k) {
    t *= -x * x / ((2 * k - 1) * (2 * k));
    s += t;
  }
  return sign * s;
}
// From Chebyshev moments to node weights, l_m = sum_i D[m][i] T_i, for 16
// nodes (d16) and, block-diagonal over b, for kChebP = 8 (dblk).
struct NodeTables {
  double dblk[16][16], d16[16][16];
};
constexpr NodeTables make_tables() {
  NodeTables t{};
  for (int m = 0; m < 16; ++m)
    for (int i = 0; i < 16; ++i) {
      t.d16[m][i] = (i ? 2.0 : 1.0) / 16.0 * cos32(i * (2 * m + 1));
      t.dblk[m][i] = m / 8 == i / 8 ? (i % 8 ? 2.0 : 1.0) / 8.0 * cos32(2 * (i % 8) * (2 * (m % 8) + 1))
                                    : 0.0;
    }
  return t;
}
static_assert(kChebP == 8, "dblk and the (b, i) rows are laid out for 8 nodes");
__device__ const NodeTables kTab = make_tables();

// What a (model, tracer, panel) unit needs of the set-up, and its range of d
// in n_sub equal stretches of the interpolation variable z = (lin ? d : log
// d) scale + shift in [0, n_sub], with 16 nodes each.  On the linear panel z
// goes on as kLinMax + kLogTail log(d scale / kLinMax) past kLinMax: half a
// decade of d per stretch.
constexpr int kLinMax = 8;
constexpr double kLogTail = 2.0 / 2.302585092994046;
struct Unit {
  const double *mt;                     // mass part of the Gaussian table
  double alpha, aq, nu0, b, si2, ci2, ra0, gam0;
  double dmin, scale, shift;
  int n_sub;
  bool lin;
};

// One term's d without the cancellation of gamma - gamma0, from r u^2 and
// 1 / h; also c1, A and 1 / a of the direct forms.
__device__ __forceinline__ double term_d(const Unit &c, double ru2, double rh, double &c1, double &A,
                                         double &ra) {
  c1 = c.alpha + ru2;
  A = fma(ru2, rh, c.aq);
  ra = rcp64(fma(c1, c.si2, A * c.ci2));
  return ru2 * (c.si2 * rh * c1 * c.alpha + c.ci2 * c.aq * A) * ra * c.ra0;
}

// Set-up of a unit by one wave.  The range of d over the panel's terms: d
// grows with u at fixed j, so the ends of each j's stretch inside the panel
// bound it.  Stretches: a decade of d (the panel spans kChebR times the
// largest 1 / h), or on the linear panel 12 units of the exponent d y^2 at the
// map's largest y up to kLinMax of them, then half-decades: a thin mass Gaussian
// near edge-on has 1 / h up to 1 / (1 - u_max^2), 4e5 at n_u = 1024, which would
// take thousands of equal stretches.  FP64 replays of one tracer with 13 mass
// Gaussians edge-on, 2-norm of the map's error: q' = 0.01, 0.005 (n_u = 160) and
// 0.001 (n_u = 1024) 2e-11, 3e-11 and 1.4e-11, the same as with equal stretches of
// 12, of which these take 361, 558 and 20,384.
__device__ __forceinline__ void unit_setup(const GeomDev &g, const double *__restrict__ tab, int k,
                                           int P, Unit &c) {
  const int K = g.K, J1 = g.J1;
  c.mt = tab + 4 * K;
  c.alpha = tab[k];
  c.aq = tab[K + k];
  c.nu0 = tab[2 * K + k];
  c.b = tab[3 * K + k];
  c.si2 = c.mt[3 * J1];
  c.ci2 = c.mt[3 * J1 + 1];
  c.ra0 = rcp64(fma(c.alpha, c.si2, c.aq * c.ci2));
  c.gam0 = c.alpha * c.aq * c.ra0;
  const double lo = g.cheb_lo[P], hi = g.cheb_lo[g.cheb_np + P];
  c.lin = lo == 0.0;
  const double u0 = g.u[0] * g.u[0], u1 = g.u[g.n_u - 1] * g.u[g.n_u - 1];
  double dmin = 1e300, dmax = 0.0;
  for (int j = threadIdx.x & 63; j < J1; j += 64) {
    const double r = c.mt[j], e2 = c.mt[J1 + j], rr = rcp64(r);
    const double ua = fmax(u0, lo * rr), ub = fmin(u1, hi * rr);
    if (ua <= ub * (1.0 + 1e-12)) {
      double c1, A, ra;
      dmin = fmin(dmin, term_d(c, r * ua, rcp64(fma(-e2, ua, 1.0)), c1, A, ra));
      dmax = fmax(dmax, term_d(c, r * ub, rcp64(fma(-e2, ub, 1.0)), c1, A, ra));
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    dmin = fmin(dmin, __shfl_xor(dmin, o, 64));
    dmax = fmax(dmax, __shfl_xor(dmax, o, 64));
  }
  // a little wider than the terms, and never empty
  dmax = fmax(dmax * (1.0 + 1e-6), 1e-280);
  c.dmin = c.lin ? 0.0 : fmin(fmax(dmin * (1.0 - 1e-6), 1e-290), dmax * (1.0 - 1e-6));
  const double ym = g.ys[g.n_uy - 1];
  const double l0 = c.lin ? 0.0 : log64(c.dmin);
  const double span = c.lin ? dmax : log64(dmax) - l0;
  const double want = c.lin ? dmax * ym * ym * (1.0 / 12.0) : span * (1.0 / 2.302585092994046);
  // (a decade of d per stretch: far fewer than 64 of them, 1 / h being bounded)
  c.n_sub = want <= 1.0 ? 1 : (want < 63.0 ? (int)want + 1 : (want >= 63.0 ? 64 : 1));
  c.scale = c.n_sub / span;
  if (c.lin && want > kLinMax) {
    c.n_sub = kLinMax + min(56, 1 + (int)(kLogTail * log64(want * (1.0 / kLinMax))));
    c.scale = want / span;
  }
  c.n_sub = __builtin_amdgcn_readfirstlane(c.n_sub);
  c.shift = -l0 * c.scale;
}

// Stretch of a term's d and Chebyshev variable in stretch `sub`.
__device__ __forceinline__ double z_of(const Unit &c, double d) {
  double z = fma(c.lin ? d : log64(d), c.scale, c.shift);
  if (c.lin && c.n_sub > kLinMax)
    z = z > kLinMax ? fma(kLogTail, log64(z * (1.0 / kLinMax)), kLinMax) : z;
  return fmin((double)c.n_sub, fmax(0.0, z));
}
__device__ __forceinline__ int sub_of(const Unit &c, double z) {
  return min(c.n_sub - 1, (int)z);
}
// d at node l (of 16) of a stretch.
__device__ __forceinline__ double node_d(const Unit &c, int sub, int l) {
  double z = sub + 0.5 + 4.0 * kTab.d16[l][1];                     // cos = 8 d16[l][1]
  if (c.lin && sub >= kLinMax) z = kLinMax * exp((z - kLinMax) * (1.0 / kLogTail));
  z /= c.scale;
  return c.lin ? z : c.dmin * exp(z);
}

// Coefficients of the term at position e of the panel-sorted list; returns z.
__device__ __forceinline__ double load_term(const GeomDev &g, const Unit &c, int e, double &C0,
                                            double &C1) {
  const int id = g.cheb_id[e], j = id >> 10, n = id & 1023;
  const double r = c.mt[j], e2 = c.mt[g.J1 + j], Kp = c.mt[2 * g.J1 + j];
  const double u = g.u[n], u2 = u * u, ru2 = r * u2;
  const double h = fma(-e2, u2, 1.0);
  const double rh = rcp64(h), rsh = rsq64(h);
  double c1, A, ra;
  const double d = term_d(c, ru2, rh, c1, A, ra);
  const double base = c.nu0 * Kp * ru2;
  const double gg = base * rcp64(A) * rh * rsh;
  const double ww = 2.0 * base * rsh;
  const double f = g.w[n] * kSqrtPi * (ra * rsq64(ra));      // sqrt(pi / a)
  C0 = f * ((c.ci2 + c.b * c.si2) * gg);
  C1 = f * (c.si2 * (ww - 2.0 * c1 * c.b * gg));
  return z_of(c, d);
}

// T_0 .. T_{N-1} of x into rows of the staging, column col.
template <int N>
__device__ __forceinline__ void put_chebyshev(double *A, int col, double x) {
  double p0 = 1.0, p1 = x;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    A[i * kStage + col] = p0;
    const double p2 = fma(2.0 * x, p1, -p0);
    p0 = p1;
    p1 = p2;
  }
}

// Sum of the kW waves' registers v in wave order, left in every wave (block
// call; `sh` holds kW x 256 doubles).
template <int kW>
__device__ __forceinline__ v4d sum_waves(v4d v, double *sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) sh[wave * 256 + r * 64 + lane] = v[r];
  __syncthreads();
  v4d o;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    double a = sh[r * 64 + lane];
#pragma unroll
    for (int w = 1; w < kW; ++w) a += sh[w * 256 + r * 64 + lane];
    o[r] = a;
  }
  return o;
}

// One unit of the forward, stretch by stretch of d.  The node weights' moments
// W, both b at once (the 16 rows are (b, i)), by matrix cores: lane = term
// forms the coefficients of 64 terms; 32 at a time write C_b T_i(xi) and
// T_j(eta) to LDS, and 8 steps of four terms contract them.  Then H on the y
// tiles that the unit reaches.  The register layouts chain (a product's D
// registers are the next one's B operand, and the A operand of its
// transpose), so moments -> weights needs no LDS:
//   V^T = W^T Dblk^T,  U^T = D16 V^T,  H = U F.
// kShare: the block's kW waves share the unit; otherwise each has its own.
template <bool kShare, int kW>
__device__ __forceinline__ void unit_forward(const GeomDev &g, const Unit &c, int P, int n_yt,
                                             double *A, double *sh, double *__restrict__ out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c16 = lane & 15, kk = lane >> 4;
  const int l32 = lane & 31, w0 = kShare ? wave : 0, nw = kShare ? kW : 1;
  double *B = A + 16 * kStage;
  const int e0 = g.cheb_ptr[P], e1 = g.cheb_ptr[P + 1];
  const int ar = c16 * kStage + kk;
  for (int sub = 0; sub < c.n_sub; ++sub) {
    v4d w = zero4();
    for (int base = e0 + w0 * 64; base < e1; base += 64 * nw) {
      const int e = base + lane;
      double C0 = 0.0, C1 = 0.0, xi = 0.0, z = -1.0;
      if (e < e1) {
        z = load_term(g, c, e, C0, C1);
        xi = g.cheb_xi[e];
      }
      const bool in = z >= 0.0 && sub_of(c, z) == sub;
      const uint64_t active = __ballot(in);
      const double eta = fma(2.0, z - sub, -1.0);
      C0 = in ? C0 : 0.0;
      C1 = in ? C1 : 0.0;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (((active >> (32 * half)) & 0xffffffffu) == 0) continue;   // uniform
        if ((lane >> 5) == half) {
          double p0 = 1.0, p1 = xi;
#pragma unroll
          for (int i = 0; i < kChebP; ++i) {
            A[i * kStage + l32] = C0 * p0;
            A[(kChebP + i) * kStage + l32] = C1 * p0;
            const double p2 = fma(2.0 * xi, p1, -p0);
            p0 = p1;
            p1 = p2;
          }
          put_chebyshev<16>(B, l32, in ? eta : 0.0);
        }
        wave_sync();
#pragma unroll
        for (int s = 0; s < 8; ++s) w = mfma64(A[ar + 4 * s], B[ar + 4 * s], w);
        wave_sync();
      }
    }
    if (kShare) w = sum_waves<kW>(w, sh);
    v4d vt = zero4(), ut = zero4();
#pragma unroll
    for (int s = 0; s < 4; ++s) vt = mfma64(w[s], kTab.dblk[c16][4 * s + kk], vt);
#pragma unroll
    for (int s = 0; s < 4; ++s) ut = mfma64(kTab.d16[c16][4 * s + kk], vt[s], ut);
    double ex[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) ex[s] = -(c.gam0 + node_d(c, sub, 4 * s + kk));
    for (int yt = w0; yt < 2 * n_yt; yt += nw) {
      const int y = 16 * yt + c16;
      const bool vy = y < g.n_uy;
      const double yv = vy ? g.ys[y] : 0.0, y2 = yv * yv;
      double *o = out + (int64_t)(yt >> 1) * 512 + (yt & 1) * 16 + c16;
      v4d h = zero4();
      if (sub > 0)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = o[(4 * r + kk) * 32];
#pragma unroll
      for (int s = 0; s < 4; ++s) h = mfma64(ut[s], vy ? exp(ex[s] * y2) : 0.0, h);
#pragma unroll
      for (int r = 0; r < 4; ++r) o[(4 * r + kk) * 32] = h[r];
    }
    if (kShare && sub + 1 < c.n_sub) __syncthreads();   // the sums' LDS is staging again
  }
}

// Unit of this wave: blocks below n_share take one item of the list with all
// kW waves, the others kW items each, a wave per item.  False past the end
// (uniform per wave; per block where shared).
template <int kW>
__device__ __forceinline__ bool unit_of(const Item *__restrict__ items, int n_it, int n_share,
                                        int blk, Item &it) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blk < n_share ? blk : n_share + kW * (blk - n_share) + wave;
  if (i >= n_it) return false;
  it = items[i];
  return true;
}

// Items (m, k, panel), the first n_share shared by a block's waves: H of the
// unit on the y tiles it reaches, blocks of [16 rows (b, m)][32 y] doubles.
template <bool kShare, int kW>
__device__ __forceinline__ void panel_item(const Item &it, const GeomDev *__restrict__ geoms,
                                           const ModelDev *__restrict__ models,
                                           const double *__restrict__ gauss,
                                           const int *__restrict__ st_ws, double *__restrict__ H,
                                           double *A, double *sh) {
  const ModelDev md = models[it.m];
  const GeomDev g = geoms[md.geom];
  if (st_ws[it.m] != 0) return;          // uniform per block where shared
  Unit c;
  unit_setup(g, gauss + md.gauss_off, it.a, it.b, c);
  const int u = it.a * g.cheb_np + it.b;
  const int h0 = g.cheb_h[u], nyt = g.cheb_h[u + 1] - h0;
  unit_forward<kShare, kW>(g, c, it.b, nyt, A, sh, H + md.cheb_off + (int64_t)h0 * 512);
}

template <int kW>
__global__ void __launch_bounds__(64 * kW, kW == 4 ? 3 : 2)
    k_cheb_panel(const GeomDev *__restrict__ geoms, const ModelDev *__restrict__ models,
                 const Item *__restrict__ items, int n_it, int n_share,
                 const double *__restrict__ gauss, const int *__restrict__ st_ws,
                 double *__restrict__ H) {
  __shared__ __attribute__((aligned(16))) double L[kW * kWaveLds];
  double *A = L + (threadIdx.x >> 6) * kWaveLds;
  Item it;
  if (!unit_of<kW>(items, n_it, n_share, blockIdx.x, it)) return;
  if ((int)blockIdx.x < n_share)
    panel_item<true, kW>(it, geoms, models, gauss, st_ws, H, A, L);
  else
    panel_item<false, kW>(it, geoms, models, gauss, st_ws, H, A, L);
}

// ---------------------------------------------------------------------------
// Map contraction: a 32 x 32 tile of N over a run of units, four waves each
// taking a quarter of the run (their tiles are added through LDS in wave
// order).  Per unit a wave reads its rows of the node exponentials (4
// doubles a lane) and the H block (8), multiplies the tracer factor on, and
// runs 16 MFMAs.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_cheb_map(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const ChebItem *__restrict__ items, int n_it,
                                                  const double *__restrict__ H,
                                                  const int *__restrict__ st_ws,
                                                  double *__restrict__ part) {
  __shared__ double red[3][1024];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, kk = lane >> 4;
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const ChebItem it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;      // uniform per block
    const int tx = it.tile % md.n_xt, ty = it.tile / md.n_xt;
    const int ldx = 32 * md.n_xt, np = g.cheb_np;
    const unsigned char *px = g.cheb_px + tx, *py = g.cheb_py + ty;
    const double *Hm = H + md.cheb_off + (int64_t)ty * 512 + kk * 32 + c16;
    const double *Em = g.cheb_E + (int64_t)kk * ldx + 32 * tx + c16;
    const double *Ek = g.cheb_Ek + 32 * tx + c16;
    double x2[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int x = 32 * tx + 16 * r + c16;
      const double v = x < g.n_ux ? g.xs[x] : 0.0;
      x2[r] = v * v;
    }
    // this wave's quarter of the run
    const int q = (it.count + 3) >> 2;
    int left = min(q, it.count - wave * q), skip = min(it.count, wave * q);
    int k = it.k0, P = it.p0;
    int pk = min((int)px[k * md.n_xt], (int)py[k * md.n_yt]);
    while (left > 0 && skip >= pk - P) {
      skip -= pk - P;
      P = 0;
      ++k;
      pk = k < g.K ? min((int)px[k * md.n_xt], (int)py[k * md.n_yt]) : 0x7fffffff;
    }
    P += skip;
    v4d acc[2][2];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int s = 0; s < 2; ++s) acc[r][s] = v4d{0.0, 0.0, 0.0, 0.0};
    while (left > 0) {
      const double ek0 = Ek[(int64_t)k * ldx], ek1 = Ek[(int64_t)k * ldx + 16];
      const int run = min(left, pk - P);
      for (int e = 0; e < run; ++e, ++P) {
        const double *h = Hm + (int64_t)g.cheb_h[k * np + P] * 512;
        const double *em = Em + (int64_t)(P * 2 * kChebP) * ldx;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          double a[2], b0[2], b1[2];
          a[0] = em[(int64_t)(4 * s) * ldx] * ek0;
          a[1] = em[(int64_t)(4 * s) * ldx + 16] * ek1;
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) {
            b0[cb] = h[(4 * s) * 32 + 16 * cb];
            b1[cb] = h[(kChebP + 4 * s) * 32 + 16 * cb];
          }
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[r][cb] = mfma64(b0[cb], a[r], acc[r][cb]);
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[r][cb] = mfma64(b1[cb], a[r] * x2[r], acc[r][cb]);
        }
      }
      left -= run;
      P = 0;
      ++k;
      pk = k < g.K ? min((int)px[k * md.n_xt], (int)py[k * md.n_yt]) : 0x7fffffff;
    }
    __syncthreads();                     // the previous item's sums are read
    if (wave > 0) {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int w = 0; w < 4; ++w) red[wave - 1][((r * 2 + cb) * 4 + w) * 64 + lane] = acc[r][cb][w];
    }
    __syncthreads();
    if (wave == 0) {
      // tile in [y][x] order
      double *o = part + md.part_off + (int64_t)it.slot * 1024;
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int e = ((r * 2 + cb) * 4 + w) * 64 + lane;
            o[(16 * cb + 4 * w + kk) * 32 + 16 * r + c16] =
                ((acc[r][cb][w] + red[0][e]) + red[1][e]) + red[2][e];
          }
    }
  }
}

// Items (m, tile * 4 + quarter, first slot, slots): N of eight rows of a
// tile as the sum of its slots in order (part NULL: not wanted), and the
// surface brightness I = sum_k I0_k E_k(x) G_k(y) from the tracer tables.
__global__ void __launch_bounds__(256) k_cheb_sum(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  ParamsDev p, const double *__restrict__ part,
                                                  double *__restrict__ pix) {
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    const int tile = it.a >> 2, xl = threadIdx.x & 31, yl = 8 * (it.a & 3) + (threadIdx.x >> 5);
    const int x = 32 * (tile % md.n_xt) + xl, y = 32 * (tile / md.n_xt) + yl;
    if (x >= g.n_ux || y >= g.n_uy) continue;
    const int64_t o = md.pix_off + (int64_t)y * g.n_ux + x;
    if (part) {
      const double *s = part + md.part_off + (int64_t)it.b * 1024 + yl * 32 + xl;
      double acc = 0.0;
      int q = 0;
      for (; q + 8 <= it.c; q += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = s[(int64_t)(q + u) * 1024];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += v[u];
      }
      for (; q < it.c; ++q) acc += s[(int64_t)q * 1024];
      pix[o] = acc;
    }
    const double *I0 = p.lum_I0 ? p.lum_I0 + md.lum_off : g.lum_I0;
    const double *ek = g.cheb_Ek + x, *gk = g.cheb_Gk + y;
    const int ldx = 32 * md.n_xt, ldy = 32 * md.n_yt;
    double acc = 0.0;
#pragma unroll 4
    for (int k = 0; k < g.K; ++k)
      acc = fma(I0[k] * ek[(int64_t)k * ldx], gk[(int64_t)k * ldy], acc);
    pix[o + g.n_pix] = acc;
  }
}

// ---------------------------------------------------------------------------
// Adjoint.  Per unit and y, T_b,m(y) = sum_x x^2b e^(-v_m x^2) E_k lambda_N
// (k_cheb_tmap); then the node sensitivities of W and of its y^2-weighted twin
//   S_b[m][l] = sum_y T F_l,  Sy_b[m][l] = sum_y y^2 T F_l,
// taken to Chebyshev coefficients, per term the four interpolants S0, S1 (of
// C0, C1) and Sy0, Sy1, with dL/dgamma = -(C0 Sy0 + C1 Sy1), and at once the
// chain to the set-up (k_cheb_adj); the terms' chain values are summed over
// runs of equal j within a chunk of 64 (pieces), and the pieces into the chain
// rows (k_cheb_rows).
// ---------------------------------------------------------------------------

// Items (m, tile row, k): T of tracer k's units on 32 map rows, a wave per
// panel, lambda E_k of the rows staged in LDS kTx columns at a time.  T blocks
// are [32 y][16 rows (b, m)], at the unit's H position.
constexpr int kTx = 256;
__global__ void __launch_bounds__(256) k_cheb_tmap(const GeomDev *__restrict__ geoms,
                                                   const ModelDev *__restrict__ models,
                                                   const Item *__restrict__ items, int n_it,
                                                   const double *__restrict__ pix,
                                                   const int *__restrict__ st_ws,
                                                   double *__restrict__ T) {
  __shared__ __attribute__((aligned(16))) double lam[32][kTx + 2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15, kk = lane >> 4;
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;      // uniform per block
    const int ty = it.a, k = it.b, np = g.cheb_np, ldx = 32 * md.n_xt;
    const double *lm = pix + md.pix_off + 2 * (int64_t)g.n_pix;
    const int reach = min((int)g.cheb_px[k * md.n_xt], (int)g.cheb_py[k * md.n_yt + ty]);
    const unsigned short *ux = g.cheb_ux + k * np;       // tile columns of each panel
    const int width = 32 * ux[0];
    for (int x0 = 0; x0 < width; x0 += kTx) {
      __syncthreads();                   // earlier reads of lam
      const int nx = min(kTx, width - x0);
      for (int yl = threadIdx.x >> 5; yl < 32; yl += 8)
        for (int xl = threadIdx.x & 31; xl < nx; xl += 32) {
          const int y = 32 * ty + yl, x = x0 + xl;
          lam[yl][xl] = (y < g.n_uy && x < g.n_ux)
                            ? lm[(int64_t)y * g.n_ux + x] * g.cheb_Ek[(int64_t)k * ldx + x]
                            : 0.0;
        }
      __syncthreads();
      for (int P = wave; P < reach; P += 4) {
        const int xe = min(nx, 32 * ux[P] - x0);
        if (x0 > 0 && xe <= 0) break;    // the next panels reach no further
        double *o = T + md.chebt_off + (int64_t)(g.cheb_h[k * np + P] + ty) * 512 + c16;
        v4d t0 = zero4(), t1 = zero4();
        if (x0 > 0) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            t0[r] = o[(4 * r + kk) * 16];
            t1[r] = o[(16 + 4 * r + kk) * 16];
          }
        }
        // two steps at a time: x = x0 + 8 s + 2 kk + (0, 1)
        const double2 *em =
            (const double2 *)(g.cheb_E + (int64_t)(P * 2 * kChebP + c16) * ldx + x0) + kk;
        const double2 *l0 = (const double2 *)lam[c16] + kk, *l1 = (const double2 *)lam[16 + c16] + kk;
#pragma unroll 4
        for (int s = 0; s < xe / 8; ++s) {
          const double2 a = em[4 * s], u = l0[4 * s], v = l1[4 * s];
          t0 = mfma64(u.x, a.x, t0);
          t1 = mfma64(v.x, a.x, t1);
          t0 = mfma64(u.y, a.y, t0);
          t1 = mfma64(v.y, a.y, t1);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          o[(4 * r + kk) * 16] = t0[r];
          o[(16 + 4 * r + kk) * 16] = t1[r];
        }
      }
    }
  }
}

// Inclination derivatives of the tracer's set-up: with q^2 = (q'^2 - cos^2 i)
// / sin^2 i, d(q^2)/di = 2 cot i (1 - q^2); so d(e2)/di = -2 cot i e2.
struct Tracer {
  double cot, dsi2, daq, dnu;           // dnu = d(ln nu0)/di
};

// A term's chain for unit amplitudes: c = (c0, c1) with C = nu0 K_j c, their
// inclination derivatives at fixed nu0, d(gamma)/di, and dc0/db, c1'.
struct Chain {
  double c0, c1, d0, d1, dg, b0, ca;
};
__device__ __forceinline__ double chain_term(const GeomDev &g, const Unit &c, const Tracer &t, int id,
                                             Chain &o) {
  const int j = id >> 10, n = id & 1023;
  const double r = c.mt[j], e2 = c.mt[g.J1 + j];
  const double u = g.u[n], u2 = u * u, ru2 = r * u2;
  const double h = fma(-e2, u2, 1.0);
  const double dh = 2.0 * t.cot * e2 * u2;
  const double rh = rcp64(h), rsh = rsq64(h), lh = dh * rh;      // lh = d ln h
  double ca, A, ra;
  const double d = term_d(c, ru2, rh, ca, A, ra);
  const double rA = rcp64(A);
  const double dA = fma(-ru2 * rh, lh, t.daq);
  const double la = ra * fma(dA, c.ci2, (ca - A) * t.dsi2);      // d ln a (d cos^2 = -d sin^2)
  o.dg = ca * ra * fma(-A, la, dA);
  const double gg = ru2 * rA * rh * rsh, ww = 2.0 * ru2 * rsh;
  const double dgg = -gg * fma(1.5, lh, dA * rA), dww = -0.5 * ww * lh;
  const double f = g.w[n] * kSqrtPi * (ra * rsq64(ra));
  const double pf = fma(c.b, c.si2, c.ci2), Pt = pf * gg;
  const double qv = fma(-2.0 * ca * c.b, gg, ww), Qt = c.si2 * qv;
  const double dP = fma((c.b - 1.0) * t.dsi2, gg, pf * dgg);
  const double dQ = fma(t.dsi2, qv, c.si2 * fma(-2.0 * ca * c.b, dgg, dww));
  o.c0 = f * Pt;
  o.c1 = f * Qt;
  o.d0 = f * fma(-0.5 * la, Pt, dP);
  o.d1 = f * fma(-0.5 * la, Qt, dQ);
  o.b0 = f * c.si2 * gg;                // dC0/db; dC1/db = -2 c1 times it
  o.ca = ca;
  return z_of(c, d);
}

// Inclusive sum over the lanes of a segment that starts at lane `first`.
__device__ __forceinline__ double seg_scan(double v, int lane, int first) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double up = __shfl_up(v, o, 64);
    v += lane - o >= first ? up : 0.0;
  }
  return v;
}

template <bool kShare, int kW>
__device__ __forceinline__ void unit_adjoint(const GeomDev &g, const Unit &c, const Tracer &tr, int P,
                                             int slice, int n_slices, int n_yt,
                                             const double *__restrict__ T, double *A, double *sh,
                                             double *__restrict__ piece) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c16 = lane & 15, kk = lane >> 4;
  const int l32 = lane & 31, w0 = kShare ? wave : 0, nw = kShare ? kW : 1;
  double *B = A + kChebP * kStage;
  const int e0 = g.cheb_ptr[P], e1 = g.cheb_ptr[P + 1];
  const int ys = (min(g.n_uy, 32 * n_yt) + 3) / 4;
  for (int sub = 0; sub < c.n_sub; ++sub) {
    const double ex = -(c.gam0 + node_d(c, sub, c16));
    v4d acc[2] = {zero4(), zero4()};
#pragma unroll 2
    for (int s = w0; s < ys; s += nw) {
      const int y = 4 * s + kk;
      const double yv = g.ys[min(y, g.n_uy - 1)], y2 = yv * yv;
      const double a = T[(int64_t)y * 16 + c16];       // zero past the map
      const double f = exp(ex * y2);
      acc[0] = mfma64(a, f, acc[0]);
      acc[1] = mfma64(a, f * y2, acc[1]);
    }
    // node sensitivities -> Chebyshev coefficients in registers:
    // X = S^T Dblk, then C^T = D16^T X, which is the A operand of C
    v4d cf[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (kShare) acc[q] = sum_waves<kW>(acc[q], sh);
      v4d x = zero4();
#pragma unroll
      for (int s = 0; s < 4; ++s) x = mfma64(acc[q][s], kTab.dblk[4 * s + kk][c16], x);
      cf[q] = zero4();
#pragma unroll
      for (int s = 0; s < 4; ++s) cf[q] = mfma64(kTab.d16[4 * s + kk][c16], x[s], cf[q]);
    }
    if (kShare) __syncthreads();         // the staging below reuses the sums' LDS
    // interpolants at the terms: z[(q, b, i)][t] = sum_j C T_j(eta_t) by matrix
    // cores, then the sum over i with T_i(xi_t); 32 terms at a time
    for (int base = e0 + (slice * nw + w0) * 64; base < e1; base += 64 * nw * n_slices) {
      const int te = base + lane;
      Chain ch = {};
      double xi = 0.0, z = -1.0;
      int id = 0;
      if (te < e1) {
        id = g.cheb_id[te];
        z = chain_term(g, c, tr, id, ch);
        xi = g.cheb_xi[te];
      }
      const bool in = z >= 0.0 && sub_of(c, z) == sub;
      const uint64_t active = __ballot(in);
      if (sub > 0 && active == 0) continue;            // uniform
      const double eta = fma(2.0, z - sub, -1.0);
      double S[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        if (((active >> (32 * half)) & 0xffffffffu) == 0) continue;   // uniform
        if ((lane >> 5) == half) {
          put_chebyshev<kChebP>(A, l32, xi);
          put_chebyshev<16>(B, l32, in ? eta : 0.0);
        }
        wave_sync();
        v4d zz[2][2] = {{zero4(), zero4()}, {zero4(), zero4()}};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const double b = B[(4 * s + kk) * kStage + 16 * q + c16];
            zz[q][0] = mfma64(cf[0][s], b, zz[q][0]);
            zz[q][1] = mfma64(cf[1][s], b, zz[q][1]);
          }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const double xa = A[kk * kStage + 16 * q + c16], xb = A[(4 + kk) * kStage + 16 * q + c16];
#pragma unroll
          for (int v = 0; v < 4; ++v) {               // S0, S1, Sy0, Sy1
            const v4d w = zz[q][v >> 1];
            double s = (v & 1) ? fma(w[3], xb, w[2] * xa) : fma(w[1], xb, w[0] * xa);
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (kk == 2 * half + q) S[v] = s;
          }
        }
        wave_sync();
      }
      // chain of the term, for unit K_j nu0 where it factors out
      double vi = 0.0, vb = 0.0, vh = 0.0;
      if (in) {
        const double amp = c.nu0 * c.mt[2 * g.J1 + (id >> 10)];
        vh = fma(S[0], ch.c0, S[1] * ch.c1);
        vi = amp * (fma(S[0], ch.d0, fma(S[1], ch.d1, tr.dnu * vh)) -
                    ch.dg * fma(ch.c0, S[2], ch.c1 * S[3]));
        vb = amp * ch.b0 * fma(-2.0 * ch.ca, S[1], S[0]);
      }
      // sums over the lanes of equal j
      const int jp = __shfl_up(id >> 10, 1, 64);
      const uint64_t start = __ballot(te < e1 && (lane == 0 || jp != (id >> 10)));
      const uint64_t upto = start & (~0ull >> (63 - lane));
      const int first = 63 - __clzll((long long)(upto | 1));
      vi = seg_scan(vi, lane, first);
      vb = seg_scan(vb, lane, first);
      vh = seg_scan(vh, lane, first);
      const bool last = te < e1 && (te + 1 == e1 || lane == 63 || ((start >> (lane + 1)) & 1));
      if (last) {
        double *o = piece + 3 * (int64_t)(g.cheb_pc[g.cheb_ch[P] + (base - e0) / 64] + __popcll(upto) - 1);
        o[0] = sub ? o[0] + vi : vi;
        o[1] = sub ? o[1] + vb : vb;
        o[2] = sub ? o[2] + vh : vh;
      }
    }
    if (kShare && sub + 1 < c.n_sub) __syncthreads();
  }
}

// Pieces [K][pieces][3] of a model, after its chain rows [K][J1][3].
__device__ __forceinline__ double *piece_base(const GeomDev &g, const ModelDev &md, double *sens) {
  return sens + md.sens_off + 3 * (int64_t)g.K * g.J1;
}

// Items (m, k, panel, slice << 1 | n_slices << 16), every panel, shared as in
// k_cheb_panel: the pieces of one slice of the panel's 64-term chunks (block
// `slice` of every n_slices; each slice forms the node sensitivities anew).
template <bool kShare, int kW>
__device__ __forceinline__ void adj_item(const Item &it, const GeomDev *__restrict__ geoms,
                                         const ModelDev *__restrict__ models, const ParamsDev &p,
                                         const double *__restrict__ gauss,
                                         const int *__restrict__ st_ws,
                                         const double *__restrict__ T, double *A, double *sh,
                                         double *__restrict__ sens) {
  const ModelDev md = models[it.m];
  const GeomDev g = geoms[md.geom];
  if (st_ws[it.m] != 0) return;          // uniform per block where shared; k_grads writes NaN
  Unit c;
  unit_setup(g, gauss + md.gauss_off, it.a, it.b, c);
  Tracer tr;
  const double si = sin(p.inc[it.m]), ci = cos(p.inc[it.m]);
  tr.cot = ci / si;
  tr.dsi2 = 2.0 * si * ci;
  const double f = tr.cot * (c.aq / c.alpha - 1.0);     // cot (1 - q^2) / q^2
  tr.daq = -2.0 * c.aq * f;
  tr.dnu = -f;
  const int u = it.a * g.cheb_np + it.b;
  const int h0 = g.cheb_h[u], nyt = g.cheb_h[u + 1] - h0;
  unit_adjoint<kShare, kW>(g, c, tr, it.b, (it.c >> 1) & 0x7fff, it.c >> 16, nyt, T + md.chebt_off + (int64_t)h0 * 512, A, sh,
                           piece_base(g, md, sens) + 3 * (int64_t)it.a * g.cheb_pieces);
}

template <int kW>
__global__ void __launch_bounds__(64 * kW, 2)
    k_cheb_adj(const GeomDev *__restrict__ geoms, const ModelDev *__restrict__ models,
               const Item *__restrict__ items, int n_it, int n_share, ParamsDev p,
               const double *__restrict__ gauss, const int *__restrict__ st_ws,
               const double *__restrict__ T, double *__restrict__ sens) {
  __shared__ __attribute__((aligned(16))) double L[kW * kWaveLds];
  double *A = L + (threadIdx.x >> 6) * kWaveLds;
  Item it;
  if (!unit_of<kW>(items, n_it, n_share, blockIdx.x, it)) return;
  if ((int)blockIdx.x < n_share)
    adj_item<true, kW>(it, geoms, models, p, gauss, st_ws, T, A, L, sens);
  else
    adj_item<false, kW>(it, geoms, models, p, gauss, st_ws, T, A, L, sens);
}

// Items (m, k, block of 64 mass Gaussians): the chain rows of k_chain, (k, j)
// as the sum of its pieces in panel order; the third value per unit I0_k M_j.
__global__ void __launch_bounds__(64) k_cheb_rows(const GeomDev *__restrict__ geoms,
                                                  const ModelDev *__restrict__ models,
                                                  const Item *__restrict__ items, int n_it,
                                                  const double *__restrict__ gauss,
                                                  const int *__restrict__ st_ws,
                                                  double *__restrict__ sens) {
  for (int i = blockIdx.x; i < n_it; i += gridDim.x) {
    const Item it = items[i];
    const ModelDev md = models[it.m];
    const GeomDev g = geoms[md.geom];
    if (st_ws[it.m] != 0) continue;
    const int k = it.a, j = it.b * 64 + threadIdx.x;
    if (j >= g.J1) continue;
    const double *pc = piece_base(g, md, sens) + 3 * (int64_t)k * g.cheb_pieces;
    double v0 = 0.0, v1 = 0.0, v2 = 0.0;
    const int q1 = g.cheb_jp[j + 1];
    int q = g.cheb_jp[j];
    for (; q + 4 <= q1; q += 4) {
      double a[4][3];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double *s = pc + 3 * (int64_t)g.cheb_jx[q + u];
        a[u][0] = s[0];
        a[u][1] = s[1];
        a[u][2] = s[2];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v0 += a[u][0];
        v1 += a[u][1];
        v2 += a[u][2];
      }
    }
    for (; q < q1; ++q) {
      const double *s = pc + 3 * (int64_t)g.cheb_jx[q];
      v0 += s[0];
      v1 += s[1];
      v2 += s[2];
    }
    const double *tab = gauss + md.gauss_off;
    const double qk = sqrt(tab[k] / tab[g.K + k]);
    const double nu1 = g.lum_q[k] / (sqrt(2.0 * kPi) * g.lum_sigma[k] * qk);   // nu0 / I0
    const double sj = j < g.J1 - 1 ? g.mass_sigma[j] : g.bh_sigma;
    const double kt = sqrt(2.0 / kPi) * grav_const() / (g.s_pc * sj);          // K_j / M_j
    double *o = sens + md.sens_off + 3 * ((int64_t)k * g.J1 + j);
    o[0] = v0;
    o[1] = v1;
    o[2] = nu1 * kt * v2;
  }
}

}  // namespace

// Workgroups of a launch; the kernels with item loops stride over longer lists.
static int grid_for(int n) { return std::min(n, 1 << 22); }
// Blocks of a unit launch: one per shared item, one per kW others.
static int unit_blocks(int n_it, int n_share, int kw) { return n_share + (n_it - n_share + kw - 1) / kw; }

void launch_cheb_panel(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, int n_share,
                       int waves, const double *gauss, const int *st_ws, double *H, hipStream_t st) {
  if (waves == 8)
    k_cheb_panel<8><<<unit_blocks(n_it, n_share, 8), 512, 0, st>>>(g, m, it, n_it, n_share, gauss,
                                                                   st_ws, H);
  else
    k_cheb_panel<4><<<unit_blocks(n_it, n_share, 4), 256, 0, st>>>(g, m, it, n_it, n_share, gauss,
                                                                   st_ws, H);
}
void launch_cheb_map(const GeomDev *g, const ModelDev *m, const ChebItem *it, int n_it,
                     const double *H, const int *st_ws, double *part, hipStream_t st) {
  k_cheb_map<<<grid_for(n_it), 256, 0, st>>>(g, m, it, n_it, H, st_ws, part);
}
void launch_cheb_sum(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, ParamsDev p,
                     const double *part, double *pix, hipStream_t st) {
  k_cheb_sum<<<grid_for(n_it), 256, 0, st>>>(g, m, it, n_it, p, part, pix);
}
void launch_cheb_tmap(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                      const double *pix, const int *st_ws, double *T, hipStream_t st) {
  k_cheb_tmap<<<grid_for(n_it), 256, 0, st>>>(g, m, it, n_it, pix, st_ws, T);
}
void launch_cheb_adj(const GeomDev *g, const ModelDev *m, const Item *it, int n_it, int n_share,
                     int waves, ParamsDev p, const double *gauss, const int *st_ws, const double *T,
                     double *sens, hipStream_t st) {
  if (waves == 8)
    k_cheb_adj<8><<<unit_blocks(n_it, n_share, 8), 512, 0, st>>>(g, m, it, n_it, n_share, p, gauss,
                                                                 st_ws, T, sens);
  else
    k_cheb_adj<4><<<unit_blocks(n_it, n_share, 4), 256, 0, st>>>(g, m, it, n_it, n_share, p, gauss,
                                                                 st_ws, T, sens);
}
void launch_cheb_rows(const GeomDev *g, const ModelDev *m, const Item *it, int n_it,
                      const double *gauss, const int *st_ws, double *sens, hipStream_t st) {
  k_cheb_rows<<<grid_for(n_it), 64, 0, st>>>(g, m, it, n_it, gauss, st_ws, sens);
}

}  // namespace jam
