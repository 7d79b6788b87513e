// Host runtime of the JAM-cyl library: the C ABI of include/jam.h.
//
// Responsibilities: validate inputs, build the device description of every
// geometry once (distinct |x'|/|y'| values of the padded sub-pixel grid, the
// PSF-and-bin weight matrix in both orientations, Gauss-Legendre nodes),
// build per-composition work lists ("plans") once, size the caller's
// workspace, and sequence the kernels on the caller's stream.
#include "jam.h"
#include "jam_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <initializer_list>
#include <list>
#include <queue>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

namespace {

thread_local std::string g_err;

jam_status fail(jam_status s, const char *fmt, ...) {
  char buf[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

#define HIP_TRY(expr)                                                                \
  do {                                                                               \
    hipError_t e_ = (expr);                                                          \
    if (e_ != hipSuccess) return fail(JAM_E_DEVICE, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

constexpr int kMaxNu = 1024;
constexpr double kPi = 3.14159265358979323846;

// n-node Gauss-Legendre rule on [0, 1]: Newton iteration on P_n from the
// asymptotic initial guess, in long double; nodes ascending.
void gauss_legendre01(int n, double *x, double *w) {
  for (int i = 0; i < n; ++i) {
    long double z = std::cos(kPi * (i + 0.75L) / (n + 0.5L));
    long double dp = 1.0L;
    for (int it = 0; it < 100; ++it) {
      long double p0 = 1.0L, p1 = z;
      for (int k = 2; k <= n; ++k) {
        const long double p2 = ((2.0L * k - 1.0L) * z * p1 - (k - 1.0L) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      if (n == 1) { p1 = z; p0 = 1.0L; }
      dp = n * (z * p1 - p0) / (z * z - 1.0L);
      const long double dz = p1 / dp;
      z -= dz;
      if (std::fabs((double)dz) < 1e-19) break;
    }
    // recompute the derivative at the converged node
    long double p0 = 1.0L, p1 = z;
    for (int k = 2; k <= n; ++k) {
      const long double p2 = ((2.0L * k - 1.0L) * z * p1 - (k - 1.0L) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    dp = (n == 1) ? 1.0L : n * (z * p1 - p0) / (z * z - 1.0L);
    const long double wi = 2.0L / ((1.0L - z * z) * dp * dp);
    // z runs from +1 downwards; store ascending on [0, 1]
    x[i] = (double)(0.5L * (1.0L - z));
    w[i] = (double)(0.5L * wi);
  }
}

// Everything the library keeps about one geometry on the host.
struct GeomHost {
  int K = 0, J = 0, J1 = 0, n_u = 0, T = 0;
  int nx = 0, ny = 0, ss = 1, psf_n = 1, h = 0, n_bins = 0;
  int nxp = 0, nyp = 0, n_ux = 0, n_uy = 0, n_pix = 0;
  double bh_sigma = 0, dist = 0, pixsize = 0, xc = 0, yc = 0, s_pc = 0;
  std::vector<double> lum_sigma, lum_q, lum_I0, mass_sigma, mass_q, mass_S0;
  std::vector<double> u, w, xs, ys;
  std::vector<int> ux, uy;
  std::vector<int> bin_ptr, bin_pix, pix_ptr, pix_bin;
  std::vector<double> bin_w, pix_w;
  int max_bin_nnz = 0;   // largest number of weights of one bin
  // spherically aligned model: polar table radii and the 8-node rule
  double sph_lnr0 = 0, sph_dlnr = 0, sph_sig_max = 0;
  double gl8_x[8] = {}, gl8_w[8] = {};
  // compressed cylindrical form (GeomDev)
  int cheb_np = 0, cheb_pieces = 0;
  // gain over the direct forms, forward and adjoint, and the forward's direct cost (ChebCost)
  double cheb_gain[2] = {}, cheb_direct = 0.0;
  std::vector<double> cheb_lo, cheb_xi, cheb_E, cheb_Ek, cheb_Gk;
  std::vector<int> cheb_ptr, cheb_id, cheb_h, cheb_ch, cheb_pc, cheb_jp, cheb_jx;
  std::vector<unsigned char> cheb_px, cheb_py;
  std::vector<unsigned short> cheb_ux;
};

jam_status validate(const jam_geometry &g, int gi) {
  auto bad = [&](const char *what) {
    return fail(JAM_E_INVALID_ARG, "geometry %d: %s", gi, what);
  };
  if (g.n_lum < 1) return bad("n_lum must be >= 1");
  if (g.n_mass < 0) return bad("n_mass must be >= 0");
  if (!g.lum_sigma || !g.lum_q || !g.lum_I0) return bad("luminous MGE arrays are NULL");
  if (g.n_mass > 0 && (!g.mass_sigma || !g.mass_q || !g.mass_S0))
    return bad("mass MGE arrays are NULL");
  for (int k = 0; k < g.n_lum; ++k) {
    if (!(g.lum_sigma[k] > 0) || !std::isfinite(g.lum_sigma[k])) return bad("lum_sigma must be > 0");
    if (!(g.lum_q[k] > 0 && g.lum_q[k] <= 1)) return bad("lum_q must be in (0, 1]");
    if (!(g.lum_I0[k] >= 0) || !std::isfinite(g.lum_I0[k])) return bad("lum_I0 must be >= 0");
  }
  for (int j = 0; j < g.n_mass; ++j) {
    if (!(g.mass_sigma[j] > 0) || !std::isfinite(g.mass_sigma[j])) return bad("mass_sigma must be > 0");
    if (!(g.mass_q[j] > 0 && g.mass_q[j] <= 1)) return bad("mass_q must be in (0, 1]");
    if (!(g.mass_S0[j] >= 0) || !std::isfinite(g.mass_S0[j])) return bad("mass_S0 must be >= 0");
  }
  if (!(g.bh_sigma > 0) || !std::isfinite(g.bh_sigma)) return bad("bh_sigma must be > 0");
  if (!(g.distance_mpc > 0) || !std::isfinite(g.distance_mpc)) return bad("distance_mpc must be > 0");
  if (g.nx < 1 || g.ny < 1) return bad("nx, ny must be >= 1");
  if (!(g.pixsize > 0) || !std::isfinite(g.pixsize)) return bad("pixsize must be > 0");
  if (!std::isfinite(g.xc) || !std::isfinite(g.yc)) return bad("xc, yc must be finite");
  if (g.supersample < 1 || g.supersample > 16) return bad("supersample must be in [1, 16]");
  if (g.psf_n < 1 || g.psf_n % 2 == 0) return bad("psf_n must be odd and >= 1");
  if (!g.psf) return bad("psf is NULL");
  for (int i = 0; i < g.psf_n * g.psf_n; ++i)
    if (!std::isfinite(g.psf[i])) return bad("psf must be finite");
  if (g.n_bins < 1) return bad("n_bins must be >= 1");
  if (!g.bin_index) return bad("bin_index is NULL");
  if (g.n_u < 1 || g.n_u > kMaxNu) return bad("n_u must be in [1, 1024]");
  const int64_t nsub_x = (int64_t)g.nx * g.supersample + g.psf_n - 1;
  const int64_t nsub_y = (int64_t)g.ny * g.supersample + g.psf_n - 1;
  if (nsub_x > 16384 || nsub_y > 16384) return bad("padded sub-pixel grid larger than 16384");
  // term counts and the weight matrix's nonzeros are indexed with 32-bit
  // integers on the device
  const int64_t T = (int64_t)g.n_lum * (g.n_mass + 1) * g.n_u;
  const int64_t T_sph = ((int64_t)(g.n_mass + 1) * g.n_u + 63) / 64 * 64;
  if (T > INT32_MAX || T_sph > INT32_MAX)
    return fail(JAM_E_UNSUPPORTED, "geometry %d: %lld terms exceed the supported 2^31 - 1", gi,
                (long long)std::max(T, T_sph));
  const int64_t nnz_max = (int64_t)g.nx * g.supersample * g.ny * g.supersample * g.psf_n * g.psf_n;
  if (nnz_max > INT32_MAX)
    return fail(JAM_E_UNSUPPORTED, "geometry %d: field sub-pixels x PSF taps exceed 2^31 - 1", gi);
  std::vector<int> cnt(g.n_bins, 0);
  for (int64_t i = 0; i < (int64_t)g.nx * g.ny; ++i) {
    const int b = g.bin_index[i];
    if (b < -1 || b >= g.n_bins) return bad("bin_index out of range");
    if (b >= 0) cnt[b]++;
  }
  for (int b = 0; b < g.n_bins; ++b)
    if (cnt[b] == 0) return fail(JAM_E_INVALID_ARG, "geometry %d: bin %d is empty", gi, b);
  return JAM_OK;
}

// Distinct |v| of a list, ascending, with the index map.
void distinct_abs(const std::vector<double> &v, std::vector<double> &vals, std::vector<int> &map) {
  vals.clear();
  for (double x : v) vals.push_back(std::fabs(x));
  std::sort(vals.begin(), vals.end());
  vals.erase(std::unique(vals.begin(), vals.end()), vals.end());
  map.resize(v.size());
  for (size_t i = 0; i < v.size(); ++i)
    map[i] = (int)(std::lower_bound(vals.begin(), vals.end(), std::fabs(v[i])) - vals.begin());
}

void build_geometry(const jam_geometry &g, GeomHost &o) {
  o.K = g.n_lum;
  o.J = g.n_mass;
  o.J1 = g.n_mass + 1;
  o.n_u = g.n_u;
  o.T = o.K * o.J1 * o.n_u;
  o.nx = g.nx;
  o.ny = g.ny;
  o.ss = g.supersample;
  o.psf_n = g.psf_n;
  o.h = (g.psf_n - 1) / 2;
  o.n_bins = g.n_bins;
  o.bh_sigma = g.bh_sigma;
  o.dist = g.distance_mpc;
  o.pixsize = g.pixsize;
  o.xc = g.xc;
  o.yc = g.yc;
  o.s_pc = g.distance_mpc * 1.0e6 * kPi / 648000.0;
  o.lum_sigma.assign(g.lum_sigma, g.lum_sigma + o.K);
  o.lum_q.assign(g.lum_q, g.lum_q + o.K);
  o.lum_I0.assign(g.lum_I0, g.lum_I0 + o.K);
  if (o.J) {
    o.mass_sigma.assign(g.mass_sigma, g.mass_sigma + o.J);
    o.mass_q.assign(g.mass_q, g.mass_q + o.J);
    o.mass_S0.assign(g.mass_S0, g.mass_S0 + o.J);
  }
  o.u.resize(o.n_u);
  o.w.resize(o.n_u);
  gauss_legendre01(o.n_u, o.u.data(), o.w.data());

  // padded sub-pixel centres (galaxy at the origin)
  const int ssx = o.nx * o.ss, ssy = o.ny * o.ss;
  o.nxp = ssx + 2 * o.h;
  o.nyp = ssy + 2 * o.h;
  const double pitch = o.pixsize / o.ss;
  std::vector<double> xp(o.nxp), yp(o.nyp);
  for (int c = 0; c < o.nxp; ++c) xp[c] = o.xc + ((double)(c - o.h) - (ssx - 1) / 2.0) * pitch;
  for (int r = 0; r < o.nyp; ++r) yp[r] = o.yc + ((double)(r - o.h) - (ssy - 1) / 2.0) * pitch;
  distinct_abs(xp, o.xs, o.ux);
  distinct_abs(yp, o.ys, o.uy);
  o.n_ux = (int)o.xs.size();
  o.n_uy = (int)o.ys.size();
  o.n_pix = o.n_ux * o.n_uy;

  // W[b, p]: the convolved map at field sub-pixel f is
  //   C(f) = sum_o psf[o + h] M(f - o),
  // so bin b's sum of C weights padded sub-pixel (f + h - o) by psf[o + h].
  // Built one bin at a time in a dense scratch row (memory O(n_pix + nnz));
  // each weight accumulates its field sub-pixels in raster order.
  std::vector<std::vector<int>> fields(o.n_bins);
  for (int fy = 0; fy < ssy; ++fy)
    for (int fx = 0; fx < ssx; ++fx) {
      const int b = g.bin_index[(fy / o.ss) * o.nx + fx / o.ss];
      if (b >= 0) fields[b].push_back(fy * ssx + fx);
    }
  const int n = o.psf_n;
  std::vector<double> row(o.n_pix, 0.0);
  std::vector<char> hit(o.n_pix, 0);
  std::vector<int> touched;
  o.bin_ptr.assign(o.n_bins + 1, 0);
  std::vector<int> pcount(o.n_pix, 0);
  o.max_bin_nnz = 0;
  for (int b = 0; b < o.n_bins; ++b) {
    touched.clear();
    for (int f : fields[b]) {
      const int fy = f / ssx, fx = f % ssx;
      for (int oy = -o.h; oy <= o.h; ++oy) {
        const int iy = o.uy[fy + o.h - oy] * o.n_ux;
        const double *kr = g.psf + (oy + o.h) * n;
        for (int ox = -o.h; ox <= o.h; ++ox) {
          const int q = iy + o.ux[fx + o.h - ox];
          if (!hit[q]) {
            hit[q] = 1;
            touched.push_back(q);
          }
          row[q] += kr[ox + o.h];
        }
      }
    }
    std::sort(touched.begin(), touched.end());
    for (int q : touched) {
      if (row[q] != 0.0) {
        o.bin_pix.push_back(q);
        o.bin_w.push_back(row[q]);
        pcount[q]++;
      }
      row[q] = 0.0;
      hit[q] = 0;
    }
    o.bin_ptr[b + 1] = (int)o.bin_pix.size();
    o.max_bin_nnz = std::max(o.max_bin_nnz, o.bin_ptr[b + 1] - o.bin_ptr[b]);
    std::vector<int>().swap(fields[b]);
  }
  o.pix_ptr.assign(o.n_pix + 1, 0);
  for (int p = 0; p < o.n_pix; ++p) o.pix_ptr[p + 1] = o.pix_ptr[p] + pcount[p];
  o.pix_bin.resize(o.bin_pix.size());
  o.pix_w.resize(o.bin_pix.size());
  std::vector<int> fill(o.pix_ptr.begin(), o.pix_ptr.end() - 1);
  for (int b = 0; b < o.n_bins; ++b)
    for (int e = o.bin_ptr[b]; e < o.bin_ptr[b + 1]; ++e) {
      const int p = o.bin_pix[e];
      o.pix_bin[fill[p]] = b;
      o.pix_w[fill[p]] = o.bin_w[e];
      fill[p]++;
    }
}

// Polar table of the spherically aligned model: radii log-spaced from half
// the smallest distance of a padded sub-pixel centre from the centre to
// 12 max sigma'_k / min q'_k; and the 8-node Gauss-Legendre rule on [-1, 1].
void build_spherical(GeomHost &o) {
  double rmin = 0.0;
  for (double x : o.xs)
    for (double y : o.ys) {
      const double r = std::sqrt(x * x + y * y);
      if (r > 0.0 && (rmin == 0.0 || r < rmin)) rmin = r;
    }
  const double r_lo = rmin > 0.0 ? 0.5 * rmin : 1e-3;
  double smax = 0.0, qmin = 1.0;
  for (int k = 0; k < o.K; ++k) {
    smax = std::max(smax, o.lum_sigma[k]);
    qmin = std::min(qmin, o.lum_q[k]);
  }
  const double r_hi = 12.0 * smax / qmin;
  o.sph_lnr0 = std::log(r_lo);
  o.sph_dlnr = (std::log(r_hi) - std::log(r_lo)) / (jam::kSphNR - 1);
  o.sph_sig_max = smax;
  double u[8], w[8];
  gauss_legendre01(8, u, w);
  for (int i = 0; i < 8; ++i) {
    o.gl8_x[i] = 2.0 * u[i] - 1.0;
    o.gl8_w[i] = 2.0 * w[i];
  }
}

std::vector<std::pair<int, int>> axis_tiles(int n, int tau) {
  const int nb = (n + 31) / 32;
  std::vector<std::pair<int, int>> out;   // (first block, blocks)
  for (int b = 0; b < nb;) {
    const int w = (n >= tau && b + 1 < nb) ? 2 : 1;
    out.push_back({b, w});
    b += w;
  }
  return out;
}

// ns of one SIMD per term: matrix instructions, exponentials and the loop; terms
// computed in place on top.  In place, 4096 models of 13000 terms: 12 x 12 pixels
// 9.9 ns, 20 x 20 16.9, 24 x 24 20.4, the block 26.6.
constexpr double kTermInPlaceNs = 4.5;
double block_ns(int BX, int BY) { return 14.5 * BX * BY + 4.1 * BX + 2.9 * BY; }
constexpr int kSmallSides[3] = {3, 5, 6};
double tiles_ns(int X, int Y) {
  const int tx = kSmallSides[X], ty = kSmallSides[Y];
  return 0.256 * tx * ty + 0.51 * tx + 0.35 * ty + 1.2;
}
constexpr double kSmallGain = 0.9;
// The cheapest cover of a larger map by 4 x 4 tilings, ns per term of the map, where
// it costs less than kSmallGain of its blocks (choose_tilings); otherwise its blocks.
struct MapCover {
  double ns = 0.0;
  int X = -1, Y = -1;           // tiling; -1: 32 x 32 blocks
};
MapCover cover_of(int n_ux, int n_uy, int tau) {
  MapCover c;
  for (const auto &x : axis_tiles(n_ux, tau))
    for (const auto &y : axis_tiles(n_uy, tau)) c.ns += block_ns(x.second, y.second);
  double best = kSmallGain * c.ns;
  for (int X = 0; X < 3; ++X)
    for (int Y = 0; Y < 3; ++Y) {
      const int w = 4 * kSmallSides[X], h = 4 * kSmallSides[Y];
      const double cost = ((n_ux + w - 1) / w) * ((n_uy + h - 1) / h) * tiles_ns(X, Y);
      if (cost < best) {
        best = cost;
        c = MapCover{cost, X, Y};
      }
    }
  return c;
}

// The compressed form's cost against the direct forms', in ns of one SIMD for a model.
// Direct: per term the map's tiles, in the adjoint its blocks; compressed: per term,
// per (tracer, panel) unit, per unit and 32 map rows that it reaches (the node
// contraction and its exponentials), per unit and tile that it reaches (FP64 MFMAs) and
// per tile (the sum of the partials).  Fitted by least squares to the difference of
// whole calls, forced into one form and the other, of 450 batches drawn at random: 1 to
// 800 models of 3 to 60 x 2 to 95 Gaussians, 33 to 300 distinct coordinates an axis, 72
// to 15000 terms per tracer, pixels of 0.02 to 0.08".  The form taken (choose_cheb) is
// there 0.3 % (forward) and 1 % (adjoint) slower than the better one on average; by more
// than a tenth in 3 and 19 of them.
struct ChebCost { double direct, term, unit, row, tile, map; };
constexpr ChebCost kChebFwd{1.06, 7.8, 2000.0, 1130.0, 787.0, 6580.0};   // direct: per ns of the tiles
constexpr ChebCost kChebAdj{32.0, 17.1, 2160.0, 4210.0, 936.0, 0.0};     // per term and block
struct ChebWork { double terms, units, rows, tiles; };   // of all tracers
double cheb_ns(const GeomHost &o, const ChebCost &c, const ChebWork &w) {
  const double bx = (o.n_ux + 31) / 32, by = (o.n_uy + 31) / 32;
  return c.term * w.terms + c.unit * w.units + c.row * w.rows + c.tile * w.tiles + c.map * bx * by;
}
// The models of a batch that take the compressed form (Tune::cheb), forward or adjoint:
// those that gain, or all that have its tables, which are built up to twice the direct
// adjoint's cost.
constexpr int kChebFwdGain = 1, kChebAdjGain = 2, kChebFwdAll = 4, kChebAdjAll = 8;
constexpr int kChebAnyFwd = kChebFwdGain | kChebFwdAll;
bool takes_cheb(const GeomHost &g, int cheb, bool adjoint) {
  return g.cheb_np > 0 && ((cheb & (adjoint ? kChebAdjAll : kChebFwdAll)) ||
                           ((cheb & (adjoint ? kChebAdjGain : kChebFwdGain)) && g.cheb_gain[adjoint] > 0.0));
}

// Tables of the compressed cylindrical form (GeomDev): panels of v = r u^2,
// the first [0, 1 / M2) with M2 the map's largest squared coordinate, then a
// factor kChebR wide each; empty ones are left out.
// Unique-pixel maps with at most this many distinct |x'| and |y'| (one 32x32
// matrix-core block) take the small-map form: terms computed in place by the
// numerator, sensitivities and chain fused in the adjoint (for at most
// jam::kSmallAdjMass mass Gaussians, the BH included).
constexpr int kSmallMap = 32;
constexpr double kChebCut = 160.0; // a unit is zero where its exponent exceeds this (FP32 sums
                                   // underflow at 87)
void build_cheb(GeomHost &o) {
  o.cheb_np = 0;
  if (o.n_ux <= kSmallMap && o.n_uy <= kSmallMap && o.J1 <= jam::kSmallAdjMass) return;
  const double m2 = std::max(o.xs.back() * o.xs.back(), o.ys.back() * o.ys.back());
  if (!(m2 > 0.0) || !std::isfinite(1.0 / m2)) return;
  const double v1 = 1.0 / m2;
  const int nt = o.J1 * o.n_u;
  std::vector<int> panel(nt);
  std::vector<double> vt(nt);
  int count[jam::kChebMaxPanels] = {}, top = 0;
  double edge[jam::kChebMaxPanels + 1];
  edge[0] = 0.0;
  for (int e = 1; e <= jam::kChebMaxPanels; ++e) edge[e] = v1 * std::pow(jam::kChebR, e - 1);
  for (int j = 0; j < o.J1; ++j) {
    const double sig = j < o.J ? o.mass_sigma[j] : o.bh_sigma;
    const double r = 0.5 / (sig * sig);
    for (int n = 0; n < o.n_u; ++n) {
      const double v = r * (o.u[n] * o.u[n]);
      if (!(v < edge[jam::kChebMaxPanels])) return;
      const int e = (int)(std::upper_bound(edge, edge + jam::kChebMaxPanels, v) - edge) - 1;
      vt[j * o.n_u + n] = v;
      panel[j * o.n_u + n] = e;
      count[e]++;
      top = std::max(top, e);
    }
  }
  std::vector<int> index(top + 1, -1);
  int np = 0;
  for (int e = 0; e <= top; ++e)
    if (count[e]) index[e] = np++;
  o.cheb_lo.assign(2 * np, 0.0);
  o.cheb_ptr.assign(np + 1, 0);
  for (int e = 0; e <= top; ++e) {
    const int P = index[e];
    if (P < 0) continue;
    o.cheb_lo[P] = edge[e];
    o.cheb_lo[np + P] = edge[e + 1];
    o.cheb_ptr[P + 1] = o.cheb_ptr[P] + count[e];
  }
  const int ntx = (o.n_ux + 31) / 32, nty = (o.n_uy + 31) / 32, ldx = 32 * ntx, ldy = 32 * nty;
  o.cheb_px.assign((size_t)o.K * ntx, 0);
  o.cheb_py.assign((size_t)o.K * nty, 0);
  o.cheb_ux.assign((size_t)o.K * np, 0);
  o.cheb_h.assign((size_t)o.K * np + 1, 0);
  ChebWork fwd{}, adj{};
  for (int k = 0; k < o.K; ++k) {
    const double a = 0.5 / (o.lum_sigma[k] * o.lum_sigma[k]), ay = a / (o.lum_q[k] * o.lum_q[k]);
    // panels reaching a tile: by its smallest coordinate (d >= v, so the
    // panel's lower end in v bounds its decay in y too)
    auto reach = [&](double alpha, double q) {
      int c = 0;
      while (c < np && (alpha + o.cheb_lo[c]) * (q * q) <= kChebCut) ++c;
      return (unsigned char)c;
    };
    unsigned char *px = o.cheb_px.data() + (size_t)k * ntx, *py = o.cheb_py.data() + (size_t)k * nty;
    for (int t = 0; t < ntx; ++t) px[t] = reach(a, o.xs[32 * t]);
    for (int t = 0; t < nty; ++t) py[t] = reach(ay, o.ys[32 * t]);
    for (int P = 0; P < np; ++P) {
      int tiles = 0, cols = 0;
      while (cols < ntx && px[cols] > P) ++cols;
      if (cols > 0)
        while (tiles < nty && py[tiles] > P) ++tiles;
      o.cheb_ux[(size_t)k * np + P] = (unsigned short)cols;
      o.cheb_h[(size_t)k * np + P + 1] = o.cheb_h[(size_t)k * np + P] + tiles;
      if (tiles > 0) {
        fwd.units += 1.0;
        fwd.terms += o.cheb_ptr[P + 1] - o.cheb_ptr[P];
      }
    }
    for (int ty = 0; ty < nty; ++ty)
      for (int tx = 0; tx < ntx; ++tx) fwd.tiles += std::min(px[tx], py[ty]);
  }
  fwd.rows = adj.rows = o.cheb_h.back();
  adj.tiles = fwd.tiles;
  adj.terms = o.T;
  adj.units = (double)o.K * np;
  const double direct_adj = kChebAdj.direct * (double)o.T * ntx * nty;
  o.cheb_direct = kChebFwd.direct * (double)o.T * cover_of(o.n_ux, o.n_uy, 0).ns;
  o.cheb_gain[0] = o.cheb_direct - cheb_ns(o, kChebFwd, fwd);
  o.cheb_gain[1] = direct_adj - cheb_ns(o, kChebAdj, adj);
  if (o.cheb_gain[0] <= 0.0 && o.cheb_gain[1] < -direct_adj) {
    for (auto *v : {&o.cheb_ptr, &o.cheb_h}) v->clear();
    for (auto *v : {&o.cheb_px, &o.cheb_py}) v->clear();
    o.cheb_lo.clear();
    o.cheb_ux.clear();
    return;
  }
  o.cheb_id.resize(nt);
  o.cheb_xi.resize(nt);
  std::vector<int> fill(o.cheb_ptr.begin(), o.cheb_ptr.end() - 1);
  const double lr = std::log(jam::kChebR);
  for (int j = 0; j < o.J1; ++j)
    for (int n = 0; n < o.n_u; ++n) {
      const int t = j * o.n_u + n, P = index[panel[t]], at = fill[P]++;
      const double lo = o.cheb_lo[P];
      o.cheb_id[at] = j << 10 | n;
      o.cheb_xi[at] = lo == 0.0 ? 2.0 * (vt[t] / v1) - 1.0 : 2.0 * (std::log(vt[t] / lo) / lr) - 1.0;
    }
  // chunks of 64 terms within a panel and their runs of equal j
  o.cheb_ch.assign(np + 1, 0);
  std::vector<std::vector<int>> of_j(o.J1);
  for (int P = 0; P < np; ++P) {
    for (int e = o.cheb_ptr[P]; e < o.cheb_ptr[P + 1]; ++e) {
      if ((e - o.cheb_ptr[P]) % 64 == 0) {
        o.cheb_pc.push_back(o.cheb_pieces);
      } else if (o.cheb_id[e] >> 10 == o.cheb_id[e - 1] >> 10) {
        continue;
      }
      of_j[o.cheb_id[e] >> 10].push_back(o.cheb_pieces++);
    }
    o.cheb_ch[P + 1] = (int)o.cheb_pc.size();
  }
  o.cheb_jp.assign(1, 0);
  for (auto &v : of_j) {
    o.cheb_jx.insert(o.cheb_jx.end(), v.begin(), v.end());
    o.cheb_jp.push_back((int)o.cheb_jx.size());
  }
  o.cheb_E.assign((size_t)np * 2 * jam::kChebP * ldx, 0.0);
  for (int P = 0; P < np; ++P)
    for (int m = 0; m < jam::kChebP; ++m) {
      const double x = 0.5 * (std::cos(kPi * (m + 0.5) / jam::kChebP) + 1.0);
      const double lo = o.cheb_lo[P], v = lo == 0.0 ? x * v1 : lo * std::exp(lr * x);
      double *row = o.cheb_E.data() + (size_t)(P * 2 * jam::kChebP + m) * ldx;
      double *sq = row + (size_t)jam::kChebP * ldx;
      for (int i = 0; i < o.n_ux; ++i) {
        const double x2 = o.xs[i] * o.xs[i];
        row[i] = std::exp(-v * x2);
        sq[i] = x2 * row[i];
      }
    }
  o.cheb_Ek.assign((size_t)o.K * ldx, 0.0);
  o.cheb_Gk.assign((size_t)o.K * ldy, 0.0);
  for (int k = 0; k < o.K; ++k) {
    const double a = 0.5 / (o.lum_sigma[k] * o.lum_sigma[k]), ay = a / (o.lum_q[k] * o.lum_q[k]);
    for (int i = 0; i < o.n_ux; ++i) o.cheb_Ek[(size_t)k * ldx + i] = std::exp(-a * (o.xs[i] * o.xs[i]));
    for (int i = 0; i < o.n_uy; ++i) o.cheb_Gk[(size_t)k * ldy + i] = std::exp(-ay * (o.ys[i] * o.ys[i]));
  }
  o.cheb_np = np;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// How a plan schedules its numerator (what the autotuner varies).
struct Tune {
  int rule = 1;     // 0 per-pixel VALU everywhere; 1 matrix cores, one wave per tile of
                    // 32x32 blocks
  int tau = 0;      // a map axis with at least tau distinct values pairs its 32-blocks
                    // into 64-wide tiles
  int gran = 0;     // slice length: units of 64 terms per MFMA item, or (k, j) pairs per
                    // per-pixel item; 0 = derived from the batch
  int launch = 0;   // 0 one workgroup per item; 1 persistent grid pulling items from a
                    // device queue
  int cheb = -1;    // derived from the batch, not tuned (-1: still to be derived): the
                    // models in the compressed form (takes_cheb)
};

// Every pointer a captured graph was recorded with (parameters, outputs,
// cotangents, gradients, workspace) in a fixed order, and the workspace
// size; a graph is replayed only when all of them match exactly.
struct GraphKey {
  static constexpr int kMax = 16;
  const void *p[kMax] = {};
  int n = 0;
  size_t ws_bytes = 0;
  GraphKey() = default;
  GraphKey(std::initializer_list<const void *> ptrs, size_t ws) : ws_bytes(ws) {
    for (const void *q : ptrs) p[n++] = q;
  }
  bool operator==(const GraphKey &o) const {
    if (n != o.n || ws_bytes != o.ws_bytes) return false;
    for (int i = 0; i < n; ++i)
      if (p[i] != o.p[i]) return false;
    return true;
  }
};

// A prepared batch composition.
struct Plan {
  std::vector<int32_t> key;
  int n = 0;
  Tune tune;
  void *arena = nullptr;
  jam::ModelDev *d_models = nullptr;
  jam::Item *d_terms = nullptr, *d_pix = nullptr, *d_num = nullptr, *d_bins = nullptr,
            *d_maps = nullptr, *d_chain = nullptr, *d_sens = nullptr, *d_sb = nullptr,
            *d_red = nullptr, *d_sph = nullptr, *d_pro = nullptr, *d_adj = nullptr,
            *d_sensw = nullptr, *d_sgrid = nullptr, *d_sgred = nullptr,
            *d_sgred3 = nullptr, *d_pcot = nullptr, *d_pfix = nullptr, *d_sgs = nullptr,
            *d_sphm = nullptr, *d_ptab = nullptr, *d_srow = nullptr, *d_numsm = nullptr, *d_cpan = nullptr, *d_csum = nullptr, *d_cadj = nullptr,
            *d_ctmap = nullptr, *d_crows = nullptr;
  jam::ChebItem *d_cmap = nullptr;
  // compressed forward: models taken together, [first, end) of their items
  // and how many of the panel items a block's waves share; the groups share
  // one H region
  struct ChebGroup { int pan0, pan1, map0, map1, pan_share; };
  std::vector<ChebGroup> cheb_groups;
  int n_terms = 0, n_pix = 0, n_num = 0, n_bins = 0, n_maps = 0, n_chain = 0, n_sens = 0,
      n_sb = 0, n_red = 0, n_sph = 0, n_pro = 0, n_adj = 0, n_sensw = 0,
      n_sgrid = 0, n_sgred = 0, n_sgred3 = 0, n_pcot = 0, n_pfix = 0, n_sgs = 0, n_sphm = 0, n_ptab = 0, n_srow = 0, n_numsm = 0,
      n_cpan = 0, n_csum = 0, n_cadj = 0, n_cmap = 0, n_ctmap = 0, n_crows = 0;
  int cadj_share = 0, cheb_waves = 4, cadj_waves = 4;   // shared adjoint items, waves per block
  int n_cheb = 0;        // models of the compressed form
  int numsm_ptr[jam::kSmallTilings + 1] = {};   // small-map items by tiling
  int adj_ptr[jam::kSmallQuads + 1] = {};       // and the adjoint's by y quads (1 ..)
  int n_bins_wave = 0;   // leading bin items summed one bin per wave
  int n_pro_fwd = 0;     // leading prologue items, all that the forward needs
  bool spherical = false;
  bool fused_prologue = true;
  int grid_num = 1, grid_sens = 1;
  int64_t total_bins = 0, total_lum = 0, total_mass = 0, total_map = 0;
  // workspace regions (bytes)
  size_t off_status = 0, off_queue = 0, off_gauss = 0, off_terms = 0, off_pix = 0, off_part = 0,
         off_bins = 0, off_vfwd = 0, off_sph = 0, off_sgrid = 0, off_sgrid3 = 0, off_sgcot = 0, off_pol = 0,
         off_sens = 0,
         off_vtmp = 0,
         off_cot = 0,
         off_sbp = 0,
         off_cheb = 0,
         off_chebt = 0,
         off_terms64 = 0,
         ws_fwd = 0, ws_vjp = 0;
  // captured evaluations (forward, adjoint, forward + chi^2, adjoint of chi^2)
  hipGraphExec_t gexec[4] = {nullptr, nullptr, nullptr, nullptr};
  GraphKey gkey[4];
  ~Plan() {
    for (auto &g : gexec)
      if (g) (void)hipGraphExecDestroy(g);
    if (arena) (void)hipFree(arena);
  }
};

}  // namespace

// Event pairs bracketing launches of one kernel, for jam_timing.
struct KernelTimer {
  static constexpr int kCap = 4096;
  std::vector<hipEvent_t> start, stop;
  int used = 0;
  bool on = false;
  void destroy() {
    for (auto e : start) (void)hipEventDestroy(e);
    for (auto e : stop) (void)hipEventDestroy(e);
    start.clear();
    stop.clear();
  }
  bool begin(hipStream_t st, bool capturing) {
    if (!on || capturing || used >= (int)start.size()) return false;
    return hipEventRecord(start[used], st) == hipSuccess;
  }
  void end(hipStream_t st) { (void)hipEventRecord(stop[used++], st); }
};

// ---------------------------------------------------------------------------
// Fixed scratch memory of jam_eval_batch_noalloc.  Each GPU the library runs
// on holds its own copy of this array until the process ends.  In host code
// its name is only a host-side stand-in: the device address is taken once
// per device with hipGetSymbolAddress (at jam_create, with that device
// current) and that address, never the name, is what host code passes on.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on device `dev`, which must be current.
jam_status scratch_address(int dev, void **out) {
  if (dev < 0 || dev >= kMaxDevices) return fail(JAM_E_UNSUPPORTED, "device %d out of range", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return JAM_OK;
}
}  // namespace

struct jam_ctx {
  int device = 0;
  int n_cu = 256;
  int occ_num_pix = 1, occ_num_mfma = 1, occ_sens = 1;
  jam_options opt{0, 0, nullptr, 0, 0, 0};
  std::string tune_path;
  std::vector<std::pair<std::string, Tune>> tuned;   // autotuner cache
  std::vector<GeomHost> gh;
  void *arena = nullptr;
  jam::GeomDev *d_geoms = nullptr;
  std::list<std::unique_ptr<Plan>> plans;   // most recent first
  KernelTimer t_num, t_sens;
  hipStream_t cap_stream = nullptr;         // graph capture only
  void *scratch = nullptr;                  // device address of the fixed scratch array
  // observed kinematics per geometry (chi^2): one device buffer each holding
  // [vrms_obs | inverse covariance], and the device table of pointers
  std::vector<void *> kin_buf;
  std::vector<jam::KinDev> kin_host;
  jam::KinDev *d_kin = nullptr;
  ~jam_ctx() {
    plans.clear();
    t_num.destroy();
    t_sens.destroy();
    if (cap_stream) (void)hipStreamDestroy(cap_stream);
    for (void *b : kin_buf)
      if (b) (void)hipFree(b);
    if (d_kin) (void)hipFree(d_kin);
    if (arena) (void)hipFree(arena);
  }
};

namespace {

constexpr size_t kMaxPlans = 8;
// Batches of at most this many models run the cylindrical prologue as one
// launch (each term block recomputes its (k, j) pairs' set-up, which costs
// latency per block but saves two launches).
constexpr int kFusedPrologueModels = 32;
// Geometries whose bins have at most this many weights each sum every bin
// with one wave (4 bins per workgroup) instead of a whole workgroup.
constexpr int kBinWaveNnz = 2048;

// Numerator variant and term-range split of one model under a schedule.
// `gran` is the slice length in units: (k, j) pairs for the per-pixel
// variant, 64 terms for the matrix-core variant.  The matrix-core variant
// covers the unique-pixel map with wave tiles of BX x BY blocks of 32x32:
// along an axis with at least tau distinct values the blocks pair up into
// 64-wide tiles (an odd last block stays 32 wide).
struct WaveTile {
  int bx, by, BX, BY;   // origin in 32-blocks, extent in blocks (1 or 2)
};

struct NumChoice {
  int kind;      // 0 per-pixel VALU, 2 matrix-core wave tiles, 5 compressed (no items here)
  bool gen = false;   // matrix core on a map of one 32x32 block, terms computed in place
  int n_slices;
  int units;     // slice units of the whole term range
  std::vector<WaveTile> tiles;   // matrix core
  int pix_blocks = 0;            // per-pixel: 64-pixel blocks
  int n_tiles() const { return kind == 0 ? pix_blocks : (int)tiles.size(); }
  double tile_units(int i) const { return kind == 0 ? 1.0 : tiles[i].BX * tiles[i].BY; }
};

// Maps in items of 4 x 4 tiles, 12, 20 or 24 pixels wide and high, instead of 32 x
// 32 blocks.  Of a map of one block, where the items compute the terms in place:
// one item rounded up to those sizes (28 x 28, 49 tiles, would cost about the block
// and take more registers than two waves a SIMD have; 16 takes the 20-wide items:
// three sizes are nine kernels, a fourth would make it sixteen).  The tiles' sums
// over their sixteen terms' blocks cost an item about as much as two chunks of a
// wave save.
// Of a larger one (terms from their table): the items that cover it cheapest,
// where they cost less than kSmallGain of its blocks, most of which are padding
// just past a multiple of 32.  64 models of 10 x 13 x 40 terms, the whole call,
// blocks / tiles: 33 x 33 67.0 / 57.7 us, 39 x 21 48.2 / 43.0, 44 x 44 68.6 /
// 68.1, 70 x 70 117.0 / 105.9, and where the rule keeps the blocks 28 x 40 52.0 /
// 57.7.  Each tiling is one more launch: choose_tilings.
constexpr int kSmallMinChunks = 2;
struct SmallTiles {
  int tiling = -1;              // -1: 32 x 32 blocks
  int nx = 1, ny = 1, w = 0, h = 0;   // items along x and y, their pixels
};
SmallTiles small_tiles(const GeomHost &g, const NumChoice &c, int tau) {
  SmallTiles s;
  if (c.kind != 2 || c.units < 4 * kSmallMinChunks * c.n_slices) return s;
  if (c.gen) {
    if (g.n_ux > 24 || g.n_uy > 24) return s;
    auto size = [](int n) { return n <= 12 ? 0 : (n <= 20 ? 1 : 2); };
    s.tiling = 3 * size(g.n_ux) + size(g.n_uy);
    return s;
  }
  const MapCover m = cover_of(g.n_ux, g.n_uy, tau);
  if (m.X < 0) return s;
  s.tiling = 9 + 3 * m.X + m.Y;
  s.w = 4 * kSmallSides[m.X];
  s.h = 4 * kSmallSides[m.Y];
  s.nx = (g.n_ux + s.w - 1) / s.w;
  s.ny = (g.n_uy + s.h - 1) / s.h;
  return s;
}

// Time of one launch in ns: its items' sum in ns of one SIMD over the chip, and
// the longest item, which a block's four waves share and which takes 1.4 times as
// long on a CU of its own.  256, 512, 1024, 4096 items of 13000 terms on 12 x 12
// pixels: 55, 87, 151 and 535 us here, 54, 84, 147 and 515 measured.  Launches of
// one stream run one after the other, so in a batch of many kinds each kind's own
// kernel is the slower choice until a launch fills the chip several times.
struct LaunchLoad {
  double sum = 0.0, longest = 0.0;
  void add(double items, double item_ns) {
    sum += items * item_ns;
    longest = std::max(longest, item_ns);
  }
  void add(const LaunchLoad &o) {
    sum += o.sum;
    longest = std::max(longest, o.longest);
  }
  double ns(int n_cu) const {
    if (sum == 0.0) return 0.0;
    const double alone = 1.4 * longest / 4.0;
    return 7000.0 + std::max(alone, sum / (4.0 * n_cu) + 0.35 * alone);
  }
};

NumChoice choose_numerator(const GeomHost &g, const Tune &t, int gran) {
  NumChoice c;
  if (t.rule == 0) {
    const int pairs = g.K * g.J1;
    const int per = std::max(1, gran);
    c.kind = 0;
    c.n_slices = std::max(1, (pairs + per - 1) / per);
    c.units = pairs;
    c.pix_blocks = (g.n_pix + 255) / 256;
    return c;
  }
  const int chunks = (g.T + 63) / 64;
  if (takes_cheb(g, t.cheb, false)) {
    c.kind = 5;
    c.n_slices = 0;
    c.units = 0;
    return c;
  }
  c.kind = 2;
  const int per = std::max(4, gran);
  c.gen = g.n_ux <= kSmallMap && g.n_uy <= kSmallMap && g.J1 <= jam::kSmallAdjMass;
  c.n_slices = std::max(1, (chunks + per - 1) / per);
  c.units = chunks;
  for (const auto &ty : axis_tiles(g.n_uy, t.tau))
    for (const auto &tx : axis_tiles(g.n_ux, t.tau))
      c.tiles.push_back({tx.first, ty.first, tx.second, ty.second});
  return c;
}

// Doubles of a model's split-term partial maps, padded to whole blocks.
int64_t part_doubles(const GeomHost &g, const NumChoice &c) {
  return (int64_t)c.n_slices * (32 * ((g.n_ux + 31) / 32)) * (32 * ((g.n_uy + 31) / 32));
}
// A single slice of a matrix-core form goes straight into the N map.  (A map of one
// block keeps its 8 KB.)
int64_t part_size(const GeomHost &g, const NumChoice &c) {
  return c.kind == 2 && c.n_slices == 1 && !c.gen ? 0 : part_doubles(g, c);
}

// Relative cost of one numerator item, for largest-first ordering and the
// schedule model: the kernels' chunk loop plus a fixed per-item cost (the
// partial-tile store and its reduction).  `tile` indexes c's tiles.
double num_item_cost(const GeomHost &g, const NumChoice &c, int slice, int tile) {
  if (c.kind == 0) {
    const int pairs = g.K * g.J1;
    const int per = (pairs + c.n_slices - 1) / c.n_slices;
    const int cnt = std::max(0, std::min(pairs, (slice + 1) * per) - slice * per);
    return cnt * (double)g.n_u * 256.0 * 5.0 / 32768.0 + 1.0;
  }
  const int chunks = (g.T + 63) / 64;
  const int per = (chunks + c.n_slices - 1) / c.n_slices;
  const int cnt = std::max(0, std::min(chunks, (slice + 1) * per) - slice * per);
  // per chunk of a wave (a quarter of the item's chunks): 32 MFMAs per block
  // and operand generation per row / column block; per item: the start
  // (dependent descriptor and coordinate loads, first chunk), the four-wave
  // sum and the tile store
  const WaveTile &w = c.tiles[tile];
  // terms computed in place: their FP64 set-up per chunk
  const double gen = c.gen ? 0.5 : 0.0;
  return ((cnt + 3) / 4) * (1.5 * w.BX * w.BY + 0.75 * (w.BX + w.BY) + gen) + 8.0;
}

// Completion time of the numerator launch as modelled: every resident
// workgroup pulls the next item, largest first, from the queue, i.e. list
// scheduling in cost order on `slots` identical workers.
double list_schedule_makespan(std::vector<double> &cost, int slots) {
  std::sort(cost.begin(), cost.end(), std::greater<double>());
  if (cost.empty()) return 0.0;
  if ((int)cost.size() <= slots) return cost[0];
  std::priority_queue<double, std::vector<double>, std::greater<double>> q;
  for (int i = 0; i < slots; ++i) q.push(0.0);
  double mk = 0.0;
  for (double c : cost) {
    const double t = q.top() + c;
    q.pop();
    mk = std::max(mk, t);
    q.push(t);
  }
  return mk;
}

// Workers of the schedule model.  A compute unit processes the workgroups
// resident on it at its full rate however many there are (co-resident
// workgroups share its SIMDs), so the model's workers are the compute units
// and its jobs the workgroup items.
int num_slots(const jam_ctx *ctx, const Tune &) { return std::max(1, ctx->n_cu); }

// Modelled time of the numerator launch with slices of `gran`; 1e300 for more items
// than most_items.
double gran_makespan(const jam_ctx *ctx, int n, const int32_t *geom_idx, const Tune &t, int gran,
                     size_t most_items) {
  std::vector<std::vector<double>> of(ctx->gh.size());   // a geometry's items
  std::vector<char> known(ctx->gh.size(), 0);
  std::vector<double> cost;
  for (int m = 0; m < n; ++m) {
    const int i = geom_idx[m];
    if (!known[i]) {
      const GeomHost &g = ctx->gh[i];
      const NumChoice c = choose_numerator(g, t, gran);
      for (int sl = 0; sl < c.n_slices; ++sl)
        for (int tl = 0; tl < c.n_tiles(); ++tl) of[i].push_back(num_item_cost(g, c, sl, tl));
      known[i] = 1;
    }
    if (cost.size() + of[i].size() > most_items) return 1e300;
    cost.insert(cost.end(), of[i].begin(), of[i].end());
  }
  return list_schedule_makespan(cost, num_slots(ctx, t));
}

// Default slice length: the one whose item list the workers finish first
// under the list-scheduling model.  Candidates are geometric around a few
// jobs per worker, plus the exact splits of the largest model, so a uniform
// item list can fill whole rounds of workers.
int default_gran(const jam_ctx *ctx, int n, const int32_t *geom_idx, const Tune &t) {
  const int slots = num_slots(ctx, t);
  double work = 0.0, big_work = -1.0;
  int big_units = 1, big_tiles = 1;
  for (int m = 0; m < n; ++m) {
    const GeomHost &g = ctx->gh[geom_idx[m]];
    const NumChoice c = choose_numerator(g, t, 1 << 29);
    const double w = (double)c.n_tiles() * c.units;
    work += w;
    if (w > big_work) {
      big_work = w;
      big_units = c.units;
      big_tiles = c.n_tiles();
    }
  }
  // jobs a worker holds at once
  const double per_slot = t.rule == 0 ? ctx->occ_num_pix : ctx->occ_num_mfma;
  const double g0 = std::max(1.0, std::ceil(work / (slots * per_slot)));
  std::vector<int> cands;
  for (int k = -8; k <= 16; ++k)
    cands.push_back((int)std::min(1.0e9, std::max(1.0, std::round(g0 * std::pow(2.0, k / 8.0)))));
  if (big_work >= 0.25 * work) {
    const int s_max = std::min(4096, (int)(4 * per_slot) * slots / std::max(1, big_tiles) + 1);
    for (int sl = 1; sl <= s_max; ++sl) cands.push_back((big_units + sl - 1) / sl);
  }
  std::sort(cands.begin(), cands.end());
  cands.erase(std::unique(cands.begin(), cands.end()), cands.end());
  double best = 1e300;
  int best_g = (int)g0;
  for (int gr : cands) {
    const double mk = gran_makespan(ctx, n, geom_idx, t, gr, (size_t)(64 * per_slot) * slots + (size_t)4 * n);
    if (mk >= 1e300) continue;   // too fine
    if (mk < best * (1.0 - 1e-9) || (mk <= best * (1.0 + 1e-9) && gr > best_g)) {
      best = mk;
      best_g = gr;
    }
  }
  return std::min(1 << 29, std::max(1, best_g));
}

void sort_by_cost(std::vector<jam::Item> &items, std::vector<double> &cost) {
  std::vector<size_t> idx(items.size());
  for (size_t i = 0; i < idx.size(); ++i) idx[i] = i;
  std::stable_sort(idx.begin(), idx.end(), [&](size_t a, size_t b) { return cost[a] > cost[b]; });
  std::vector<jam::Item> out(items.size());
  for (size_t i = 0; i < idx.size(); ++i) out[i] = items[idx[i]];
  items.swap(out);
}

// The wide adjoint form (k_sens_wide) is used on maps of at least two x
// tiles with at least this many distinct |y|: each 32-term group then runs
// over enough y steps to amortise its accumulator set-up and epilogue
// (measured: faster than the one-tile form at 215, slower at <= 128).
constexpr int kWideMinY = 160;

struct WidePart { int m, pt, xt, groups; };

// Cut the wide parts into items.  A part of xt tiles takes items of
// per(c, xt) 32-term groups, c for four tiles and proportionally more for
// fewer, a multiple of the workgroup's waves; c is chosen by the modelled
// completion time on n_cu compute units (one workgroup each, items taken
// largest first), an item costing its critical wave's (group x tile) count
// plus one for staging lambda.  Items are emitted largest first.
void wide_items(const std::vector<WidePart> &parts, int n_cu, std::vector<jam::Item> &out) {
  out.clear();
  if (parts.empty()) return;
  constexpr int kWW = jam::kWideWaves;
  int64_t tot = 0;
  for (const WidePart &w : parts) tot += (int64_t)w.xt * w.groups;
  const int64_t share = std::max<int64_t>(1, (tot / 4 + n_cu - 1) / std::max(1, n_cu));
  auto per_of = [](int64_t c, int xt) {
    constexpr int64_t w = jam::kWideWaves;
    return (int)std::max<int64_t>(w, (c * 4 / xt + w - 1) / w * w);
  };
  auto cost_of = [](int ng, int xt) {
    constexpr int w = jam::kWideWaves;
    return (double)((ng + w - 1) / w) * xt + 1.0;
  };
  const int64_t step = std::max<int64_t>(kWW, share / 64 / kWW * kWW);
  int64_t best = kWW;
  double best_t = -1.0;
  std::vector<double> cost;
  for (int64_t c = std::max<int64_t>(kWW, share / 4 / kWW * kWW); c <= 2 * share + kWW; c += step) {
    cost.clear();
    for (const WidePart &w : parts) {
      const int per = per_of(c, w.xt);
      for (int g0 = 0; g0 < w.groups; g0 += per) cost.push_back(cost_of(std::min(per, w.groups - g0), w.xt));
    }
    const double t = list_schedule_makespan(cost, n_cu);
    if (best_t < 0.0 || t < best_t) { best = c; best_t = t; }
  }
  cost.clear();
  for (const WidePart &w : parts) {
    const int per = per_of(best, w.xt);
    for (int g0 = 0; g0 < w.groups; g0 += per) {
      const int g1 = std::min(w.groups, g0 + per);
      out.push_back({w.m, w.pt | (w.xt << 16), g0, g1});
      cost.push_back(cost_of(g1 - g0, w.xt));
    }
  }
  sort_by_cost(out, cost);
}

// Panels of tracer k that reach a tile of the compressed form's map, and
// every tile's total over the tracers.
int cheb_reach(const GeomHost &g, int k, int tile) {
  const int ntx = (g.n_ux + 31) / 32, nty = (g.n_uy + 31) / 32;
  return std::min(g.cheb_px[(size_t)k * ntx + tile % ntx], g.cheb_py[(size_t)k * nty + tile / ntx]);
}
template <typename F>
void for_cheb_tiles(const GeomHost &g, F f) {
  const int tiles = ((g.n_ux + 31) / 32) * ((g.n_uy + 31) / 32);
  for (int t = 0; t < tiles; ++t) {
    int units = 0;
    for (int k = 0; k < g.K; ++k) units += cheb_reach(g, k, t);
    f(t, units);
  }
}

constexpr double kShareTerms = 512.0;

// Which models of a batch take the compressed form: of direct, all and those that gain
// the choice with the least modelled time, for the forward and the adjoint.  All: the
// forward has one launch more than the direct one and, in a few models, fewer workgroups
// to hide its latency, which costs kChebLatencyNs, the less the longer the direct call is
// (a decay over kChebLatencyOver): one model of 102 x 102 distinct pixels, 16 x 31 x 112
// terms takes 45.7 us compressed and 49.3 direct, 66 x 66 with 12 x 61 x 128 terms 51.6
// and 50.3; 300 models of 34 x 36, 3 x 14 x 160 terms 153 and 169, 72 of 72 x 43, 20 x
// 10 x 120 terms 220 and 224.  The direct adjoint's two launches are the longer ones of
// a small batch (6 models of 86 x 86, 7 x 8 x 70 terms: 77 us, 107 direct), worth
// kChebAdjNs.  Beside other models' launches, one after the other, with their tails, the
// form's own cost kChebBesideNs and kChebBesideAdjNs: 63 models of 67 to 203 pixels a
// side, 5 x 8 x 90 terms, adjoint 317 us direct, 226 compressed and 411 with those
// compressed that gain.  Another pair of forward launches for another group of models
// takes kChebGroupNs (160 models of 68 x 68, 10 x 13 x 100 terms: one group 276 us, eight
// 531).
constexpr double kChebLatencyNs = 15000.0;
constexpr double kChebLatencyOver = 30000.0;
constexpr double kChebAdjNs = 5000.0;
constexpr double kChebBesideNs = 20000.0;
constexpr double kChebBesideAdjNs = 80000.0;
constexpr double kChebGroupNs = 36000.0;
struct ChebBatch {
  double all = 0.0, some = 0.0, direct = 0.0;   // gain on the whole chip; the direct cost
  bool every = true, small = false;             // every larger map has the tables; small maps
};
ChebBatch cheb_batch(const jam_ctx *ctx, int n, const int32_t *geom_idx, bool adjoint) {
  ChebBatch b;
  for (int m = 0; m < n; ++m) {
    const GeomHost &g = ctx->gh[geom_idx[m]];
    if (g.cheb_np > 0) {
      const double gain = g.cheb_gain[adjoint] / (4.0 * ctx->n_cu);
      b.all += gain;
      b.some += std::max(0.0, gain);
      b.direct += g.cheb_direct / (4.0 * ctx->n_cu);
    } else if (g.n_ux <= kSmallMap && g.n_uy <= kSmallMap && g.J1 <= jam::kSmallAdjMass) {
      b.small = true;
    } else {
      b.every = false;
    }
  }
  return b;
}
int choose_cheb(const jam_ctx *ctx, int n, const int32_t *geom_idx, const Tune &t) {
  if (t.rule != 1 || ctx->opt.alignment == 1 || ctx->opt.form == 2) return 0;
  int forms = 0;
  for (const bool adjoint : {false, true}) {
    const ChebBatch b = cheb_batch(ctx, n, geom_idx, adjoint);
    const double beside = adjoint ? kChebBesideAdjNs : kChebBesideNs;
    double all = adjoint ? b.all + kChebAdjNs
                         : b.all - (b.small ? kChebBesideNs
                                            : kChebLatencyNs * std::exp(-b.direct / kChebLatencyOver));
    if (!b.every || b.direct == 0.0) all = 0.0;
    const double some = b.some - beside;
    if (std::max(all, some) <= 0.0) continue;
    if (all >= some)
      forms |= adjoint ? kChebAdjAll : kChebFwdAll;
    else
      forms |= adjoint ? kChebAdjGain : kChebFwdGain;
  }
  return forms;
}

// The tilings of a batch's maps, by geometry (n_models of each in the batch; gran
// as in the plan).  A model may run in any tiling at least as large as its map, with
// the same sums, or in the 32 x 32 blocks' kernel, which is launched anyway where
// others need it.  In place: the set of tilings with the least time over all
// launches.  From the table: then each tiling that lowers it further.
// Measured, models of 13000 terms on maps of 8 .. 32 pixels a side drawn at random,
// forward call, a launch for every tiling / this: 16 models 64 / 26 us, 256 705 /
// 124, 1024 903 / 424.
std::vector<SmallTiles> choose_tilings(const jam_ctx *ctx, const std::vector<int> &n_models,
                                       const Tune &tune) {
  const size_t ng = ctx->gh.size();
  std::vector<SmallTiles> out(ng);
  LaunchLoad blocks;                           // what has no choice
  std::vector<LaunchLoad> place(9 * 10);       // in place: [own tiling][tiling, or 9 the blocks]
  std::vector<LaunchLoad> table(9), table_blocks(9);
  bool used[9] = {};
  for (size_t i = 0; i < ng; ++i) {
    if (!n_models[i]) continue;
    const GeomHost &g = ctx->gh[i];
    const NumChoice c = choose_numerator(g, tune, tune.gran);
    if (c.kind != 2) continue;
    const SmallTiles s = out[i] = small_tiles(g, c, tune.tau);
    const double items = (double)n_models[i] * c.n_slices, terms = (double)g.T / c.n_slices;
    LaunchLoad b;
    for (const WaveTile &t : c.tiles)
      b.add(items, terms * (block_ns(t.BX, t.BY) + (c.gen ? kTermInPlaceNs : 0.0)));
    if (s.tiling < 0) {
      blocks.add(b);
    } else if (s.tiling < 9) {
      used[s.tiling] = true;
      for (int t = 0; t < 9; ++t)
        place[10 * s.tiling + t].add(items, terms * (tiles_ns(t / 3, t % 3) + kTermInPlaceNs));
      place[10 * s.tiling + 9].add(b);
    } else {
      table[s.tiling - 9].add(items * s.nx * s.ny, terms * tiles_ns((s.tiling - 9) / 3, s.tiling % 3));
      table_blocks[s.tiling - 9].add(b);
    }
  }
  // in place: every set of tilings, each kind in the cheapest of the set that holds it
  int present = 0;
  for (int t = 0; t < 9; ++t) present |= used[t] << t;
  double best = 1e300;
  int to[9];
  LaunchLoad best_blocks = blocks;
  for (int set = 0; set < 512; ++set) {
    if (set & ~present) continue;              // a larger tiling than any kind's own is never cheaper
    LaunchLoad load[10];
    load[9] = blocks;
    int at[9];
    for (int k = 0; k < 9; ++k) {
      if (!used[k]) continue;
      at[k] = 9;
      for (int t = 0; t < 9; ++t)
        if ((set >> t & 1) && t / 3 >= k / 3 && t % 3 >= k % 3 &&
            place[10 * k + t].sum < place[10 * k + at[k]].sum)
          at[k] = t;
      load[at[k]].add(place[10 * k + at[k]]);
    }
    double ns = 0.0;
    for (const LaunchLoad &l : load) ns += l.ns(ctx->n_cu);
    if (ns < best) {
      best = ns;
      best_blocks = load[9];
      std::copy(at, at + 9, to);
    }
  }
  // from the table
  bool keep[9];
  for (int t = 0; t < 9; ++t) {
    LaunchLoad with = best_blocks;
    for (int o = t + 1; o < 9; ++o) with.add(table_blocks[o]);
    LaunchLoad merged = with;
    merged.add(table_blocks[t]);
    keep[t] = table[t].ns(ctx->n_cu) + with.ns(ctx->n_cu) < merged.ns(ctx->n_cu);
    if (!keep[t]) best_blocks.add(table_blocks[t]);
  }
  for (SmallTiles &s : out) {
    if (s.tiling >= 9)
      s.tiling = keep[s.tiling - 9] ? s.tiling : -1;
    else if (s.tiling >= 0)
      s.tiling = to[s.tiling] == 9 ? -1 : to[s.tiling];
  }
  return out;
}

// The y quads of the small maps' adjoint kernel that each number of quads runs in
// (at least as many; the padding adds zeros): the partition of the quads into runs
// with the least time over the launches.  Per term 21 (12 x 12 pixels) to 64 ns (32
// x 32) of one SIMD, fitted; with six quads and more two waves a SIMD for three.
// The batches above, chi^2 and gradient, a launch for every number of quads (and
// every tiling) / this: 256 models 1416 / 361 us, 1024 2107 / 1236.
struct AdjKind {
  double terms = 0.0, longest = 0.0, x_terms = 0.0;   // x_terms: terms times quads of x
};
void choose_quads(int n_cu, const AdjKind (&kinds)[jam::kSmallQuads + 1],
                  int (&to)[jam::kSmallQuads + 1]) {
  constexpr int Q = jam::kSmallQuads;
  double best[Q + 1] = {};       // of the quads up to q
  int first[Q + 1] = {};
  for (int q = 1; q <= Q; ++q) {
    best[q] = 1e300;
    const double f = q > 5 ? 1.15 : 1.0;
    LaunchLoad l;
    for (int p = q; p >= 1; --p) {             // one launch of q for p .. q
      const AdjKind &k = kinds[p];
      if (k.terms > 0.0) {
        const double per = f * (12.0 + 0.45 * q + (0.75 + 0.55 * q) * k.x_terms / k.terms);
        l.sum += k.terms * per;
        l.longest = std::max(l.longest, k.longest * per);
      }
      const double ns = best[p - 1] + l.ns(n_cu);
      if (ns < best[q]) {
        best[q] = ns;
        first[q] = p;
      }
    }
  }
  for (int q = Q; q >= 1; q = first[q] - 1)
    for (int p = first[q]; p <= q; ++p) to[p] = q;
}

// h_limit: a group of compressed models is closed once its H takes this many
// doubles (a single model's is never split).
jam_status build_plan(jam_ctx *ctx, int32_t n, const int32_t *geom_idx, const Tune &tune_in,
                      std::unique_ptr<Plan> &out, int64_t h_limit = INT64_MAX) {
  auto p = std::make_unique<Plan>();
  p->key.assign(geom_idx, geom_idx + n);
  p->n = n;
  p->tune = tune_in;
  if (p->tune.cheb < 0) p->tune.cheb = choose_cheb(ctx, n, geom_idx, p->tune);
  if (p->tune.gran <= 0) p->tune.gran = default_gran(ctx, n, geom_idx, p->tune);
  const Tune &tune = p->tune;
  std::vector<jam::ModelDev> md(n);
  std::vector<jam::Item> it_terms, it_pix, it_num, it_bins, it_maps, it_chain, it_sens, it_sb,
      it_red, it_sph, it_pro, it_adj, it_sensw, it_sgrid, it_sgred, it_sgred3, it_pcot,
      it_pfix, it_sgs, it_sphm, it_ptab, it_srow, it_numsm, it_cpan, it_csum, it_cadj, it_ctmap, it_crows, it_sbpro;
  std::vector<jam::ChebItem> it_cmap;
  std::vector<double> c_num, c_sens, c_sensw;
  // wide-sensitivity parts (model, part, x tiles, 32-term groups); their
  // items are cut after the model loop (wide_items)
  std::vector<WidePart> wide_parts;
  int64_t gauss = 0, terms = 0, pixd = 0, part = 0, bins = 0, sens = 0, sph = 0, sbp = 0,
          sgrid = 0, sgrid3 = 0, sgcot = 0, pol = 0, terms64 = 0;
  const bool spherical = ctx->opt.alignment == 1;
  // compressed form: units per map item, two items per compute unit where
  // the batch is small enough (a unit on a tile is 16 FP64 MFMAs of a wave)
  auto fwd_cheb = [&](const GeomHost &g) { return takes_cheb(g, tune.cheb, false); };
  auto adj_cheb = [&](const GeomHost &g) { return takes_cheb(g, tune.cheb, true); };
  int64_t cheb_units = 0, cheb_panels = 0, cadj_panels = 0;
  int cheb_most = 0;   // terms of the largest panel
  int64_t small_terms = 0;
  for (int m = 0; m < n; ++m) {
    const GeomHost &g = ctx->gh[geom_idx[m]];
    if (g.n_ux <= kSmallMap && g.n_uy <= kSmallMap) small_terms += g.T;
    if (fwd_cheb(g)) {
      for_cheb_tiles(g, [&](int, int units) { cheb_units += units; });
      cheb_panels += (int64_t)g.K * g.cheb_np;
    }
    if (adj_cheb(g)) cadj_panels += (int64_t)g.K * g.cheb_np;
    for (int P = 0; P < g.cheb_np; ++P) cheb_most = std::max(cheb_most, g.cheb_ptr[P + 1] - g.cheb_ptr[P]);
  }
  // terms per item of the small maps' adjoint: at least two items per compute
  // unit down to one pass of a block
  const int adj_terms = (int)std::max<int64_t>(256, std::min<int64_t>(8192, small_terms / (2 * ctx->n_cu)));
  const int cheb_per = (int)std::max<int64_t>(
      16, std::min<int64_t>(160, (cheb_units + 2 * ctx->n_cu - 1) / (2 * ctx->n_cu)));
  // A block's waves share a unit whose panel has more than kShareTerms
  // terms, and every unit of a batch too small to give each SIMD one (eight
  // waves then, where a panel has enough terms for them).
  const bool share_f = cheb_panels <= 4 * (int64_t)ctx->n_cu, share_a = cadj_panels <= 4 * (int64_t)ctx->n_cu;
  p->cheb_waves = share_f && cheb_most > 512 ? 8 : 4;
  p->cadj_waves = share_a && cheb_most > 512 ? 8 : 4;
  int64_t cheb_h = 0, cheb_hmax = 0, cheb_t = 0;
  std::vector<double> c_cpan, c_cadj;
  it_cpan.reserve(cheb_panels);
  c_cpan.reserve(cheb_panels);
  it_cadj.reserve(cadj_panels);
  c_cadj.reserve(cadj_panels);
  Plan::ChebGroup grp{};
  // shared items first, largest first, then the others as they come
  // (a large batch has 1e5 units and mostly none shared: they stay as they are)
  auto order_units = [&](std::vector<jam::Item> &v, std::vector<double> &cost, int first) {
    int shared = 0;
    for (size_t i = first; i < v.size(); ++i) shared += v[i].c & 1;
    if (shared == 0) return 0;
    std::vector<jam::Item> sub, rest;
    std::vector<double> cs;
    sub.reserve(shared);
    rest.reserve(v.size() - first - shared);
    for (size_t i = first; i < v.size(); ++i) {
      if (v[i].c & 1) {
        sub.push_back(v[i]);
        cs.push_back(cost[i]);
      } else {
        rest.push_back(v[i]);
      }
    }
    sort_by_cost(sub, cs);
    std::copy(sub.begin(), sub.end(), v.begin() + first);
    std::copy(rest.begin(), rest.end(), v.begin() + first + sub.size());
    return (int)sub.size();
  };
  auto close_group = [&]() {
    grp.pan1 = (int)it_cpan.size();
    grp.map1 = (int)it_cmap.size();
    if (grp.pan1 > grp.pan0 || grp.map1 > grp.map0) {
      grp.pan_share = order_units(it_cpan, c_cpan, grp.pan0);
      std::stable_sort(it_cmap.begin() + grp.map0, it_cmap.end(),
                       [](const jam::ChebItem &a, const jam::ChebItem &b) { return a.count > b.count; });
      p->cheb_groups.push_back(grp);
    }
    grp.pan0 = grp.pan1;
    grp.map0 = grp.map1;
    cheb_hmax = std::max(cheb_hmax, cheb_h);
    cheb_h = 0;
  };
  // spherical forward: the potential grid (form 1: sums at every node)
  const bool use_sgrid = spherical && ctx->opt.form != 1;
  std::vector<SmallTiles> tiles_of;
  if (!spherical) {
    std::vector<int> models(ctx->gh.size(), 0);
    for (int m = 0; m < n; ++m) ++models[geom_idx[m]];
    tiles_of = choose_tilings(ctx, models, tune);
  }
  for (int m = 0; m < n; ++m) {
    const int gi = geom_idx[m];
    const GeomHost &g = ctx->gh[gi];
    jam::ModelDev &d = md[m];
    std::memset(&d, 0, sizeof d);
    d.geom = gi;
    d.lum_off = (int)p->total_lum;
    d.mass_off = (int)p->total_mass;
    d.out_off = (int)p->total_bins;
    const NumChoice nc = choose_numerator(g, tune, tune.gran);
    d.n_slices = nc.n_slices;
    const bool small = !spherical && nc.gen;
    const bool cheb = !spherical && nc.kind == 5, cadj = adj_cheb(g);
    d.form = nc.kind == 0 ? 1 : (cheb ? 5 : (small ? 3 : 2));
    // adjoint sensitivity blocks: one (per-pixel), none (small map), one per
    // x tile (one tile), one per part of up to four x tiles (wide)
    // (the wide form pays off where each term group runs over many y steps:
    // its per-group epilogue and accumulator set-up are fixed costs)
    const int n_xt = (g.n_ux + 31) / 32;
    const bool wide = !spherical && !small && !cadj && d.form != 1 && n_xt >= 2 && g.n_uy >= kWideMinY;
    d.n_sens_parts = d.form == 1 ? 1 : (small || cadj ? 0 : (wide ? (n_xt + 3) / 4 : n_xt));
    d.n_xt = (g.n_ux + 31) / 32;
    d.n_yt = (g.n_uy + 31) / 32;
    d.gauss_off = gauss;
    d.term_off = terms;
    d.pix_off = pixd;
    d.part_off = part;
    d.map_off = p->total_map;
    d.sens_off = sens;
    d.bin_off = bins;
    d.sph_off = sph;
    d.sbp_off = sbp;
    sbp += (int64_t)g.K * jam::sb_tiles(g.n_ux, g.n_uy);
    if (spherical) {
      sph += (int64_t)jam::kSphNR * jam::kSphNT * 3;
      if (!use_sgrid)
        for (int q = 0; q < jam::kSphCells; ++q) it_sph.push_back({m, q, 0, 0});
      for (int q = 0; q < jam::kSphCells / 64; ++q) it_srow.push_back({m, q, 0, 0});
      // moments at the nodes: four table points (a wave each)
      if (!use_sgrid)
        for (int q = 0; q < jam::kSphCells / 4; ++q) it_sphm.push_back({m, q, 0, 0});
    }
    if (use_sgrid) {
      const int64_t pts = (int64_t)jam::kPolN * jam::kPolC;
      const int sl = jam::pol_slices(jam::sph_terms_padded(g.J1, g.n_u));
      d.sgrid_slices = sl;
      d.sgrid_off = sgrid;
      d.sgrid3_off = sgrid3;
      d.pol_off = pol;
      sgrid += sl * 2 * pts;
      sgrid3 += sl * (int64_t)jam::kPolAdjGrid;
      pol += jam::pol_size(g.K);
      for (int q = 0; q < jam::pol_groups(g.K) * jam::kSphNR / 4; ++q) it_sphm.push_back({m, q, 0, 0});
      for (int q = 0; q < jam::kSphCells / 16; ++q) it_ptab.push_back({m, q, 0, 0});
      for (int row = 0; row < jam::kPolN / 4; ++row)
        for (int q = 0; q < sl; ++q) it_sgrid.push_back({m, row, q, 0});
      if (sl > 1) {
        for (int b = 0; b < 2 * pts / 1024; ++b) it_sgred.push_back({m, b, 0, 0});
        for (int b = 0; b < pts / 256; ++b) it_sgred3.push_back({m, b, 0, 0});
      }
    }
    gauss += jam::gauss_size(g.K, g.J1);
    const int tsph = jam::sph_terms_padded(g.J1, g.n_u);
    // spherical: float4 terms, then floats; small maps compute their terms in
    // place; cylindrical tables are zero-padded to a multiple of 32 terms
    d.term64_off = terms64;
    if (spherical) terms64 += (int64_t)tsph * jam::kSphTermDoubles;
    terms += spherical ? tsph + tsph / 4 : (small || (cheb && cadj) ? 0 : jam::padded_terms(g.T));
    pixd += 4 * (int64_t)g.n_pix;
    part += part_size(g, nc);
    const int np = g.cheb_np;
    if (cheb || cadj)
      for (int k = 0; k < g.K; ++k)
        for (int P = 0; P < np; ++P) {
          const int nyt = g.cheb_h[k * np + P + 1] - g.cheb_h[k * np + P];
          const double terms_p = g.cheb_ptr[P + 1] - g.cheb_ptr[P];
          if (cheb && nyt > 0) {
            it_cpan.push_back({m, k, P, share_f || terms_p > kShareTerms});
            c_cpan.push_back(terms_p + 40.0 * nyt);
          }
          if (cadj) {
            // a small batch's long panels in slices of one chunk per wave
            const int sl = share_a ? (int)std::min(1024.0, std::ceil(terms_p / (64.0 * p->cadj_waves))) : 1;
            for (int q = 0; q < sl; ++q) {
              it_cadj.push_back({m, k, P, (share_a || terms_p > kShareTerms) | q << 1 | sl << 16});
              c_cadj.push_back(terms_p / sl + 30.0 * nyt);
            }
          }
        }
    if (cheb) {
      const int64_t hm = (int64_t)g.cheb_h.back() * 512;
      d.cheb_off = cheb_h;
      cheb_h += hm;
      p->n_cheb++;
      // runs of equal length, a multiple of four units (four waves share one)
      int slot = 0;
      for_cheb_tiles(g, [&](int tile, int units) {
        const int s0 = slot, runs = (units + cheb_per - 1) / cheb_per;
        const int len = runs ? ((units + runs - 1) / runs + 3) / 4 * 4 : 0;
        // a run starts at unit at = 0, len, 2 len, ... of the tile
        for (int k = 0, first = 0, at = 0; at < units; ++k) {
          const int reach = cheb_reach(g, k, tile);
          for (; at < first + reach; at += len)
            it_cmap.push_back({m, tile, k, at - first, std::min(len, units - at), slot++});
          first += reach;
        }
        for (int q = 0; q < 4; ++q) it_csum.push_back({m, 4 * tile + q, s0, slot - s0});
      });
      part += (int64_t)slot * 1024;
      if (cheb_h >= h_limit) close_group();
    }
    if (cadj) {
      d.chebt_off = cheb_t;
      cheb_t += (int64_t)g.cheb_h.back() * 512;
      for (int ty = 0; ty < d.n_yt; ++ty)
        for (int k = 0; k < g.K; ++k)
          if (cheb_reach(g, k, ty * d.n_xt) > 0) it_ctmap.push_back({m, ty, k, 0});
      for (int k = 0; k < g.K; ++k)
        for (int jb = 0; jb < (g.J1 + 63) / 64; ++jb) it_crows.push_back({m, k, jb, 0});
    }
    bins += 2 * (int64_t)g.n_bins;
    if (spherical) {
      // term sensitivities: point ranges, or (with the potential grid) parts
      // of the grid rows
      d.n_sens_parts = use_sgrid ? jam::kPolParts : jam::sph_ranges(g.K);
      sens += jam::sph_adj_size(g.K, g.n_pix, tsph, d.n_sens_parts);
    } else {
      sens += 3 * (int64_t)d.n_sens_parts * g.T + (int64_t)g.K * 3 * g.J1 +
              (cadj ? 3 * (int64_t)g.K * g.cheb_pieces : 0);
    }
    p->total_lum += g.K;
    p->total_mass += g.J;
    p->total_bins += g.n_bins;
    p->total_map += (int64_t)g.nxp * g.nyp;
    if (!small && !(cheb && cadj))
      for (int tb = 0; tb < ((spherical ? tsph : g.T) + 255) / 256; ++tb)
        it_terms.push_back({m, tb, 0, 0});
    if (spherical && use_sgrid) {
      d.sgcot_off = sgcot;
      sgcot += jam::pol_cot_size(g.K);
      // from the outer rows in: they hold more nodes (the rules of all radii
      // inside reach them), and the short items then fill the tail
      for (int b = jam::kPolBins - 1; b >= 0; --b)
        for (int q = 0; q < jam::pol_cot_groups(g.K); ++q) it_pcot.push_back({m, b, q, 0});
      for (int b = 0; b < jam::kPolN * jam::kPolC / 256; ++b) it_pfix.push_back({m, b, 0, 0});
      for (int tb = 0; tb < (tsph + 511) / 512; ++tb)
        for (int ip = 0; ip < jam::kPolParts; ++ip) it_sgs.push_back({m, tb, ip, 0});
    } else if (spherical) {
      for (int tt = 0; tt < (tsph + 255) / 256; ++tt)
        for (int r = 0; r < d.n_sens_parts; ++r) {
          it_sens.push_back({m, tt, r, 0});
          c_sens.push_back((double)jam::sph_range_len(g.K, d.n_sens_parts));
        }
    } else if (cadj) {
      // it_cadj
    } else if (small) {
      // fused sensitivities + chain: items of whole tracers, about 8192 terms
      // each, or in a batch too small to give the chip that many, of whole rows
      // of one tracer
      const int row_terms = g.n_u, quads = (g.n_uy + 3) / 4;
      const int whole = std::max(512, adj_terms);
      if (whole >= g.J1 * row_terms) {
        const int per = std::max(1, std::min(jam::kSmallAdjTracers, whole / (g.J1 * row_terms)));
        for (int k = 0; k < g.K; k += per) {
          const int k1 = std::min(g.K, k + per);
          it_adj.push_back({m, k | (k1 << 16), ((k1 - k) * g.J1) << 16, quads});
        }
      } else {
        const int per = std::max(1, adj_terms / row_terms);
        for (int k = 0; k < g.K; ++k)
          for (int r = 0; r < g.J1; r += per)
            it_adj.push_back({m, k | ((k + 1) << 16), r | (std::min(g.J1, r + per) << 16), quads});
      }
    } else if (d.form == 1) {
      for (int tb = 0; tb < (g.T + 255) / 256; ++tb) {
        it_sens.push_back({m, tb, 0, 0});
        c_sens.push_back((double)g.n_pix);
      }
    } else if (wide) {
      // parts of up to four x tiles
      for (int pt = 0; pt < d.n_sens_parts; ++pt)
        wide_parts.push_back({m, pt, std::min(4, n_xt - 4 * pt), (g.T + 31) / 32});
    } else {
      for (int xt = 0; xt < d.n_sens_parts; ++xt)
        for (int tt = 0; tt < (g.T + jam::kSensTerms - 1) / jam::kSensTerms; ++tt) {
          it_sens.push_back({m, xt, tt, 1});
          c_sens.push_back(8.0 * 32.0 * g.n_uy);
        }
    }
    for (int pb = 0; pb < (g.n_pix + 255) / 256; ++pb) it_pix.push_back({m, pb, 0, 0});
    // the compressed form's maps are summed by k_cheb_sum, a single slice of a
    // matrix-core form is the sum
    const SmallTiles tiles = spherical ? SmallTiles() : tiles_of[gi];
    if (spherical || (!cheb && !(d.n_slices == 1 && nc.kind == 2)))
      for (int pb = 0; pb < (g.n_pix + 63) / 64; ++pb) it_red.push_back({m, pb, 0, 0});
    for (int rb = 0; rb < (g.n_uy + 7) / 8; ++rb)
      for (int cb = 0; cb < (g.n_ux + 63) / 64; ++cb) {
        it_sb.push_back({m, rb, cb, 0});
        if (!cheb) it_sbpro.push_back({m, rb, cb, 0});
      }
    if (tiles.tiling >= 0)
      for (int s = 0; s < d.n_slices; ++s)
        for (int ty = 0; ty < tiles.ny; ++ty)
          for (int tx = 0; tx < tiles.nx; ++tx)
            it_numsm.push_back({m, tx * tiles.w | (ty * tiles.h << 16), s, tiles.tiling});
    for (int s = 0; s < d.n_slices && tiles.tiling < 0; ++s)
      for (int tl = 0; tl < nc.n_tiles(); ++tl) {
        if (nc.kind == 0) {
          it_num.push_back({m, tl, s, 0});
        } else {
          const WaveTile &w = nc.tiles[tl];
          it_num.push_back({m, w.bx | (w.by << 16), s,
                            small ? 6 : 2 + (w.BX - 1) + 2 * (w.BY - 1)});
        }
        c_num.push_back(num_item_cost(g, nc, s, tl));
      }
    if (g.max_bin_nnz <= kBinWaveNnz)
      for (int b = 0; b < g.n_bins; b += 4) it_bins.push_back({m, b, 0, 1});
    else
      for (int b = 0; b < g.n_bins; ++b) it_bins.push_back({m, b, 0, 0});
    for (int r = 0; r < g.nyp; ++r) it_maps.push_back({m, r, 0, 0});
    if (!spherical && !small && !cadj)
      for (int k = 0; k < g.K; ++k)
        for (int jb = 0; jb < (g.J1 + 3) / 4; ++jb) it_chain.push_back({m, k, jb, 0});
  }
  close_group();
  p->cadj_share = order_units(it_cadj, c_cadj, 0);
  if (p->total_bins > INT32_MAX || p->total_lum > INT32_MAX || p->total_mass > INT32_MAX)
    return fail(JAM_E_UNSUPPORTED, "batch too large");
  // prologue of the cylindrical model: a few models run set-up, terms and
  // surface brightness in one launch (terms from the parameters); many run
  // the set-up first and then terms from its table beside the tiles
  p->fused_prologue = n <= kFusedPrologueModels;
  if (p->fused_prologue)
    for (int m = 0; m < n; ++m) it_pro.push_back({m, 0, 0, 0});
  // (last the terms of models that only the adjoint sums directly)
  auto push_terms = [&](bool compressed) {
    for (const jam::Item &t : it_terms)
      if (spherical || (md[t.m].form == 5) == compressed)
        it_pro.push_back({t.m, t.a, 0, p->fused_prologue ? 1 : 3});
  };
  push_terms(false);
  for (const jam::Item &t : it_sbpro) it_pro.push_back({t.m, t.a, t.b, 2});
  p->n_pro_fwd = (int)it_pro.size();
  if (!spherical) push_terms(true);
  // bin items: the one-bin-per-wave ones first (a launch of 256-thread
  // blocks), then the one-bin-per-block ones (1024-thread blocks)
  std::stable_partition(it_bins.begin(), it_bins.end(), [](const jam::Item &t) { return t.c == 1; });
  p->n_bins_wave = (int)std::count_if(it_bins.begin(), it_bins.end(),
                                      [](const jam::Item &t) { return t.c == 1; });
  sort_by_cost(it_num, c_num);
  std::stable_sort(it_numsm.begin(), it_numsm.end(),
                   [](const jam::Item &a, const jam::Item &b) { return a.c < b.c; });
  AdjKind kinds[jam::kSmallQuads + 1];
  for (const jam::Item &t : it_adj) {
    const GeomHost &g = ctx->gh[geom_idx[t.m]];
    AdjKind &k = kinds[t.c];
    const double terms = (double)((t.b >> 16) - (t.b & 0xffff)) * g.n_u;
    k.terms += terms;
    k.x_terms += terms * ((g.n_ux + 3) / 4);
    k.longest = std::max(k.longest, terms);
  }
  int quads_to[jam::kSmallQuads + 1];
  choose_quads(ctx->n_cu, kinds, quads_to);
  for (jam::Item &t : it_adj) t.c = quads_to[t.c];
  std::stable_sort(it_adj.begin(), it_adj.end(),
                   [](const jam::Item &a, const jam::Item &b) { return a.c < b.c; });
  for (const jam::Item &t : it_adj) ++p->adj_ptr[t.c];
  for (int t = 0; t < jam::kSmallQuads; ++t) p->adj_ptr[t + 1] += p->adj_ptr[t];
  for (const jam::Item &t : it_numsm) ++p->numsm_ptr[t.c + 1];
  for (int t = 0; t < jam::kSmallTilings; ++t) p->numsm_ptr[t + 1] += p->numsm_ptr[t];
  sort_by_cost(it_sens, c_sens);
  wide_items(wide_parts, ctx->n_cu, it_sensw);

  constexpr int kLists = 28;
  std::vector<jam::Item> *lists[kLists] = {&it_terms, &it_pix, &it_num, &it_bins,
                                           &it_maps,  &it_chain, &it_sens, &it_sb,
                                           &it_red,   &it_sph, &it_pro, &it_adj,
                                           &it_sensw, &it_sgrid, &it_sgred, &it_sgred3,
                                           &it_pcot,  &it_pfix,  &it_sgs,  &it_sphm, &it_ptab, &it_srow, &it_numsm, &it_cpan,
                                           &it_csum,  &it_cadj,  &it_ctmap, &it_crows};
  if (it_cmap.size() > (size_t)INT32_MAX) return fail(JAM_E_UNSUPPORTED, "batch too large");
  for (auto *l : lists)
    if (l->size() > (size_t)INT32_MAX) return fail(JAM_E_UNSUPPORTED, "batch too large");
  // one device arena: models then the item lists
  size_t off = 0;
  const size_t o_models = off;
  off = align256(off + sizeof(jam::ModelDev) * n);
  size_t o_it[kLists];
  for (int i = 0; i < kLists; ++i) {
    o_it[i] = off;
    off = align256(off + sizeof(jam::Item) * std::max<size_t>(1, lists[i]->size()));
  }
  const size_t o_cmap = off;
  off = align256(off + sizeof(jam::ChebItem) * std::max<size_t>(1, it_cmap.size()));
  const std::unique_ptr<char[]> stage(new char[off]);   // what lies between the lists is not read
  if (!it_cmap.empty())
    std::memcpy(stage.get() + o_cmap, it_cmap.data(), sizeof(jam::ChebItem) * it_cmap.size());
  std::memcpy(stage.get() + o_models, md.data(), sizeof(jam::ModelDev) * n);
  for (int i = 0; i < kLists; ++i)
    if (!lists[i]->empty())
      std::memcpy(stage.get() + o_it[i], lists[i]->data(), sizeof(jam::Item) * lists[i]->size());
  HIP_TRY(hipMalloc(&p->arena, off));
  HIP_TRY(hipMemcpy(p->arena, stage.get(), off, hipMemcpyHostToDevice));
  char *base = (char *)p->arena;
  p->d_models = (jam::ModelDev *)(base + o_models);
  jam::Item **dl[kLists] = {&p->d_terms, &p->d_pix,  &p->d_num, &p->d_bins,
                            &p->d_maps,  &p->d_chain, &p->d_sens, &p->d_sb,
                            &p->d_red,   &p->d_sph,   &p->d_pro,  &p->d_adj,
                            &p->d_sensw, &p->d_sgrid, &p->d_sgred, &p->d_sgred3,
                            &p->d_pcot,  &p->d_pfix,  &p->d_sgs,  &p->d_sphm, &p->d_ptab, &p->d_srow, &p->d_numsm, &p->d_cpan,
                            &p->d_csum,  &p->d_cadj,  &p->d_ctmap, &p->d_crows};
  p->d_cmap = (jam::ChebItem *)(base + o_cmap);
  p->n_cmap = (int)it_cmap.size();
  int *cnt[kLists] = {&p->n_terms, &p->n_pix,  &p->n_num, &p->n_bins,
                      &p->n_maps,  &p->n_chain, &p->n_sens, &p->n_sb,
                      &p->n_red,   &p->n_sph,   &p->n_pro,  &p->n_adj,
                      &p->n_sensw, &p->n_sgrid, &p->n_sgred, &p->n_sgred3,
                      &p->n_pcot,  &p->n_pfix,  &p->n_sgs,  &p->n_sphm, &p->n_ptab, &p->n_srow, &p->n_numsm, &p->n_cpan,
                      &p->n_csum,  &p->n_cadj,  &p->n_ctmap, &p->n_crows};
  for (int i = 0; i < kLists; ++i) {
    *dl[i] = (jam::Item *)(base + o_it[i]);
    *cnt[i] = (int)lists[i]->size();
  }
  const int num_wg = p->n_num;   // one workgroup per numerator item
  if (tune.launch == 1) {
    const int occ = tune.rule == 0 ? ctx->occ_num_pix : ctx->occ_num_mfma;
    p->grid_num = std::max(1, std::min(num_wg, ctx->n_cu * occ));
    p->grid_sens = std::max(1, std::min(p->n_sens, ctx->n_cu * ctx->occ_sens));
  } else {
    p->grid_num = std::max(1, num_wg);
    p->grid_sens = std::max(1, p->n_sens);
  }
  // workspace layout
  size_t w = 0;
  p->off_status = w; w = align256(w + sizeof(int) * n);
  p->off_queue = w;  w = align256(w + sizeof(int) * 2);
  p->off_gauss = w;  w = align256(w + sizeof(double) * gauss);
  p->off_terms = w;  w = align256(w + sizeof(float4) * terms);
  p->off_pix = w;    w = align256(w + sizeof(double) * pixd);
  p->off_part = w;   w = align256(w + sizeof(double) * part);
  p->off_bins = w;   w = align256(w + sizeof(double) * bins);
  p->off_vfwd = w;   w = align256(w + sizeof(double) * p->total_bins);
  p->off_sph = w;    w = align256(w + sizeof(double) * sph);
  p->off_sgrid = w;  w = align256(w + sizeof(float) * sgrid);
  p->off_pol = w;    w = align256(w + sizeof(double) * pol);
  p->off_cheb = w;   w = align256(w + sizeof(double) * cheb_hmax);
  p->ws_fwd = w;
  p->spherical = spherical;
  p->off_sens = w;   w = align256(w + sizeof(double) * sens);
  p->off_vtmp = w;   w = align256(w + sizeof(double) * p->total_bins);
  p->off_cot = w;    w = align256(w + sizeof(double) * p->total_bins);
  p->off_sbp = w;    w = align256(w + sizeof(double) * sbp);
  p->off_terms64 = w; w = align256(w + sizeof(double) * terms64);
  p->off_sgrid3 = w; w = align256(w + sizeof(double) * sgrid3);
  p->off_sgcot = w;  w = align256(w + sizeof(double) * sgcot);
  p->off_chebt = w;  w = align256(w + sizeof(double) * cheb_t);
  p->ws_vjp = w;
  out = std::move(p);
  return JAM_OK;
}

jam::ParamsDev params_of(const jam_batch *b) {
  return jam::ParamsDev{b->inc, b->mass_scale, b->m_bh, b->beta, b->lum_I0, b->mass_S0};
}

// The numerator kernels of a cylindrical batch, up to the partial maps.
void launch_numerator(jam_ctx *ctx, Plan *p, char *ws, hipStream_t st) {
  const int *st_ws = (const int *)(ws + p->off_status);
  int *queue = p->tune.launch == 1 ? (int *)(ws + p->off_queue) : nullptr;
  const double *gauss = (const double *)(ws + p->off_gauss);
  const float4 *terms = (const float4 *)(ws + p->off_terms);
  double *part = (double *)(ws + p->off_part);
  double *H = (double *)(ws + p->off_cheb);
  for (const Plan::ChebGroup &q : p->cheb_groups) {
    if (q.pan1 > q.pan0)
      jam::launch_cheb_panel(ctx->d_geoms, p->d_models, p->d_cpan + q.pan0, q.pan1 - q.pan0,
                             q.pan_share, p->cheb_waves, gauss, st_ws, H, st);
    if (q.map1 > q.map0)
      jam::launch_cheb_map(ctx->d_geoms, p->d_models, p->d_cmap + q.map0, q.map1 - q.map0, H, st_ws,
                           part, st);
  }
  for (int t = 0; t < jam::kSmallTilings; ++t)
    if (p->numsm_ptr[t + 1] > p->numsm_ptr[t])
      jam::launch_num_small(ctx->d_geoms, p->d_models, p->d_numsm + p->numsm_ptr[t],
                            p->numsm_ptr[t + 1] - p->numsm_ptr[t], t, terms, gauss, st_ws, part,
                            (double *)(ws + p->off_pix), st);
  if (!p->n_num) return;
  jam::launch_num(ctx->d_geoms, p->d_models, p->d_num, p->n_num, terms, gauss, st_ws, part, (double *)(ws + p->off_pix), queue,
                    p->grid_num, p->tune.rule == 1, st);
}

// Set-up, term table and SB map; optionally the numerator map.  Leaves N and
// I in the workspace pix region.  adjoint: with the terms that only the adjoint reads.
void launch_forward_maps(jam_ctx *ctx, Plan *p, const jam::ParamsDev &pd, int32_t *status,
                         char *ws, hipStream_t st, bool need_numerator, bool capturing,
                         bool adjoint = false) {
  int *st_ws = (int *)(ws + p->off_status);
  int *queue = (int *)(ws + p->off_queue);
  double *gauss = (double *)(ws + p->off_gauss);
  float4 *terms = (float4 *)(ws + p->off_terms);
  double *pix = (double *)(ws + p->off_pix);
  double *part = (double *)(ws + p->off_part);
  if (p->spherical) {
    jam::launch_setup(ctx->d_geoms, p->d_models, p->n, pd, gauss, st_ws, status, queue, st);
    jam::launch_sph_terms(ctx->d_geoms, p->d_models, p->d_terms, p->n_terms, gauss, st_ws, terms,
                          adjoint ? (double *)(ws + p->off_terms64) : nullptr,
                          (double *)(ws + p->off_pol), st);
    jam::launch_sb(ctx->d_geoms, p->d_models, p->d_sb, p->n_sb, pd, pix, st);
  } else {
    if (!p->fused_prologue)
      jam::launch_setup(ctx->d_geoms, p->d_models, p->n, pd, gauss, st_ws, status, queue, st);
    const int n_pro = adjoint ? p->n_pro : p->n_pro_fwd;
    if (n_pro)
      jam::launch_prologue(ctx->d_geoms, p->d_models, p->d_pro, n_pro, pd, gauss, st_ws, status,
                         queue, terms, pix, p->fused_prologue, st);
  }
  if (p->spherical) {
    if (!need_numerator) return;
    double *tabs = (double *)(ws + p->off_sph);
    float *sgrid = p->n_sgrid ? (float *)(ws + p->off_sgrid) : nullptr;
    const bool timed = ctx->t_num.begin(st, capturing);
    if (sgrid) {
      double *pol = (double *)(ws + p->off_pol);
      jam::launch_pol_grid(ctx->d_geoms, p->d_models, p->d_sgrid, p->n_sgrid, p->d_sgred,
                           p->n_sgred, terms, st_ws, pol, sgrid, st);
      jam::launch_pol_moments(ctx->d_geoms, p->d_models, p->d_sphm, p->n_sphm, p->d_ptab,
                              p->n_ptab, gauss, terms, st_ws, sgrid, pol, tabs, st);
    } else {
      jam::launch_sph_moments(ctx->d_geoms, p->d_models, p->d_sphm, p->n_sphm, gauss, terms, st_ws,
                              tabs, st);
    }
    if (timed) ctx->t_num.end(st);
    jam::launch_sph_num(ctx->d_geoms, p->d_models, p->d_red, p->n_red, gauss, st_ws, tabs, pix, st);
    return;
  }
  if (need_numerator) {
    const bool timed = ctx->t_num.begin(st, capturing);
    launch_numerator(ctx, p, ws, st);
    if (timed) ctx->t_num.end(st);
    if (p->n_red) jam::launch_reduce(ctx->d_geoms, p->d_models, p->d_red, p->n_red, part, pix, st);
  }
  if (p->n_csum)
    jam::launch_cheb_sum(ctx->d_geoms, p->d_models, p->d_csum, p->n_csum, pd,
                         need_numerator ? part : nullptr, pix, st);
}

void launch_eval(jam_ctx *ctx, Plan *p, const jam_batch *b, double *vrms2, int32_t *status,
                 char *w, hipStream_t st, bool capturing) {
  launch_forward_maps(ctx, p, params_of(b), status, w, st, true, capturing);
  jam::launch_bins(ctx->d_geoms, p->d_models, p->d_bins, p->n_bins, p->n_bins_wave, (const double *)(w + p->off_pix),
                   (const int *)(w + p->off_status), vrms2, (double *)(w + p->off_bins), st);
}

// Adjoint of sum_b cot_b V_b; with chi2_cot != NULL the cotangent is instead
// chi2_cot[m] * d chi^2_m / dV_b, formed in the workspace from V (given or
// recomputed).
void launch_vjp(jam_ctx *ctx, Plan *p, const jam_batch *b, const double *vrms2, const double *cot,
                const jam_grads *grads, char *w, hipStream_t st, bool capturing,
                const double *chi2_cot = nullptr) {
  const int *st_ws = (const int *)(w + p->off_status);
  int *queue = (int *)(w + p->off_queue);
  double *pix = (double *)(w + p->off_pix);
  double *binws = (double *)(w + p->off_bins);
  double *sens = (double *)(w + p->off_sens);
  const jam::ParamsDev pd = params_of(b);
  const bool recompute = (vrms2 == nullptr);
  if (p->spherical) {
    // the spherical adjoint needs the moment table: one pass computes it with
    // the node sums of the characteristic integrals' adjoint.  When V is
    // recomputed it comes from the forward's own path (with the potential
    // grid, the forward's table and numerator map first, then the adjoint's
    // table over it), so that it equals the forward's V bit for bit
    const bool fwd_v = recompute && p->n_sgrid > 0;
    launch_forward_maps(ctx, p, pd, nullptr, w, st, fwd_v, capturing, true);
    const double *gauss = (const double *)(w + p->off_gauss);
    double *tabs = (double *)(w + p->off_sph);
    if (p->n_sgrid > 0) {
      double *pol = (double *)(w + p->off_pol), *sgrid3 = (double *)(w + p->off_sgrid3);
      const double *terms64 = (const double *)(w + p->off_terms64);
      jam::launch_pol_grid_adj(ctx->d_geoms, p->d_models, p->d_sgrid, p->n_sgrid, p->d_sgred3,
                               p->n_sgred3, terms64, st_ws, pol, sgrid3, st);
      jam::launch_pol_moments_adj(ctx->d_geoms, p->d_models, p->d_sphm, p->n_sphm, p->d_ptab,
                                  p->n_ptab, gauss, terms64, st_ws, sgrid3, pol, tabs, sens,
                                  (double *)(w + p->off_sgcot), st);
    } else {
      const float4 *terms = (const float4 *)(w + p->off_terms);
      jam::launch_sph_moments_jac(ctx->d_geoms, p->d_models, p->d_sph, p->n_sph, gauss, terms,
                                  st_ws, tabs, sens, st);
    }
    if (recompute && !fwd_v)
      jam::launch_sph_num(ctx->d_geoms, p->d_models, p->d_red, p->n_red, gauss, st_ws, tabs, pix,
                          st);
  } else {
    launch_forward_maps(ctx, p, pd, nullptr, w, st, recompute, capturing, true);
  }
  // V per bin: the caller's forward output, or recomputed into workspace.
  const double *V = vrms2;
  if (recompute) {
    double *vtmp = (double *)(w + p->off_vtmp);
    jam::launch_bins(ctx->d_geoms, p->d_models, p->d_bins, p->n_bins, p->n_bins_wave, pix, st_ws, vtmp, binws, st);
    V = vtmp;
  } else {
    jam::launch_bins(ctx->d_geoms, p->d_models, p->d_bins, p->n_bins, p->n_bins_wave, pix, st_ws, nullptr, binws, st);
  }
  if (chi2_cot) {
    double *c = (double *)(w + p->off_cot);
    jam::launch_chi2(ctx->d_geoms, p->d_models, p->n, ctx->d_kin, V, st_ws, nullptr, chi2_cot, c,
                     st);
    cot = c;
  }
  jam::launch_bins_adjoint(ctx->d_geoms, p->d_models, p->d_pix, p->n_pix, V, cot, binws, st_ws, pix, st);
  double *sbp = (double *)(w + p->off_sbp);
  jam::launch_sb_adjoint(ctx->d_geoms, p->d_models, p->d_sb, p->n_sb, st_ws, pix, sbp, st);
  const jam::GradsDev gd{grads->inc, grads->mass_scale, grads->m_bh, grads->beta, grads->lum_I0,
                         grads->mass_S0};
  if (p->spherical) {
    const bool ts = ctx->t_sens.begin(st, capturing);
    const double *gauss = (const double *)(w + p->off_gauss);
    const double *terms64 = (const double *)(w + p->off_terms64);
    jam::launch_sph_adjoint(ctx->d_geoms, p->d_models, p->n, p->d_red, p->n_red, p->d_srow, p->n_srow,
                            gauss, st_ws, (const double *)(w + p->off_sph), pix, sens, st);
    if (p->n_pcot)
      jam::launch_pol_adjoint(ctx->d_geoms, p->d_models, p->d_pcot, p->n_pcot, p->d_pfix, p->n_pfix,
                              p->d_sgs, p->n_sgs, gauss, terms64, st_ws,
                              (const double *)(w + p->off_pol), sens,
                              (double *)(w + p->off_sgcot), st);
    else
      jam::launch_sph_sens(ctx->d_geoms, p->d_models, p->d_sens, p->n_sens, gauss,
                           (const float4 *)(w + p->off_terms), st_ws, sens, st);
    jam::launch_sph_chain(ctx->d_geoms, p->d_models, p->n, p->d_terms, p->n_terms, pd, gauss,
                          terms64, st_ws, sbp, sens, gd, st);
    if (ts) ctx->t_sens.end(st);
    return;
  }
  const bool timed = ctx->t_sens.begin(st, capturing);
  if (p->n_sens)
    jam::launch_sens(ctx->d_geoms, p->d_models, p->d_sens, p->n_sens,
                     (const float4 *)(w + p->off_terms), pix, st_ws, sens,
                     p->tune.launch == 1 ? queue + 1 : nullptr, p->grid_sens, st);
  if (p->n_sensw)
    jam::launch_sens_wide(ctx->d_geoms, p->d_models, p->d_sensw, p->n_sensw,
                          (const float4 *)(w + p->off_terms), pix, st_ws, sens, nullptr,
                          p->n_sensw, st);
  if (p->n_cadj) {
    double *T = (double *)(w + p->off_chebt);
    const double *gauss = (const double *)(w + p->off_gauss);
    if (p->n_ctmap)
      jam::launch_cheb_tmap(ctx->d_geoms, p->d_models, p->d_ctmap, p->n_ctmap, pix, st_ws, T, st);
    jam::launch_cheb_adj(ctx->d_geoms, p->d_models, p->d_cadj, p->n_cadj, p->cadj_share,
                         p->cadj_waves, pd, gauss, st_ws, T, sens, st);
    jam::launch_cheb_rows(ctx->d_geoms, p->d_models, p->d_crows, p->n_crows, gauss, st_ws, sens, st);
  }
  if (p->n_adj)
    for (int t = 1; t <= jam::kSmallQuads; ++t)
      if (p->adj_ptr[t] > p->adj_ptr[t - 1])
        jam::launch_adj_small(ctx->d_geoms, p->d_models, p->d_adj + p->adj_ptr[t - 1],
                              p->adj_ptr[t] - p->adj_ptr[t - 1], t, pd, pix, st_ws, sens, st);
  if (timed) ctx->t_sens.end(st);
  if (p->n_chain)
    jam::launch_chain(ctx->d_geoms, p->d_models, p->d_chain, p->n_chain, pd, sens, st_ws, st);
  jam::launch_grads(ctx->d_geoms, p->d_models, p->n, pd, sens, sbp, st_ws, gd, st);
}

// ---------------------------------------------------------------------------
// Autotuner.  Candidates differ in the numerator schedule only (variant rule,
// 64x64-tile threshold, items' term granularity, persistent or one workgroup
// per item); each is timed on the batch composition with fixed valid
// parameters (edge-on, isotropic, unit mass scale) in a scratch workspace.
// Results are cached per composition signature, in memory and optionally in
// a text file (one "key rule tau gran launch" line per entry).
// ---------------------------------------------------------------------------
std::string tune_key(const jam_ctx *ctx, int n, const int32_t *geom_idx) {
  uint64_t h = 1469598103934665603ull;
  auto mix = [&](uint64_t v) {
    for (int i = 0; i < 8; ++i) {
      h ^= (v >> (8 * i)) & 0xff;
      h *= 1099511628211ull;
    }
  };
  for (int m = 0; m < n; ++m) {
    const GeomHost &g = ctx->gh[geom_idx[m]];
    mix((uint64_t)g.n_ux | ((uint64_t)g.n_uy << 20) | ((uint64_t)g.n_u << 40));
    // the forms a map takes depend on these and not on their product alone
    mix((uint64_t)g.K | ((uint64_t)g.J1 << 32));
    mix((uint64_t)g.cheb_np | (g.cheb_gain[0] > 0.0 ? 1ull << 32 : 0) | (g.cheb_gain[1] > 0.0 ? 1ull << 33 : 0));
  }
  char buf[128];
  snprintf(buf, sizeof buf, "gfx950/v3/n%d/%016llx", n, (unsigned long long)h);
  return buf;
}

void load_tune_file(jam_ctx *ctx) {
  if (ctx->tune_path.empty()) return;
  FILE *f = fopen(ctx->tune_path.c_str(), "r");
  if (!f) return;
  char key[160];
  Tune t;
  while (fscanf(f, "%159s %d %d %d %d", key, &t.rule, &t.tau, &t.gran, &t.launch) == 5)
    ctx->tuned.push_back({key, t});
  fclose(f);
}

void save_tune_file(const jam_ctx *ctx) {
  if (ctx->tune_path.empty()) return;
  FILE *f = fopen(ctx->tune_path.c_str(), "w");
  if (!f) return;
  for (auto &e : ctx->tuned)
    fprintf(f, "%s %d %d %d %d\n", e.first.c_str(), e.second.rule, e.second.tau, e.second.gran,
            e.second.launch);
  fclose(f);
}

jam_status autotune(jam_ctx *ctx, int32_t n, const int32_t *geom_idx, Tune &best) {
  std::vector<Tune> cands;
  Tune base;
  base.cheb = choose_cheb(ctx, n, geom_idx, base);   // its models have no slices
  const int g0 = default_gran(ctx, n, geom_idx, base);
  for (int launch = 0; launch < 2; ++launch)
    for (int tau : {0, 1 << 30})
      for (double mul : {0.5, 0.75, 1.0, 1.5, 2.0}) {
        Tune t;
        t.rule = 1;
        t.cheb = base.cheb;
        t.tau = tau;
        t.gran = std::max(1, (int)std::lround(g0 * mul));
        t.launch = launch;
        cands.push_back(t);
      }
  {
    Tune t;
    t.rule = 0;
    t.gran = 0;
    cands.push_back(t);
  }
  std::vector<std::unique_ptr<Plan>> plans(cands.size());
  size_t ws_max = 0;
  for (size_t i = 0; i < cands.size(); ++i) {
    const jam_status s = build_plan(ctx, n, geom_idx, cands[i], plans[i]);
    if (s != JAM_OK) return s;
    ws_max = std::max(ws_max, plans[i]->ws_fwd);
  }
  int64_t nl = 0;
  for (int m = 0; m < n; ++m) nl += ctx->gh[geom_idx[m]].K;
  void *ws = nullptr, *prm = nullptr;
  hipStream_t st = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  auto cleanup = [&]() {
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (st) (void)hipStreamDestroy(st);
    if (prm) (void)hipFree(prm);
    if (ws) (void)hipFree(ws);
  };
  std::vector<double> host(3 * (size_t)n + nl, 0.0);
  for (int m = 0; m < n; ++m) {
    host[m] = kPi / 2;                 // inclination
    host[n + m] = 1.0;                 // mass scale
    host[2 * n + m] = 1.0e8;           // BH mass
  }
  if (hipMalloc(&ws, ws_max) != hipSuccess || hipMalloc(&prm, host.size() * 8) != hipSuccess ||
      hipStreamCreate(&st) != hipSuccess || hipEventCreate(&e0) != hipSuccess ||
      hipEventCreate(&e1) != hipSuccess ||
      hipMemcpy(prm, host.data(), host.size() * 8, hipMemcpyHostToDevice) != hipSuccess) {
    cleanup();
    return fail(JAM_E_DEVICE, "autotune: device allocation failed");
  }
  const double *pp = (const double *)prm;
  const jam::ParamsDev pd{pp, pp + n, pp + 2 * n, pp + 3 * n, nullptr, nullptr};
  double best_ms = 1e300;
  size_t best_i = 0;
  for (size_t i = 0; i < cands.size(); ++i) {
    Plan *p = plans[i].get();
    char *w = (char *)ws;
    float ms = 0.f, tot = 0.f;
    for (int rep = 0; rep < 3; ++rep) {
      launch_forward_maps(ctx, p, pd, nullptr, w, st, false, true);
      (void)hipEventRecord(e0, st);
      launch_numerator(ctx, p, w, st);
      (void)hipEventRecord(e1, st);
      if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
        cleanup();
        return fail(JAM_E_DEVICE, "autotune: timing failed");
      }
      if (rep > 0) tot += ms;    // first run warms caches and clocks
    }
    if (tot < best_ms) {
      best_ms = tot;
      best_i = i;
    }
  }
  const hipError_t e = hipGetLastError();
  cleanup();
  if (e != hipSuccess) return fail(JAM_E_DEVICE, "autotune: %s", hipGetErrorString(e));
  best = plans[best_i]->tune;
  best.cheb = -1;   // derived from the batch, not tuned
  return JAM_OK;
}

// Forward workspace of a cylindrical batch in the direct forms, as build_plan lays
// it out (all_parts: with the partial maps of single slices too); `fixed` the regions
// that no schedule changes.
size_t direct_ws(const jam_ctx *ctx, int n, const int32_t *geom_idx, const Tune &t, bool all_parts,
                 size_t *fixed) {
  int64_t gauss = 0, terms = 0, pix = 0, part = 0, bins = 0, total_bins = 0;
  std::vector<int64_t> models(ctx->gh.size(), 0);
  for (int m = 0; m < n; ++m) ++models[geom_idx[m]];
  for (size_t i = 0; i < models.size(); ++i) {
    if (models[i] == 0) continue;
    const GeomHost &g = ctx->gh[i];
    const NumChoice c = choose_numerator(g, t, t.gran);
    gauss += models[i] * jam::gauss_size(g.K, g.J1);
    terms += models[i] * (c.gen ? 0 : jam::padded_terms(g.T));
    pix += models[i] * 4 * g.n_pix;
    part += models[i] * (all_parts ? part_doubles(g, c) : part_size(g, c));
    bins += models[i] * 2 * g.n_bins;
    total_bins += models[i] * g.n_bins;
  }
  size_t w = align256(sizeof(int) * n);
  w = align256(w + sizeof(int) * 2);
  w = align256(w + sizeof(double) * gauss);
  w = align256(w + sizeof(float4) * terms);
  w = align256(w + sizeof(double) * pix);
  w = align256(w + sizeof(double) * bins);
  w = align256(w + sizeof(double) * total_bins);
  *fixed = w;
  return align256(w + sizeof(double) * part);
}

// Lengthens a direct schedule's slices (t.gran given) until the partial maps fit the
// fixed scratch.  False if they never do, or if that costs the launch more than
// kLongerSlices of its modelled time (130 models of 50 x 50, 20 x 10 x 113 terms: 326
// us, 489 with the slices that would fit).
constexpr double kLongerSlices = 1.1;
bool lengthen_slices(const jam_ctx *ctx, int n, const int32_t *geom_idx, Tune &t) {
  std::vector<int> grans;
  for (int gran = t.gran; gran < (1 << 24); gran += 1 + gran / 8) grans.push_back(gran);
  size_t fixed = 0;
  Tune longer = t;
  auto fits = [&](int gran) {
    longer.gran = gran;
    return direct_ws(ctx, n, geom_idx, longer, false, &fixed) <= kScratchBytes;
  };
  if (grans.empty() || !fits(grans.back())) return false;
  // the partial maps only shrink as the slices grow
  longer.gran = *std::partition_point(grans.begin(), grans.end(), [&](int gran) { return !fits(gran); });
  const double time = gran_makespan(ctx, n, geom_idx, t, longer.gran, SIZE_MAX);
  if (time > kLongerSlices * gran_makespan(ctx, n, geom_idx, t, t.gran, SIZE_MAX)) return false;
  t = longer;
  return true;
}

jam_status get_plan_impl(jam_ctx *ctx, int32_t n, const int32_t *geom_idx, Plan *&out) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  if (n < 1) return fail(JAM_E_INVALID_ARG, "batch size must be >= 1");
  if (!geom_idx) return fail(JAM_E_INVALID_ARG, "geom_idx is NULL");
  for (int m = 0; m < n; ++m)
    if (geom_idx[m] < 0 || geom_idx[m] >= (int)ctx->gh.size())
      return fail(JAM_E_INVALID_ARG, "geom_idx[%d] = %d out of range", m, geom_idx[m]);
  for (auto itp = ctx->plans.begin(); itp != ctx->plans.end(); ++itp) {
    Plan *p = itp->get();
    if (p->n == n && std::equal(p->key.begin(), p->key.end(), geom_idx)) {
      if (itp != ctx->plans.begin()) ctx->plans.splice(ctx->plans.begin(), ctx->plans, itp);
      out = p;
      return JAM_OK;
    }
  }
  Tune t;
  if (ctx->opt.form == 1) t.rule = 0;
  if (ctx->opt.launch == 1) t.launch = 1;
  if (ctx->opt.form == 0 && ctx->opt.autotune) {
    const std::string key = tune_key(ctx, n, geom_idx);
    bool found = false;
    for (auto &e : ctx->tuned)
      if (e.first == key) {
        t = e.second;
        found = true;
        break;
      }
    if (!found) {
      const jam_status s = autotune(ctx, n, geom_idx, t);
      if (s != JAM_OK) return s;
      ctx->tuned.push_back({key, t});
      save_tune_file(ctx);
    }
  }
  std::unique_ptr<Plan> p;
  jam_status s = build_plan(ctx, n, geom_idx, t, p);
  if (s != JAM_OK) return s;
  // The allocation-free entry point's scratch.  A direct batch takes it with slices as
  // long as its partial maps need.  A compressed one that the direct forms fit goes in
  // groups of models that share the H region, two or as many as still pay, and
  // otherwise in those.
  if (p->ws_fwd > kScratchBytes && p->tune.rule == 1 && !p->spherical) {
    if (p->n_cheb == 0) {
      Tune td = p->tune;
      if (lengthen_slices(ctx, n, geom_idx, td) && (s = build_plan(ctx, n, geom_idx, td, p)) != JAM_OK)
        return s;
    } else {
      Tune td = t;
      td.cheb = p->tune.cheb & ~kChebAnyFwd;
      size_t fixed = 0;
      auto fits = [&]() { return direct_ws(ctx, n, geom_idx, td, true, &fixed) <= kScratchBytes; };
      bool direct = true;
      if (td.gran <= 0) {
        td.gran = 1 << 24;   // the smallest partial maps
        direct = fits();
        if (direct) td.gran = default_gran(ctx, n, geom_idx, td);
      }
      if (direct && fits()) {
        // closing a group at h_limit leaves it at most one model over
        const size_t rest = p->off_cheb + 4096;   // the regions before H
        int64_t big = 0, all_h = 0;
        for (int m = 0; m < n; ++m)
          if (takes_cheb(ctx->gh[geom_idx[m]], p->tune.cheb, false)) {
            const int64_t h = (int64_t)ctx->gh[geom_idx[m]].cheb_h.back() * 512;
            big = std::max(big, h);
            all_h += h;
          }
        const int64_t room = rest < kScratchBytes ? (int64_t)((kScratchBytes - rest) / 8) - big : 0;
        const int64_t more = room > 0 ? (all_h - 1) / room : INT32_MAX;   // groups but the first
        const ChebBatch b = cheb_batch(ctx, n, geom_idx, false);
        const double gain = p->tune.cheb & kChebFwdAll ? b.all : b.some;
        if (more > 1 && gain < kChebGroupNs * more)
          s = build_plan(ctx, n, geom_idx, td, p);
        else
          s = build_plan(ctx, n, geom_idx, t, p, room);
        if (s != JAM_OK) return s;
      }
    }
  }
  out = p.get();
  ctx->plans.push_front(std::move(p));
  while (ctx->plans.size() > kMaxPlans) ctx->plans.pop_back();
  return JAM_OK;
}

// The plan of a batch composition, built (and autotuned) at its first use;
// host memory exhaustion while building it is returned as a status.
jam_status get_plan(jam_ctx *ctx, int32_t n, const int32_t *geom_idx, Plan *&out) {
  try {
    return get_plan_impl(ctx, n, geom_idx, out);
  } catch (const std::bad_alloc &) {
    return fail(JAM_E_UNSUPPORTED, "host memory exhausted while preparing a batch of %d", n);
  } catch (...) {
    return fail(JAM_E_UNSUPPORTED, "unexpected host error while preparing a batch of %d", n);
  }
}

// A prepared plan of this composition, or NULL; builds nothing.
Plan *find_plan(jam_ctx *ctx, int32_t n, const int32_t *geom_idx) {
  for (auto &pl : ctx->plans)
    if (pl->n == n && std::equal(pl->key.begin(), pl->key.end(), geom_idx)) return pl.get();
  return nullptr;
}

// Switch to the context's device for the duration of a call.
struct DeviceGuard {
  int prev = -1;
  bool ok = true;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) { ok = false; return; }
    if (prev != dev && hipSetDevice(dev) != hipSuccess) ok = false;
  }
  ~DeviceGuard() {
    int cur;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

jam_status check_batch(const jam_batch *b) {
  if (!b) return fail(JAM_E_INVALID_ARG, "batch is NULL");
  if (!b->inc || !b->mass_scale || !b->m_bh || !b->beta)
    return fail(JAM_E_INVALID_ARG, "batch inc, mass_scale, m_bh and beta are required");
  return JAM_OK;
}

jam_status check_ws(void *ws, size_t ws_bytes, size_t need) {
  if (need > ws_bytes) return fail(JAM_E_WORKSPACE, "workspace of %zu bytes < %zu needed", ws_bytes, need);
  if (!ws) return fail(JAM_E_WORKSPACE, "workspace is NULL");
  if (((uintptr_t)ws & 255) != 0) return fail(JAM_E_WORKSPACE, "workspace must be 256-byte aligned");
  return JAM_OK;
}

// Replay the plan's captured graph `which` (0 forward, 1 adjoint) if it was
// recorded with exactly these pointers; otherwise record it first on the
// context's capture stream.  `record` launches the sequence on a stream.
template <typename F>
jam_status run_graph(jam_ctx *ctx, Plan *p, int which, const GraphKey &key, hipStream_t st,
                     F record) {
  if (!p->gexec[which] || !(p->gkey[which] == key)) {
    if (p->gexec[which]) {
      HIP_TRY(hipGraphExecDestroy(p->gexec[which]));
      p->gexec[which] = nullptr;
    }
    if (!ctx->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking));
    HIP_TRY(hipStreamBeginCapture(ctx->cap_stream, hipStreamCaptureModeThreadLocal));
    record(ctx->cap_stream);
    hipGraph_t graph = nullptr;
    HIP_TRY(hipStreamEndCapture(ctx->cap_stream, &graph));
    const hipError_t e = hipGraphInstantiate(&p->gexec[which], graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) {
      p->gexec[which] = nullptr;
      return fail(JAM_E_DEVICE, "hipGraphInstantiate: %s", hipGetErrorString(e));
    }
    p->gkey[which] = key;
  }
  HIP_TRY(hipGraphLaunch(p->gexec[which], st));
  return JAM_OK;
}

// Inverse of a symmetric positive definite n x n matrix (row-major) by its
// Cholesky factor C = L L^T: L^-1 by forward substitution, then
// C^-1 = L^-T L^-1, written symmetric.  False if C is not positive definite.
bool spd_inverse(int n, const double *c, std::vector<double> &inv) {
  std::vector<long double> L((size_t)n * n, 0.0L), Li((size_t)n * n, 0.0L);
  for (int j = 0; j < n; ++j) {
    long double d = c[(size_t)j * n + j];
    for (int k = 0; k < j; ++k) d -= L[(size_t)j * n + k] * L[(size_t)j * n + k];
    if (!(d > 0.0L)) return false;
    const long double ljj = std::sqrt(d);
    L[(size_t)j * n + j] = ljj;
    for (int i = j + 1; i < n; ++i) {
      long double v = c[(size_t)i * n + j];
      for (int k = 0; k < j; ++k) v -= L[(size_t)i * n + k] * L[(size_t)j * n + k];
      L[(size_t)i * n + j] = v / ljj;
    }
  }
  for (int j = 0; j < n; ++j) {          // column j of L^-1
    Li[(size_t)j * n + j] = 1.0L / L[(size_t)j * n + j];
    for (int i = j + 1; i < n; ++i) {
      long double v = 0.0L;
      for (int k = j; k < i; ++k) v += L[(size_t)i * n + k] * Li[(size_t)k * n + j];
      Li[(size_t)i * n + j] = -v / L[(size_t)i * n + i];
    }
  }
  inv.assign((size_t)n * n, 0.0);
  for (int i = 0; i < n; ++i)
    for (int j = i; j < n; ++j) {
      long double v = 0.0L;
      for (int k = j; k < n; ++k) v += Li[(size_t)k * n + i] * Li[(size_t)k * n + j];
      inv[(size_t)i * n + j] = inv[(size_t)j * n + i] = (double)v;
    }
  return true;
}

// Constants of the one-dimensional MGE transform: Euler nodes
// beta_k = P ln(10)/3 + i pi k and signed binomial weights (-1)^k xi_k,
// k = 0..2P, and per Gaussian the factor w_n dlog(sigma) 2 10^(P/3) that,
// with the transform's 2 sqrt(2 pi) and the expansion's 1/sqrt(2 pi), turns
// sum_k (-1)^k xi_k Re F(sigma_n chi_k) into the peak amplitude.
jam_status mge_constants(int32_t n_comp, int32_t n_sigma, const double *sigma, int32_t P,
                         jam::MgeConst &k) {
  if (n_comp < 1 || n_comp > jam::kMgeMaxComp)
    return fail(JAM_E_INVALID_ARG, "n_comp must be in [1, %d]", jam::kMgeMaxComp);
  if (n_sigma < 1 || n_sigma > jam::kMgeMaxSigma)
    return fail(JAM_E_INVALID_ARG, "n_sigma must be in [1, %d]", jam::kMgeMaxSigma);
  if (P < 1 || 2 * P + 1 > jam::kMgeMaxTerms)
    return fail(JAM_E_INVALID_ARG, "euler_p must be in [1, %d]", (jam::kMgeMaxTerms - 1) / 2);
  if (!sigma) return fail(JAM_E_INVALID_ARG, "sigma is NULL");
  for (int n = 0; n < n_sigma; ++n) {
    if (!(sigma[n] > 0.0) || !std::isfinite(sigma[n]))
      return fail(JAM_E_INVALID_ARG, "sigma[%d] must be positive and finite", n);
    if (n > 0 && !(sigma[n] > sigma[n - 1]))
      return fail(JAM_E_INVALID_ARG, "sigma must be strictly increasing");
  }
  std::memset(&k, 0, sizeof k);
  k.n_terms = 2 * P + 1;
  k.n_sigma = n_sigma;
  const long double pi = 3.141592653589793238462643383279502884L;
  k.beta_re = (double)(P * std::log(10.0L) / 3.0L);
  long double xi[jam::kMgeMaxTerms] = {};
  xi[0] = 0.5L;
  for (int j = 1; j <= P; ++j) xi[j] = 1.0L;
  const long double pw = std::ldexp(1.0L, -P);
  xi[2 * P] = pw;
  long double binom = 1.0L;   // binom(P, j), built up with j
  for (int j = 1; j < P; ++j) {
    binom = binom * (P - j + 1) / j;
    xi[2 * P - j] = xi[2 * P - j + 1] + pw * binom;
  }
  for (int j = 0; j <= 2 * P; ++j) {
    k.beta_im[j] = (double)(pi * j);
    k.eta[j] = (double)((j % 2 ? -xi[j] : xi[j]));
  }
  const long double dlog =
      n_sigma > 1 ? (std::log((long double)sigma[n_sigma - 1]) - std::log((long double)sigma[0])) /
                        (n_sigma - 1)
                  : 1.0L;
  const long double f = 2.0L * std::pow(10.0L, P / 3.0L) * dlog;
  for (int n = 0; n < n_sigma; ++n) {
    k.sigma2[n] = sigma[n] * sigma[n];
    const long double w = (n_sigma > 1 && (n == 0 || n == n_sigma - 1)) ? 0.5L : 1.0L;
    k.scale[n] = (double)(w * f);
  }
  return JAM_OK;
}

jam_status check_kinematics(const jam_ctx *ctx, const jam_batch *b) {
  for (int m = 0; m < b->n; ++m) {
    const int gi = b->geom_idx[m];
    if (gi < 0 || gi >= (int)ctx->kin_host.size())
      return fail(JAM_E_INVALID_ARG, "geom_idx[%d] out of range", m);
    if (!ctx->kin_host[gi].prec)
      return fail(JAM_E_INVALID_ARG, "no kinematics set for geometry %d (model %d)", gi, m);
  }
  return JAM_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// C ABI.
// ---------------------------------------------------------------------------
extern "C" {

const char *jam_last_error(void) { return g_err.c_str(); }

jam_status jam_timing(jam_ctx *ctx, int32_t enable, double *numerator_ms,
                      int64_t *numerator_launches, double *sens_ms, int64_t *sens_launches) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  KernelTimer *ts[2] = {&ctx->t_num, &ctx->t_sens};
  if (enable) {
    for (KernelTimer *t : ts) {
      if (t->start.empty()) {
        t->start.resize(KernelTimer::kCap);
        t->stop.resize(KernelTimer::kCap);
        for (int i = 0; i < KernelTimer::kCap; ++i) {
          HIP_TRY(hipEventCreate(&t->start[i]));
          HIP_TRY(hipEventCreate(&t->stop[i]));
        }
      }
      t->used = 0;
      t->on = true;
    }
    return JAM_OK;
  }
  double ms[2] = {0.0, 0.0};
  for (int k = 0; k < 2; ++k) {
    KernelTimer *t = ts[k];
    t->on = false;
    for (int i = 0; i < t->used; ++i) {
      HIP_TRY(hipEventSynchronize(t->stop[i]));
      float e = 0.f;
      HIP_TRY(hipEventElapsedTime(&e, t->start[i], t->stop[i]));
      ms[k] += e;
    }
  }
  if (numerator_ms) *numerator_ms = ms[0];
  if (numerator_launches) *numerator_launches = ctx->t_num.used;
  if (sens_ms) *sens_ms = ms[1];
  if (sens_launches) *sens_launches = ctx->t_sens.used;
  return JAM_OK;
}

jam_status jam_gauss_legendre(int32_t n, double *nodes, double *weights) {
  if (n < 1 || n > kMaxNu) return fail(JAM_E_INVALID_ARG, "n must be in [1, 1024]");
  if (!nodes || !weights) return fail(JAM_E_INVALID_ARG, "output arrays are NULL");
  gauss_legendre01(n, nodes, weights);
  return JAM_OK;
}

jam_status jam_create(int32_t n_geom, const jam_geometry *geoms, const jam_options *opt,
                      jam_ctx **out) {
  g_err.clear();
  if (!out) return fail(JAM_E_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (n_geom < 1 || !geoms) return fail(JAM_E_INVALID_ARG, "need at least one geometry");
  for (int i = 0; i < n_geom; ++i) {
    const jam_status s = validate(geoms[i], i);
    if (s != JAM_OK) return s;
  }
  if (opt && (opt->form < 0 || opt->form > 2))
    return fail(JAM_E_INVALID_ARG, "options.form must be 0, 1 or 2");
  if (opt && (opt->launch < 0 || opt->launch > 1))
    return fail(JAM_E_INVALID_ARG, "options.launch must be 0 or 1");
  if (opt && (opt->alignment < 0 || opt->alignment > 1))
    return fail(JAM_E_INVALID_ARG, "options.alignment must be 0 or 1");
  auto ctx = std::make_unique<jam_ctx>();
  if (opt) ctx->opt = *opt;
  if (opt && opt->tune_cache) ctx->tune_path = opt->tune_cache;
  ctx->opt.tune_cache = nullptr;   // the path is copied
  HIP_TRY(hipGetDevice(&ctx->device));
  HIP_TRY(hipDeviceGetAttribute(&ctx->n_cu, hipDeviceAttributeMultiprocessorCount, ctx->device));
  ctx->occ_num_pix = jam::occupancy_num(false);
  ctx->occ_num_mfma = jam::occupancy_num(true);
  ctx->occ_sens = jam::occupancy_sens();
  {
    const jam_status s = scratch_address(ctx->device, &ctx->scratch);
    if (s != JAM_OK) return s;
  }
  load_tune_file(ctx.get());
  ctx->gh.resize(n_geom);
  {
    const unsigned nt = std::max(1u, std::min(8u, std::thread::hardware_concurrency()));
    std::vector<std::thread> pool;
    std::vector<int> failed(nt, -1);
    for (unsigned t = 0; t < nt; ++t)
      pool.emplace_back([&, t] {
        for (int i = (int)t; i < n_geom; i += (int)nt) {
          try {
            build_geometry(geoms[i], ctx->gh[i]);
            build_spherical(ctx->gh[i]);
            if (ctx->opt.alignment == 0 && ctx->opt.form == 0) build_cheb(ctx->gh[i]);
          } catch (...) {   // out of host memory: reported below, never past the thread
            failed[t] = i;
            return;
          }
        }
      });
    for (auto &th : pool) th.join();
    for (unsigned t = 0; t < nt; ++t)
      if (failed[t] >= 0)
        return fail(JAM_E_UNSUPPORTED, "geometry %d: host memory exhausted while building it",
                    failed[t]);
  }
  // device arena: GeomDev array then every geometry's arrays
  size_t off = align256(sizeof(jam::GeomDev) * n_geom);
  struct Offs { size_t ls, lq, li, ms, mq, mS, u, w, xs, ys, ux, uy, bp, bpix, bw, pp, pb, pw, cl, cx, cE, cEk, cGk, cp, ci, ch, cch, cpc, cjp, cjx, cpx, cpy, cux; };
  std::vector<Offs> offs(n_geom);
  auto take = [&](size_t bytes) { const size_t o = off; off = align256(off + std::max<size_t>(bytes, 8)); return o; };
  for (int i = 0; i < n_geom; ++i) {
    const GeomHost &g = ctx->gh[i];
    Offs &o = offs[i];
    o.ls = take(8 * g.K); o.lq = take(8 * g.K); o.li = take(8 * g.K);
    o.ms = take(8 * g.J); o.mq = take(8 * g.J); o.mS = take(8 * g.J);
    o.u = take(8 * g.n_u); o.w = take(8 * g.n_u);
    o.xs = take(8 * g.n_ux); o.ys = take(8 * g.n_uy);
    o.ux = take(4 * g.nxp); o.uy = take(4 * g.nyp);
    o.bp = take(4 * g.bin_ptr.size()); o.bpix = take(4 * g.bin_pix.size()); o.bw = take(8 * g.bin_w.size());
    o.pp = take(4 * g.pix_ptr.size()); o.pb = take(4 * g.pix_bin.size()); o.pw = take(8 * g.pix_w.size());
    o.cl = take(8 * g.cheb_lo.size()); o.cx = take(8 * g.cheb_xi.size());
    o.cE = take(8 * g.cheb_E.size()); o.cEk = take(8 * g.cheb_Ek.size());
    o.cGk = take(8 * g.cheb_Gk.size());  o.cp = take(4 * g.cheb_ptr.size());
    o.ci = take(4 * g.cheb_id.size()); o.ch = take(4 * g.cheb_h.size());
    o.cch = take(4 * g.cheb_ch.size()); o.cpc = take(4 * g.cheb_pc.size());
    o.cjp = take(4 * g.cheb_jp.size()); o.cjx = take(4 * g.cheb_jx.size());
    o.cux = take(2 * g.cheb_ux.size()); o.cpx = take(g.cheb_px.size()); o.cpy = take(g.cheb_py.size());
  }
  std::vector<char> stage(off, 0);
  HIP_TRY(hipMalloc(&ctx->arena, off));
  char *base = (char *)ctx->arena;
  std::vector<jam::GeomDev> gd(n_geom);
  auto put = [&](size_t o, const void *src, size_t bytes) {
    if (bytes) std::memcpy(stage.data() + o, src, bytes);
    return base + o;
  };
  for (int i = 0; i < n_geom; ++i) {
    const GeomHost &g = ctx->gh[i];
    const Offs &o = offs[i];
    jam::GeomDev &d = gd[i];
    d.K = g.K; d.J1 = g.J1; d.n_u = g.n_u; d.T = g.T;
    d.n_ux = g.n_ux; d.n_uy = g.n_uy; d.n_pix = g.n_pix; d.n_bins = g.n_bins;
    d.nxp = g.nxp; d.nyp = g.nyp; d.pad0 = d.pad1 = 0;
    d.s_pc = g.s_pc; d.bh_sigma = g.bh_sigma;
    d.lum_sigma = (const double *)put(o.ls, g.lum_sigma.data(), 8 * g.K);
    d.lum_q = (const double *)put(o.lq, g.lum_q.data(), 8 * g.K);
    d.lum_I0 = (const double *)put(o.li, g.lum_I0.data(), 8 * g.K);
    d.mass_sigma = (const double *)put(o.ms, g.mass_sigma.data(), 8 * g.J);
    d.mass_q = (const double *)put(o.mq, g.mass_q.data(), 8 * g.J);
    d.mass_S0 = (const double *)put(o.mS, g.mass_S0.data(), 8 * g.J);
    d.u = (const double *)put(o.u, g.u.data(), 8 * g.n_u);
    d.w = (const double *)put(o.w, g.w.data(), 8 * g.n_u);
    d.xs = (const double *)put(o.xs, g.xs.data(), 8 * g.n_ux);
    d.ys = (const double *)put(o.ys, g.ys.data(), 8 * g.n_uy);
    d.ux = (const int *)put(o.ux, g.ux.data(), 4 * g.nxp);
    d.uy = (const int *)put(o.uy, g.uy.data(), 4 * g.nyp);
    d.bin_ptr = (const int *)put(o.bp, g.bin_ptr.data(), 4 * g.bin_ptr.size());
    d.bin_pix = (const int *)put(o.bpix, g.bin_pix.data(), 4 * g.bin_pix.size());
    d.bin_w = (const double *)put(o.bw, g.bin_w.data(), 8 * g.bin_w.size());
    d.pix_ptr = (const int *)put(o.pp, g.pix_ptr.data(), 4 * g.pix_ptr.size());
    d.pix_bin = (const int *)put(o.pb, g.pix_bin.data(), 4 * g.pix_bin.size());
    d.pix_w = (const double *)put(o.pw, g.pix_w.data(), 8 * g.pix_w.size());
    d.cheb_np = g.cheb_np;
    d.cheb_pieces = g.cheb_pieces;
    d.cheb_lo = (const double *)put(o.cl, g.cheb_lo.data(), 8 * g.cheb_lo.size());
    d.cheb_xi = (const double *)put(o.cx, g.cheb_xi.data(), 8 * g.cheb_xi.size());
    d.cheb_E = (const double *)put(o.cE, g.cheb_E.data(), 8 * g.cheb_E.size());
    d.cheb_Ek = (const double *)put(o.cEk, g.cheb_Ek.data(), 8 * g.cheb_Ek.size());
    d.cheb_Gk = (const double *)put(o.cGk, g.cheb_Gk.data(), 8 * g.cheb_Gk.size());
    d.cheb_ch = (const int *)put(o.cch, g.cheb_ch.data(), 4 * g.cheb_ch.size());
    d.cheb_pc = (const int *)put(o.cpc, g.cheb_pc.data(), 4 * g.cheb_pc.size());
    d.cheb_jp = (const int *)put(o.cjp, g.cheb_jp.data(), 4 * g.cheb_jp.size());
    d.cheb_jx = (const int *)put(o.cjx, g.cheb_jx.data(), 4 * g.cheb_jx.size());
    d.cheb_ux = (const unsigned short *)put(o.cux, g.cheb_ux.data(), 2 * g.cheb_ux.size());
    d.cheb_ptr = (const int *)put(o.cp, g.cheb_ptr.data(), 4 * g.cheb_ptr.size());
    d.cheb_id = (const int *)put(o.ci, g.cheb_id.data(), 4 * g.cheb_id.size());
    d.cheb_h = (const int *)put(o.ch, g.cheb_h.data(), 4 * g.cheb_h.size());
    d.cheb_px = (const unsigned char *)put(o.cpx, g.cheb_px.data(), g.cheb_px.size());
    d.cheb_py = (const unsigned char *)put(o.cpy, g.cheb_py.data(), g.cheb_py.size());
    d.sph_lnr0 = g.sph_lnr0;
    d.sph_dlnr = g.sph_dlnr;
    d.sph_sig_max = g.sph_sig_max;
    for (int q = 0; q < 8; ++q) {
      d.gl8_x[q] = g.gl8_x[q];
      d.gl8_w[q] = g.gl8_w[q];
    }
  }
  std::memcpy(stage.data(), gd.data(), sizeof(jam::GeomDev) * n_geom);
  HIP_TRY(hipMemcpy(ctx->arena, stage.data(), off, hipMemcpyHostToDevice));
  ctx->d_geoms = (jam::GeomDev *)ctx->arena;
  ctx->kin_buf.assign(n_geom, nullptr);
  ctx->kin_host.assign(n_geom, jam::KinDev{nullptr, nullptr});
  HIP_TRY(hipMalloc(&ctx->d_kin, sizeof(jam::KinDev) * n_geom));
  HIP_TRY(hipMemcpy(ctx->d_kin, ctx->kin_host.data(), sizeof(jam::KinDev) * n_geom,
                    hipMemcpyHostToDevice));
  *out = ctx.release();
  return JAM_OK;
}

void jam_destroy(jam_ctx *ctx) { delete ctx; }

jam_status jam_batch_sizes(const jam_ctx *ctx, int32_t n, const int32_t *geom_idx,
                           int64_t *n_bins_total, int64_t *n_lum_total, int64_t *n_mass_total) {
  if (!ctx || n < 1 || !geom_idx) return fail(JAM_E_INVALID_ARG, "invalid arguments");
  int64_t b = 0, l = 0, ms = 0;
  for (int m = 0; m < n; ++m) {
    if (geom_idx[m] < 0 || geom_idx[m] >= (int)ctx->gh.size())
      return fail(JAM_E_INVALID_ARG, "geom_idx[%d] out of range", m);
    const GeomHost &g = ctx->gh[geom_idx[m]];
    b += g.n_bins;
    l += g.K;
    ms += g.J;
  }
  if (n_bins_total) *n_bins_total = b;
  if (n_lum_total) *n_lum_total = l;
  if (n_mass_total) *n_mass_total = ms;
  return JAM_OK;
}

jam_status jam_prepare(jam_ctx *ctx, int32_t n, const int32_t *geom_idx) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  return get_plan(ctx, n, geom_idx, p);
}

jam_status jam_workspace_size(jam_ctx *ctx, int32_t n, const int32_t *geom_idx, int32_t with_vjp,
                              size_t *bytes) {
  if (!bytes) return fail(JAM_E_INVALID_ARG, "bytes is NULL");
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  const jam_status s = get_plan(ctx, n, geom_idx, p);
  if (s != JAM_OK) return s;
  *bytes = with_vjp ? p->ws_vjp : p->ws_fwd;
  return JAM_OK;
}

jam_status jam_eval_batch(jam_ctx *ctx, const jam_batch *batch, double *vrms2, int32_t *status,
                          void *ws, size_t ws_bytes, void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  jam_status s = check_batch(batch);
  if (s != JAM_OK) return s;
  if (!vrms2) return fail(JAM_E_INVALID_ARG, "vrms2 is NULL");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  if ((s = get_plan(ctx, batch->n, batch->geom_idx, p)) != JAM_OK) return s;
  if ((s = check_ws(ws, ws_bytes, p->ws_fwd)) != JAM_OK) return s;
  hipStream_t st = (hipStream_t)stream;
  char *w = (char *)ws;
  if (ctx->opt.graph) {
    const GraphKey k({batch->inc, batch->mass_scale, batch->m_bh, batch->beta, batch->lum_I0,
                      batch->mass_S0, vrms2, status, ws}, ws_bytes);
    const jam_batch b = *batch;
    s = run_graph(ctx, p, 0, k, st, [&](hipStream_t cs) {
      launch_eval(ctx, p, &b, vrms2, status, w, cs, true);
    });
    if (s != JAM_OK) return s;
  } else {
    launch_eval(ctx, p, batch, vrms2, status, w, st, false);
  }
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_eval(jam_ctx *ctx, const jam_batch *one, double *vrms2, int32_t *status, void *ws,
                    size_t ws_bytes, void *stream) {
  if (one && one->n != 1) return fail(JAM_E_INVALID_ARG, "jam_eval takes exactly one model");
  return jam_eval_batch(ctx, one, vrms2, status, ws, ws_bytes, stream);
}

jam_status jam_eval_batch_noalloc(jam_ctx *ctx, const jam_batch *batch, double *vrms2,
                                  int32_t *status, void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  jam_status s = check_batch(batch);
  if (s != JAM_OK) return s;
  if (!vrms2) return fail(JAM_E_INVALID_ARG, "vrms2 is NULL");
  if (batch->n < 1 || !batch->geom_idx) return fail(JAM_E_INVALID_ARG, "invalid batch");
  if (!ctx->scratch) return fail(JAM_E_DEVICE, "fixed scratch memory is not available");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = find_plan(ctx, batch->n, batch->geom_idx);
  if (!p)
    return fail(JAM_E_INVALID_ARG,
                "batch composition not prepared: call jam_prepare (which allocates) first");
  if (p->ws_fwd > kScratchBytes)
    return fail(JAM_E_WORKSPACE, "composition needs %zu bytes of workspace, above the %zu bytes "
                "of fixed scratch", p->ws_fwd, kScratchBytes);
  // eager launches only (instantiating a graph allocates); no timing events
  launch_eval(ctx, p, batch, vrms2, status, (char *)ctx->scratch, (hipStream_t)stream, true);
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_eval_maps(jam_ctx *ctx, const jam_batch *batch, double *N_map, double *I_map,
                         int32_t *status, void *ws, size_t ws_bytes, void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  jam_status s = check_batch(batch);
  if (s != JAM_OK) return s;
  if (!N_map || !I_map) return fail(JAM_E_INVALID_ARG, "map outputs are NULL");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  if ((s = get_plan(ctx, batch->n, batch->geom_idx, p)) != JAM_OK) return s;
  if ((s = check_ws(ws, ws_bytes, p->ws_fwd)) != JAM_OK) return s;
  hipStream_t st = (hipStream_t)stream;
  char *w = (char *)ws;
  launch_forward_maps(ctx, p, params_of(batch), status, w, st, true, false);
  jam::launch_maps(ctx->d_geoms, p->d_models, p->d_maps, p->n_maps, (const double *)(w + p->off_pix),
                   (const int *)(w + p->off_status), N_map, I_map, st);
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_vjp(jam_ctx *ctx, const jam_batch *batch, const double *vrms2, const double *cot,
                   jam_grads *grads, void *ws, size_t ws_bytes, void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  jam_status s = check_batch(batch);
  if (s != JAM_OK) return s;
  if (!cot || !grads) return fail(JAM_E_INVALID_ARG, "cot and grads are required");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  if ((s = get_plan(ctx, batch->n, batch->geom_idx, p)) != JAM_OK) return s;
  if ((s = check_ws(ws, ws_bytes, p->ws_vjp)) != JAM_OK) return s;
  hipStream_t st = (hipStream_t)stream;
  char *w = (char *)ws;
  if (ctx->opt.graph) {
    // gradient outputs are part of the recorded launches
    const GraphKey k({batch->inc, batch->mass_scale, batch->m_bh, batch->beta, batch->lum_I0,
                      batch->mass_S0, vrms2, cot, ws, grads->inc, grads->mass_scale, grads->m_bh,
                      grads->beta, grads->lum_I0, grads->mass_S0},
                     ws_bytes);
    const jam_batch b = *batch;
    const jam_grads g = *grads;
    s = run_graph(ctx, p, 1, k, st, [&](hipStream_t cs) {
      launch_vjp(ctx, p, &b, vrms2, cot, &g, w, cs, true);
    });
    if (s != JAM_OK) return s;
  } else {
    launch_vjp(ctx, p, batch, vrms2, cot, grads, w, st, false);
  }
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

static jam_status set_kinematics_impl(jam_ctx *ctx, int32_t geom, const double *vrms_obs,
                                      const double *cov) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  if (geom < 0 || geom >= (int)ctx->gh.size()) return fail(JAM_E_INVALID_ARG, "geometry %d out of range", geom);
  if (!vrms_obs || !cov) return fail(JAM_E_INVALID_ARG, "vrms_obs and cov are required");
  const int nb = ctx->gh[geom].n_bins;
  if (nb > jam::kChi2MaxBins)
    return fail(JAM_E_UNSUPPORTED, "chi^2 supports at most %d bins (geometry %d has %d)",
                jam::kChi2MaxBins, geom, nb);
  double cmax = 0.0;
  for (int i = 0; i < nb; ++i) {
    if (!std::isfinite(vrms_obs[i])) return fail(JAM_E_INVALID_ARG, "vrms_obs[%d] is not finite", i);
    for (int j = 0; j < nb; ++j) {
      const double v = cov[(size_t)i * nb + j];
      if (!std::isfinite(v)) return fail(JAM_E_INVALID_ARG, "cov[%d][%d] is not finite", i, j);
      cmax = std::max(cmax, std::fabs(v));
    }
  }
  for (int i = 0; i < nb; ++i)
    for (int j = i + 1; j < nb; ++j)
      if (std::fabs(cov[(size_t)i * nb + j] - cov[(size_t)j * nb + i]) > 1e-12 * cmax)
        return fail(JAM_E_INVALID_ARG, "cov is not symmetric at (%d, %d)", i, j);
  std::vector<double> host((size_t)nb + (size_t)nb * nb);
  std::vector<double> inv;
  if (!spd_inverse(nb, cov, inv)) return fail(JAM_E_INVALID_ARG, "cov is not positive definite");
  std::copy(vrms_obs, vrms_obs + nb, host.begin());
  std::copy(inv.begin(), inv.end(), host.begin() + nb);
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  HIP_TRY(hipDeviceSynchronize());      // no evaluation may still read the old buffer
  void *buf = nullptr;
  HIP_TRY(hipMalloc(&buf, host.size() * sizeof(double)));
  if (hipMemcpy(buf, host.data(), host.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipFree(buf);
    return fail(JAM_E_DEVICE, "copy of the kinematics failed");
  }
  const jam::KinDev kd{(const double *)buf, (const double *)buf + nb};
  if (hipMemcpy(ctx->d_kin + geom, &kd, sizeof kd, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipFree(buf);
    return fail(JAM_E_DEVICE, "copy of the kinematics table failed");
  }
  if (ctx->kin_buf[geom]) HIP_TRY(hipFree(ctx->kin_buf[geom]));
  ctx->kin_buf[geom] = buf;
  ctx->kin_host[geom] = kd;
  return JAM_OK;
}

jam_status jam_set_kinematics(jam_ctx *ctx, int32_t geom, const double *vrms_obs,
                              const double *cov) {
  try {
    return set_kinematics_impl(ctx, geom, vrms_obs, cov);
  } catch (...) {
    return fail(JAM_E_UNSUPPORTED, "host memory exhausted while setting the kinematics");
  }
}

jam_status jam_chi2(jam_ctx *ctx, const jam_batch *batch, const double *vrms2, double *chi2,
                    double *dchi2, void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  if (!batch || batch->n < 1 || !batch->geom_idx) return fail(JAM_E_INVALID_ARG, "invalid batch");
  if (!vrms2 || !chi2) return fail(JAM_E_INVALID_ARG, "vrms2 and chi2 are required");
  jam_status s = check_kinematics(ctx, batch);
  if (s != JAM_OK) return s;
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  if ((s = get_plan(ctx, batch->n, batch->geom_idx, p)) != JAM_OK) return s;
  jam::launch_chi2(ctx->d_geoms, p->d_models, p->n, ctx->d_kin, vrms2, nullptr, chi2, nullptr,
                   dchi2, (hipStream_t)stream);
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_eval_chi2(jam_ctx *ctx, const jam_batch *batch, double *chi2, double *vrms2,
                         int32_t *status, void *ws, size_t ws_bytes, void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  jam_status s = check_batch(batch);
  if (s != JAM_OK) return s;
  if (!chi2) return fail(JAM_E_INVALID_ARG, "chi2 is NULL");
  if ((s = check_kinematics(ctx, batch)) != JAM_OK) return s;
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  if ((s = get_plan(ctx, batch->n, batch->geom_idx, p)) != JAM_OK) return s;
  if ((s = check_ws(ws, ws_bytes, p->ws_fwd)) != JAM_OK) return s;
  hipStream_t st = (hipStream_t)stream;
  char *w = (char *)ws;
  double *V = vrms2 ? vrms2 : (double *)(w + p->off_vfwd);
  auto record = [&](const jam_batch *b, hipStream_t cs, bool capturing) {
    launch_eval(ctx, p, b, V, status, w, cs, capturing);
    jam::launch_chi2(ctx->d_geoms, p->d_models, p->n, ctx->d_kin, V,
                     (const int *)(w + p->off_status), chi2, nullptr, nullptr, cs);
  };
  if (ctx->opt.graph) {
    const GraphKey k({batch->inc, batch->mass_scale, batch->m_bh, batch->beta, batch->lum_I0,
                      batch->mass_S0, V, status, ws, chi2, ctx->d_kin},
                     ws_bytes);
    const jam_batch b = *batch;
    s = run_graph(ctx, p, 2, k, st, [&](hipStream_t cs) { record(&b, cs, true); });
    if (s != JAM_OK) return s;
  } else {
    record(batch, st, false);
  }
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_vjp_chi2(jam_ctx *ctx, const jam_batch *batch, const double *vrms2,
                        const double *cot, jam_grads *grads, void *ws, size_t ws_bytes,
                        void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  jam_status s = check_batch(batch);
  if (s != JAM_OK) return s;
  if (!cot || !grads) return fail(JAM_E_INVALID_ARG, "cot and grads are required");
  if ((s = check_kinematics(ctx, batch)) != JAM_OK) return s;
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  if ((s = get_plan(ctx, batch->n, batch->geom_idx, p)) != JAM_OK) return s;
  if ((s = check_ws(ws, ws_bytes, p->ws_vjp)) != JAM_OK) return s;
  hipStream_t st = (hipStream_t)stream;
  char *w = (char *)ws;
  if (ctx->opt.graph) {
    const GraphKey k({batch->inc, batch->mass_scale, batch->m_bh, batch->beta, batch->lum_I0,
                      batch->mass_S0, vrms2, cot, ws, grads->inc, grads->mass_scale, grads->m_bh,
                      grads->beta, grads->lum_I0, grads->mass_S0, ctx->d_kin},
                     ws_bytes);
    const jam_batch b = *batch;
    const jam_grads g = *grads;
    s = run_graph(ctx, p, 3, k, st, [&](hipStream_t cs) {
      launch_vjp(ctx, p, &b, vrms2, nullptr, &g, w, cs, true, cot);
    });
    if (s != JAM_OK) return s;
  } else {
    launch_vjp(ctx, p, batch, vrms2, nullptr, grads, w, st, false, cot);
  }
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_mge1d(int32_t n_prof, int32_t n_comp, const double *comp, int32_t n_sigma,
                     const double *sigma, int32_t euler_p, double *amp, void *stream) {
  if (n_prof < 1 || n_prof > (1 << 24)) return fail(JAM_E_INVALID_ARG, "n_prof must be in [1, 2^24]");
  if (!comp || !amp) return fail(JAM_E_INVALID_ARG, "comp and amp are required");
  jam::MgeConst k;
  const jam_status s = mge_constants(n_comp, n_sigma, sigma, euler_p, k);
  if (s != JAM_OK) return s;
  jam::launch_mge1d(n_prof, n_comp, comp, k, amp, (hipStream_t)stream);
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_mge1d_vjp(int32_t n_prof, int32_t n_comp, const double *comp, int32_t n_sigma,
                         const double *sigma, int32_t euler_p, const double *cot, double *grad,
                         void *stream) {
  if (n_prof < 1 || n_prof > (1 << 24)) return fail(JAM_E_INVALID_ARG, "n_prof must be in [1, 2^24]");
  if (!comp || !cot || !grad) return fail(JAM_E_INVALID_ARG, "comp, cot and grad are required");
  jam::MgeConst k;
  const jam_status s = mge_constants(n_comp, n_sigma, sigma, euler_p, k);
  if (s != JAM_OK) return s;
  jam::launch_mge1d_vjp(n_prof, n_comp, comp, k, cot, grad, (hipStream_t)stream);
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_beta_logistic(jam_ctx *ctx, const jam_batch *batch, const double *prof, double *beta,
                             void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  if (!batch || batch->n < 1 || !batch->geom_idx) return fail(JAM_E_INVALID_ARG, "invalid batch");
  if (!prof || !beta) return fail(JAM_E_INVALID_ARG, "prof and beta are required");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  const jam_status s = get_plan(ctx, batch->n, batch->geom_idx, p);
  if (s != JAM_OK) return s;
  jam::launch_beta_logistic(ctx->d_geoms, p->d_models, p->n, prof, beta, (hipStream_t)stream);
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_beta_logistic_vjp(jam_ctx *ctx, const jam_batch *batch, const double *prof,
                                 const double *cot, double *grad, void *stream) {
  if (!ctx) return fail(JAM_E_INVALID_ARG, "ctx is NULL");
  if (!batch || batch->n < 1 || !batch->geom_idx) return fail(JAM_E_INVALID_ARG, "invalid batch");
  if (!prof || !cot || !grad) return fail(JAM_E_INVALID_ARG, "prof, cot and grad are required");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  const jam_status s = get_plan(ctx, batch->n, batch->geom_idx, p);
  if (s != JAM_OK) return s;
  jam::launch_beta_logistic_vjp(ctx->d_geoms, p->d_models, p->n, prof, cot, grad,
                                (hipStream_t)stream);
  HIP_TRY(hipGetLastError());
  return JAM_OK;
}

jam_status jam_plan_info(jam_ctx *ctx, int32_t n, const int32_t *geom_idx, int32_t *info) {
  if (!ctx || !info) return fail(JAM_E_INVALID_ARG, "invalid arguments");
  DeviceGuard dg(ctx->device);
  if (!dg.ok) return fail(JAM_E_DEVICE, "cannot select the context's device");
  Plan *p = nullptr;
  const jam_status s = get_plan(ctx, n, geom_idx, p);
  if (s != JAM_OK) return s;
  info[0] = p->tune.rule;
  info[1] = p->tune.tau;
  info[2] = p->tune.gran;
  info[3] = p->tune.launch;
  info[4] = p->n_num + p->n_numsm + p->n_cmap;
  info[5] = (p->n_num || !(p->n_cmap || p->n_numsm) ? p->grid_num : 0) + p->n_numsm + p->n_cmap;
  info[6] = p->n_sens + p->n_sensw + p->n_adj + p->n_cadj;
  info[7] = (p->n_sens ? p->grid_sens : 0) + p->n_sensw + p->n_adj + p->n_cadj;
  info[8] = p->spherical ? 3 : (p->tune.rule == 0 ? 0 : (p->n_cheb == p->n ? 4 : 1));
  return JAM_OK;
}

}  // extern "C"
