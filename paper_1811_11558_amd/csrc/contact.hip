// The Polonsky-Keer iteration of frictionless contact (Sec. 5.1) and the
// normal surface compliance, as few launches as its global sums allow.
//
// One iteration on an nx x ny surface (p > 0: the contact set):
//   dir      mean of g on the contact set and sum (g - mean)^2 give beta;
//            t = g - mean + beta t on the contact set, its rows transformed
//   columns  column transform, 2 / (E* |q|) / (nx ny), inverse column
//            transform, in place
//   curv     rows transformed back to r = M[t];          sums for the step
//   update   tau from those sums, p_new = max(p - tau t, 0), re-admission of
//            overlaps, its rows transformed;             sum p_new, overlaps
//   columns  the same, times the load renormalisation W / (dA sum p_new)
//   gap      rows transformed back to u = M[p]; p renormalised, g = u - h;
//            sum |p - p_old|, and the sums for the next dir
// Every global sum is one kernel boundary: its block sums are totalled, in one
// fixed order, by each block of the next kernel that needs them.  (Where two
// kernels take the same total, the load scale of columns and gap, blocks of other
// sizes, nx != ny, may add it in another order: p and u then differ in their scale's
// last bit.)  The two
// centred sums, sum (g - mean)^2 and sum (r - mean r) t, take no pass of their
// own either: a block centres its values on its own means and the blocks'
// moments are combined about the total mean,
//   sum (a - A)(b - B) = sum_blocks [C_b + n_b (A_b - A)(B_b - B)],
// which cancels nothing.  (Taken as sum r t - (mean r) sum t instead, the
// step's denominator is lost to rounding once t is at the rounding floor, and
// the iterate with it.)
//
#include <algorithm>

#include "common.hpp"
#include "contact.hpp"
#include "surf_dev.hpp"

namespace fvim {
namespace {

constexpr int GT = 256;                 // threads of the pointwise kernels
constexpr int GB = 256;                 // their most blocks

// blocks of the row kernels of an nx x ny surface (pairs of rows)
int pk_row_blocks(int nx, int ny) {
  const int m = nx / 4, nth = m < 64 ? 64 : m, seq = nth / m;
  return (ny / 2 + seq - 1) / seq;
}
int pk_ldp(int nx, int ny) { return pk_row_blocks(nx, ny); }

// rows of the block sums: update (sum p, overlaps), gap (sum |dp|, sum g,
// count, centred g^2 and g), curv (sum g t, sum r, sum t, count, centred r t)
enum { PU = 0, PG = 2, PR = 7, PROWS = 12 };

// one row pair of the thread's sequence: rows 2 s and 2 s + 1
struct Pair {
  int b, jj, s;
  bool on;
  size_t off;                           // of row 2 s
};
template <int LOGN>
__device__ __forceinline__ Pair row_pair(int ny) {
  using S = Surf<LOGN>;
  Pair q;
  q.b = threadIdx.x / S::M;
  q.jj = threadIdx.x & (S::M - 1);
  q.s = blockIdx.x * S::SEQ + q.b;
  q.on = 2 * q.s < ny;
  q.off = (size_t)2 * q.s * S::N;
  return q;
}

// the 8 values of the thread's row pair, (row a, row b) at x = jj + m M
template <int LOGN>
__device__ __forceinline__ void load_pair(const double* __restrict__ f, const Pair& q, cpx<double> (&v)[4]) {
  using S = Surf<LOGN>;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const size_t i = q.off + q.jj + m * S::M;
    v[m] = q.on ? mk(f[i], f[i + S::N]) : zero<double>();
  }
}
template <int LOGN>
__device__ __forceinline__ void store_pair(double* __restrict__ f, const Pair& q, const cpx<double> (&v)[4]) {
  using S = Surf<LOGN>;
  if (!q.on) return;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const size_t i = q.off + q.jj + m * S::M;
    f[i] = v[m].x;
    f[i + S::N] = v[m].y;
  }
}

// transform of the packed rows v and their half spectra into X
template <int LOGN>
__device__ __forceinline__ void rows_out(cpx<double> (&v)[1][4], cpx<double>* buf, const Pair& q,
                                         const SurfTw<LOGN>& t, cpx<double>* __restrict__ X) {
  using S = Surf<LOGN>;
  constexpr int kxh = S::N / 2 + 1;
  surf_fft<LOGN, false, 1>(v, buf, 0, q.b, q.jj, t);
  cpx<double>* Xa = X + (size_t)2 * q.s * kxh;
  surf_store_spectra<LOGN>(v[0], buf + (surf_last<LOGN>(0) ^ 1) * S::TILE, q.b, q.jj, q.on, Xa, Xa + kxh);
}
template <int LOGN>
__device__ __forceinline__ void rows_in(cpx<double> (&v)[1][4], cpx<double>* buf, const Pair& q,
                                        const SurfTw<LOGN>& t, const cpx<double>* __restrict__ X) {
  constexpr int kxh = Surf<LOGN>::N / 2 + 1;
  const cpx<double>* Xa = X + (size_t)2 * q.s * kxh;
  surf_load_inverse<LOGN>(v, buf, q.b, q.jj, q.on, Xa, Xa + kxh, t);
}

template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_rows_fwd(const double* __restrict__ in,
                                                             cpx<double>* __restrict__ X, int ny,
                                                             const cpx<double>* __restrict__ tw) {
  __shared__ cpx<double> buf[2 * Surf<LOGN>::TILE];
  const Pair q = row_pair<LOGN>(ny);
  SurfTw<LOGN> t;
  cpx<double> v[1][4];
  load_pair<LOGN>(in, q, v[0]);
  surf_load_tw<LOGN>(tw, q.jj, t);
  rows_out<LOGN>(v, buf, q, t, X);
}

template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_rows_inv(const cpx<double>* __restrict__ X,
                                                             double* __restrict__ out, int ny,
                                                             const cpx<double>* __restrict__ tw) {
  __shared__ cpx<double> buf[2 * Surf<LOGN>::TILE];
  const Pair q = row_pair<LOGN>(ny);
  SurfTw<LOGN> t;
  surf_load_tw<LOGN>(tw, q.jj, t);
  cpx<double> v[1][4];
  rows_in<LOGN>(v, buf, q, t, X);
  store_pair<LOGN>(out, q, v[0]);
}

// W / (dA sum p_new) from the update's block sums, and the overlap count
template <int NW>
__device__ __forceinline__ double load_scale(const double* __restrict__ part, int ldp, int nb,
                                             const double* __restrict__ sc, double* sh, double& overlaps) {
  double s[2];
  part += PU * ldp;
  surf_totals<2, NW>(nb, sh, s, [&](int i, double (&a)[2]) {
    a[0] += part[i];
    a[1] += part[ldp + i];
  });
  overlaps = s[1];
  return s[0] > 0.0 ? sc[S_W] / (sc[S_DA] * s[0]) : 1.0;
}

// Column transform of length ny = 2^LOGN, multiplier, inverse transform, in
// place on X; one block holds SEQ columns.  part: multiply by the load scale
// of the update's block sums too.
template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_columns(cpx<double>* __restrict__ X, int nx, double lx,
                                                            double ly, double fac,
                                                            const cpx<double>* __restrict__ tw,
                                                            const double* __restrict__ part, int ldp, int nb,
                                                            const double* __restrict__ sc) {
  using S = Surf<LOGN>;
  __shared__ cpx<double> buf[2 * S::TILE];
  __shared__ double sh[2 * S::NW];
  const int kxh = nx / 2 + 1;
  const int b = threadIdx.x / S::M, jj = threadIdx.x & (S::M - 1);
  const int kx = xcd_block() * S::SEQ + b;
  const bool on = kx < kxh;
  SurfTw<LOGN> t;
  cpx<double> v[1][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) v[0][m] = on ? X[(size_t)(jj + m * S::M) * kxh + kx] : zero<double>();
  surf_load_tw<LOGN>(tw, jj, t);
  // the modes' factors (a square root and a division each) while the loads are
  // under way: 33.1 -> 31.6 us per iteration at 256^2, 43.3 -> 42.5 at 512^2
  const double twopi = 6.283185307179586476925286766559;
  const double q1 = twopi * kx / lx;
  double c[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int ky = jj + m * S::M;
    const int k2 = (ky * 2 <= S::N) ? ky : ky - S::N;
    const double q2 = twopi * k2 / ly;
    c[m] = (kx == 0 && ky == 0) ? 0.0 : fac / sqrt(q1 * q1 + q2 * q2);
  }
  if (part) {
    double ov;
    const double scale = load_scale<S::NW>(part, ldp, nb, sc, sh, ov);
#pragma unroll
    for (int m = 0; m < 4; ++m) c[m] *= scale;
  }
  surf_fft<LOGN, false, 1>(v, buf, 0, b, jj, t);
#pragma unroll
  for (int m = 0; m < 4; ++m) v[0][m] = scl(v[0][m], c[m]);
  surf_fft<LOGN, true, 1>(v, buf, surf_last<LOGN>(0) ^ 1, b, jj, t);
  if (!on) return;
#pragma unroll
  for (int m = 0; m < 4; ++m) X[(size_t)(jj + m * S::M) * kxh + kx] = v[0][m];
}

// p renormalised to the load (from the update's block sums; FIRST: as it
// is), g = M[p] - h
template <int LOGN, bool FIRST>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_pk_gap(const cpx<double>* __restrict__ X,
                                                           const double* __restrict__ h, double* __restrict__ p,
                                                           const double* __restrict__ pold,
                                                           double* __restrict__ g, int ny,
                                                           const cpx<double>* __restrict__ tw, double* part, int ldp,
                                                           int nb, double* sc) {
  using S = Surf<LOGN>;
  __shared__ cpx<double> buf[2 * S::TILE];
  __shared__ double sh[3 * S::NW];
  const Pair q = row_pair<LOGN>(ny);
  SurfTw<LOGN> t;
  cpx<double> v[1][4], pv[4], hv[4], po[4];
  if (!S::TIGHT) {
    load_pair<LOGN>(p, q, pv);
    load_pair<LOGN>(h, q, hv);
    if (!FIRST) load_pair<LOGN>(pold, q, po);
  }
  surf_load_tw<LOGN>(tw, q.jj, t);
  double scale = 1.0, ov = 0.0;
  if (!FIRST) scale = load_scale<S::NW>(part, ldp, nb, sc, sh, ov);
  rows_in<LOGN>(v, buf, q, t, X);
  if (S::TIGHT) {
    load_pair<LOGN>(p, q, pv);
    load_pair<LOGN>(h, q, hv);
    if (!FIRST) load_pair<LOGN>(pold, q, po);
  }
  double s[3] = {0.0, 0.0, 0.0}, o[3];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (!FIRST) {
      pv[m] = scl(pv[m], scale);
      s[0] += fabs(pv[m].x - po[m].x) + fabs(pv[m].y - po[m].y);
    }
    v[0][m] = sub(v[0][m], hv[m]);
    if (pv[m].x > 0.0) {
      s[1] += v[0][m].x;
      s[2] += 1.0;
    }
    if (pv[m].y > 0.0) {
      s[1] += v[0][m].y;
      s[2] += 1.0;
    }
  }
  if (!FIRST) {
    store_pair<LOGN>(p, q, pv);
    // a restart after an iteration that re-admitted points
    if (blockIdx.x == 0 && threadIdx.x == 0) sc[S_DELTA] = ov > 0.0 ? 0.0 : 1.0;
  }
  store_pair<LOGN>(g, q, v[0]);
  surf_sums<3, S::NW>(s, sh, o);
  const double gb = o[2] > 0.0 ? o[1] / o[2] : 0.0;
  double c[2] = {0.0, 0.0}, oc[2];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const double dx = v[0][m].x - gb, dy = v[0][m].y - gb;
    if (pv[m].x > 0.0) {
      c[0] += dx * dx;
      c[1] += dx;
    }
    if (pv[m].y > 0.0) {
      c[0] += dy * dy;
      c[1] += dy;
    }
  }
  surf_sums<2, S::NW>(c, sh, oc);
  const double w5[5] = {o[0], o[1], o[2], oc[0], oc[1]};
  surf_put<5>(part + PG * ldp, ldp, w5);
}

// mean of g on the contact set and its points
template <int NW>
__device__ __forceinline__ double gap_mean(const double* __restrict__ part, int ldp, int nb, double* sh,
                                           double& count) {
  double s[2];
  part += PG * ldp;
  surf_totals<2, NW>(nb, sh, s, [&](int i, double (&a)[2]) {
    a[0] += part[ldp + i];
    a[1] += part[2 * ldp + i];
  });
  count = s[1];
  return s[1] > 0.0 ? s[0] / s[1] : 0.0;
}

// g minus its mean on the contact set (after the last iteration)
__global__ __launch_bounds__(GT) void k_pk_gap_mean(double* __restrict__ g, int n, const double* __restrict__ part,
                                                   int ldp, int nb, double* sc) {
  __shared__ double sh[2 * GT / 64];
  double count;
  const double gbar = gap_mean<GT / 64>(part, ldp, nb, sh, count);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc[S_GBAR] = gbar;
    sc[S_CNT] = count;
  }
  for (int i = blockIdx.x * GT + threadIdx.x; i < n; i += gridDim.x * GT) g[i] -= gbar;
}

// conjugate direction on the contact set, 0 elsewhere, and its row spectra
template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_pk_dir(const double* __restrict__ p,
                                                           const double* __restrict__ g, double* __restrict__ t,
                                                           cpx<double>* __restrict__ X, int ny,
                                                           const cpx<double>* __restrict__ tw,
                                                           const double* __restrict__ part, int ldp, int nb,
                                                           double* sc) {
  using S = Surf<LOGN>;
  __shared__ cpx<double> buf[2 * S::TILE];
  __shared__ double sh[2 * S::NW];
  const Pair q = row_pair<LOGN>(ny);
  SurfTw<LOGN> w;
  cpx<double> v[1][4], pv[4], gv[4];
  load_pair<LOGN>(p, q, pv);
  load_pair<LOGN>(g, q, gv);
  load_pair<LOGN>(t, q, v[0]);
  if (!S::TIGHT) surf_load_tw<LOGN>(tw, q.jj, w);
  // The mean as gbar + glo: gbar alone is off by its rounding, which at the
  // gap's rounding floor is as large as the gap itself and, once in t, is
  // carried and amplified from direction to direction.
  double count, e[2];
  const double gbar = gap_mean<S::NW>(part, ldp, nb, sh, count);
  const double* pg = part + PG * ldp;
  surf_totals<2, S::NW>(nb, sh, e, [&](int i, double (&a)[2]) {
    const double ni = pg[2 * ldp + i];
    if (ni > 0.0) {
      const double d = pg[ldp + i] / ni - gbar, D = pg[4 * ldp + i];
      a[0] += pg[3 * ldp + i] + d * (2.0 * D + ni * d);
      a[1] += D + ni * d;
    }
  });
  const double glo = count > 0.0 ? e[1] / count : 0.0;
  const double G = e[0] - e[1] * glo;
  const double gold = sc[S_GOLD];
  const double beta = gold > 0.0 ? sc[S_DELTA] * G / gold : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc[S_G] = G;                        // S_GOLD of the next iteration (k_pk_curv)
    sc[S_GBAR] = gbar;
    sc[S_GLO] = glo;
  }
  // beta = 0 (first iteration, restart) must not take the previous
  // direction: 0 * t would carry a NaN through
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    v[0][m].x = pv[m].x > 0.0 ? gv[m].x - gbar - glo + (beta != 0.0 ? beta * v[0][m].x : 0.0) : 0.0;
    v[0][m].y = pv[m].y > 0.0 ? gv[m].y - gbar - glo + (beta != 0.0 ? beta * v[0][m].y : 0.0) : 0.0;
  }
  store_pair<LOGN>(t, q, v[0]);
  if (S::TIGHT) surf_load_tw<LOGN>(tw, q.jj, w);
  rows_out<LOGN>(v, buf, q, w, X);
}

// r = M[t]: sums over the contact set for the step (g taken about its mean)
template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_pk_curv(const cpx<double>* __restrict__ X,
                                                            const double* __restrict__ p,
                                                            const double* __restrict__ g,
                                                            const double* __restrict__ t, int ny,
                                                            const cpx<double>* __restrict__ tw, double* part, int ldp,
                                                            double* sc) {
  using S = Surf<LOGN>;
  __shared__ cpx<double> buf[2 * S::TILE];
  __shared__ double sh[4 * S::NW];
  const Pair q = row_pair<LOGN>(ny);
  SurfTw<LOGN> w;
  cpx<double> v[1][4], pv[4], gv[4], tv[4];
  if (!S::TIGHT) {
    load_pair<LOGN>(p, q, pv);
    load_pair<LOGN>(g, q, gv);
    load_pair<LOGN>(t, q, tv);
  }
  surf_load_tw<LOGN>(tw, q.jj, w);
  const double gbar = sc[S_GBAR], glo = sc[S_GLO];
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[S_GOLD] = sc[S_G];
  rows_in<LOGN>(v, buf, q, w, X);
  if (S::TIGHT) {
    load_pair<LOGN>(p, q, pv);
    load_pair<LOGN>(g, q, gv);
    load_pair<LOGN>(t, q, tv);
  }
  double s[4] = {0.0, 0.0, 0.0, 0.0}, o[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (pv[m].x > 0.0) {
      s[0] += (gv[m].x - gbar - glo) * tv[m].x;
      s[1] += v[0][m].x;
      s[2] += tv[m].x;
      s[3] += 1.0;
    }
    if (pv[m].y > 0.0) {
      s[0] += (gv[m].y - gbar - glo) * tv[m].y;
      s[1] += v[0][m].y;
      s[2] += tv[m].y;
      s[3] += 1.0;
    }
  }
  surf_sums<4, S::NW>(s, sh, o);
  const double rb = o[3] > 0.0 ? o[1] / o[3] : 0.0, tb = o[3] > 0.0 ? o[2] / o[3] : 0.0;
  double c[1] = {0.0}, oc[1];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (pv[m].x > 0.0) c[0] += (v[0][m].x - rb) * (tv[m].x - tb);
    if (pv[m].y > 0.0) c[0] += (v[0][m].y - rb) * (tv[m].y - tb);
  }
  surf_sums<1, S::NW>(c, sh, oc);
  const double w5[5] = {o[0], o[1], o[2], o[3], oc[0]};
  surf_put<5>(part + PR * ldp, ldp, w5);
}

// step, projection onto p >= 0, re-admission of the overlap set (points of
// negative gap enter with a pressure proportional to the overlap; when the
// conjugate-gradient step vanishes -- the gap already uniform on the contact
// set, e.g. a set of one point -- with the step of a point load, 1 / M_ii);
// block sums of the new pressure and of the points that entered, row spectra
__device__ __forceinline__ double pk_step(double p, double g, double t, double tau, double tre, double& entered) {
  double pn = p - tau * t;
  if (pn < 0.0) pn = 0.0;
  if (pn == 0.0 && g < 0.0) {
    pn = -tre * g;
    entered += 1.0;
  }
  return pn;
}

template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_pk_update(double* __restrict__ p, double* __restrict__ pold,
                                                              const double* __restrict__ g,
                                                              const double* __restrict__ t,
                                                              cpx<double>* __restrict__ X, int ny,
                                                              const cpx<double>* __restrict__ tw, double* part,
                                                              int ldp, int nb, const double* __restrict__ sc) {
  using S = Surf<LOGN>;
  __shared__ cpx<double> buf[2 * S::TILE];
  __shared__ double sh[4 * S::NW];
  const Pair q = row_pair<LOGN>(ny);
  SurfTw<LOGN> w;
  cpx<double> v[1][4], gv[4], tv[4];
  load_pair<LOGN>(p, q, v[0]);
  load_pair<LOGN>(g, q, gv);
  load_pair<LOGN>(t, q, tv);
  if (!S::TIGHT) surf_load_tw<LOGN>(tw, q.jj, w);
  const double gbar = sc[S_GBAR], glo = sc[S_GLO];
  const double* pr = part + PR * ldp;
  double a[4], den[1];
  surf_totals<4, S::NW>(nb, sh, a, [&](int i, double (&x)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] += pr[k * ldp + i];
  });
  const double rbar = a[3] > 0.0 ? a[1] / a[3] : 0.0, tbar = a[3] > 0.0 ? a[2] / a[3] : 0.0;
  surf_totals<1, S::NW>(nb, sh, den, [&](int i, double (&x)[1]) {
    const double ni = pr[3 * ldp + i];
    if (ni > 0.0) x[0] += pr[4 * ldp + i] + ni * (pr[ldp + i] / ni - rbar) * (pr[2 * ldp + i] / ni - tbar);
  });
  const double tau = den[0] != 0.0 ? a[0] / den[0] : 0.0;
  const double tre = tau != 0.0 ? tau : sc[S_TAU0];
  store_pair<LOGN>(pold, q, v[0]);
  double s[2] = {0.0, 0.0}, o[2];
  if (q.on) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      v[0][m].x = pk_step(v[0][m].x, gv[m].x - gbar - glo, tv[m].x, tau, tre, s[1]);
      v[0][m].y = pk_step(v[0][m].y, gv[m].y - gbar - glo, tv[m].y, tau, tre, s[1]);
      s[0] += v[0][m].x + v[0][m].y;
    }
  }
  store_pair<LOGN>(p, q, v[0]);
  surf_sums<2, S::NW>(s, sh, o);
  surf_put<2>(part + PU * ldp, ldp, o);
  if (S::TIGHT) surf_load_tw<LOGN>(tw, q.jj, w);
  rows_out<LOGN>(v, buf, q, w, X);
}

__global__ __launch_bounds__(GT) void k_pk_err(const double* __restrict__ part, int ldp, int nb, double* sc,
                                              double* mirror) {
  __shared__ double sh[GT / 64];
  double s[1];
  part += PG * ldp;
  surf_totals<1, GT / 64>(nb, sh, s, [&](int i, double (&a)[1]) { a[0] += part[i]; });
  if (threadIdx.x == 0) {
    const double err = sc[S_DA] * s[0] / sc[S_W];
    sc[S_ERR] = err;
    mirror[S_ERR] = err;
  }
}

// ---------------------------------------------------- one-workgroup iteration
// Small surfaces (16 to 64 points a side) by one workgroup: every thread keeps its
// row pair's p, g, t and h in registers and the half spectrum X is in LDS (34 KiB
// at 64 x 64), so an iteration has barriers where the launches above have kernel
// boundaries, and the convergence test is in the loop.  Bound by that chain of
// barriers (about 45 per iteration) and, at 64 x 64, by one CU's LDS.  us per
// iteration of a solve to 1e-12, launches with a test on the host after each
// iteration -> one workgroup: 16^2 39.5 -> 6.2, 64 x 16 40.5 -> 8.9, 32^2 41.0 -> 10.9,
// 64^2 42.2 -> 20.9.  (128^2 does not fit the LDS; its launches take 28.2.)
template <int LX, int LY>
struct Solo {
  static constexpr int NX = 1 << LX, NY = 1 << LY, KXH = NX / 2 + 1;
  static constexpr int NTH = NX * NY / 8 < 64 ? 64 : NX * NY / 8, NW = NTH / 64;
  static constexpr int WT = 2 * (Surf<LX>::TILE > Surf<LY>::TILE ? Surf<LX>::TILE : Surf<LY>::TILE);
  static constexpr int COLS = NW * Surf<LY>::SEQ;    // columns transformed at a time
  static constexpr int PASSES = (KXH + COLS - 1) / COLS;
};

template <int LX, int LY>
__global__ __launch_bounds__((Solo<LX, LY>::NTH)) void k_pk_solo(PkBufs a, int count, double tol, int first,
                                                              int last) {
  using C = Solo<LX, LY>;
  using SX = Surf<LX>;
  using SY = Surf<LY>;
  constexpr int NW = C::NW, KXH = C::KXH;
  __shared__ cpx<double> X[C::NY * KXH];
  __shared__ cpx<double> tiles[NW * C::WT];
  __shared__ double sh[4 * NW];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  cpx<double>* buf = tiles + wave * C::WT;           // each wave's sequences have tiles of their own
  Pair q;
  q.b = lane / SX::M;
  q.jj = lane & (SX::M - 1);
  q.s = wave * SX::SEQ + q.b;
  q.on = 2 * q.s < C::NY;
  q.off = (size_t)2 * q.s * C::NX;
  cpx<double>* Xa = X + (q.on ? 2 * q.s * KXH : 0);
  cpx<double>* Xb = Xa + KXH;
  const int cb = lane / SY::M, cj = lane & (SY::M - 1);
  SurfTw<LX> tx;
  SurfTw<LY> ty;
  surf_load_tw<LX>(a.twx, q.jj, tx);
  surf_load_tw<LY>(a.twy, cj, ty);
  double mult[C::PASSES][4];
  {
    const double twopi = 6.283185307179586476925286766559;
    const double fac = 2.0 / a.estar / ((double)C::NX * C::NY);
#pragma unroll
    for (int u = 0; u < C::PASSES; ++u) {
      const int kx = u * C::COLS + wave * SY::SEQ + cb;
      const double q1 = twopi * kx / a.lx;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int ky = cj + m * SY::M;
        const int k2 = (ky * 2 <= C::NY) ? ky : ky - C::NY;
        const double q2 = twopi * k2 / a.ly;
        mult[u][m] = (kx == 0 && ky == 0) ? 0.0 : fac / sqrt(q1 * q1 + q2 * q2);
      }
    }
  }
  // v <- M[v]
  auto comply = [&](cpx<double> (&v)[1][4]) {
    __syncthreads();                                 // the last call's tiles have been read
    surf_fft<LX, false, 1>(v, buf, 0, q.b, q.jj, tx);
    surf_store_spectra<LX>(v[0], buf + (surf_last<LX>(0) ^ 1) * SX::TILE, q.b, q.jj, q.on, Xa, Xb);
#pragma unroll
    for (int u = 0; u < C::PASSES; ++u) {
      __syncthreads();
      const int kx = u * C::COLS + wave * SY::SEQ + cb;
      const bool on = kx < KXH;
      cpx<double> z[1][4];
#pragma unroll
      for (int m = 0; m < 4; ++m) z[0][m] = on ? X[(cj + m * SY::M) * KXH + kx] : zero<double>();
      surf_fft<LY, false, 1>(z, buf, 0, cb, cj, ty);
#pragma unroll
      for (int m = 0; m < 4; ++m) z[0][m] = scl(z[0][m], mult[u][m]);
      surf_fft<LY, true, 1>(z, buf, surf_last<LY>(0) ^ 1, cb, cj, ty);
      if (on) {
#pragma unroll
        for (int m = 0; m < 4; ++m) X[(cj + m * SY::M) * KXH + kx] = z[0][m];
      }
    }
    __syncthreads();
    surf_load_inverse<LX>(v, buf, q.b, q.jj, q.on, Xa, Xb, tx);
  };
  cpx<double> p[4], g[4], t[4], h[4], v[1][4];
  load_pair<LX>(a.p, q, p);
  load_pair<LX>(a.h, q, h);
  double dp = 0.0, o[3];
  // the sums over the contact set of the gap: sum |p - p_old|, sum g, points
  auto gap_sums = [&]() {
    double s[3] = {dp, 0.0, 0.0};
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      if (p[m].x > 0.0) { s[1] += g[m].x; s[2] += 1.0; }
      if (p[m].y > 0.0) { s[1] += g[m].y; s[2] += 1.0; }
    }
    surf_sums<3, NW>(s, sh, o);
  };
  double delta = 0.0, gold = 1.0;
  if (first) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      t[m] = zero<double>();
      v[0][m] = p[m];
    }
    comply(v);
#pragma unroll
    for (int m = 0; m < 4; ++m) g[m] = sub(v[0][m], h[m]);
  } else {
    load_pair<LX>(a.g, q, g);
    load_pair<LX>(a.t, q, t);
    delta = a.sc[S_DELTA];
    gold = a.sc[S_GOLD];
  }
  const double W = a.sc[S_W], dA = a.sc[S_DA], tau0 = a.sc[S_TAU0];
  gap_sums();
  double err = 0.0;
  int it = 0;
  bool stop = false;
  while (it < count && !stop) {                      // (uniform: every thread has the same sums)
    ++it;
    // direction (k_pk_dir)
    const double cnt = o[2], gbar = cnt > 0.0 ? o[1] / cnt : 0.0;
    double c2[2] = {0.0, 0.0}, e[2];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const double dx = g[m].x - gbar, dy = g[m].y - gbar;
      if (p[m].x > 0.0) { c2[0] += dx * dx; c2[1] += dx; }
      if (p[m].y > 0.0) { c2[0] += dy * dy; c2[1] += dy; }
    }
    surf_sums<2, NW>(c2, sh, e);
    const double glo = cnt > 0.0 ? e[1] / cnt : 0.0;
    const double G = e[0] - e[1] * glo;
    const double beta = gold > 0.0 ? delta * G / gold : 0.0;
    gold = G;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      t[m].x = p[m].x > 0.0 ? g[m].x - gbar - glo + (beta != 0.0 ? beta * t[m].x : 0.0) : 0.0;
      t[m].y = p[m].y > 0.0 ? g[m].y - gbar - glo + (beta != 0.0 ? beta * t[m].y : 0.0) : 0.0;
      v[0][m] = t[m];
    }
    comply(v);
    // step (k_pk_curv, k_pk_update)
    double s4[4] = {0.0, 0.0, 0.0, 0.0}, r[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      if (p[m].x > 0.0) { s4[0] += (g[m].x - gbar - glo) * t[m].x; s4[1] += v[0][m].x; s4[2] += t[m].x; }
      if (p[m].y > 0.0) { s4[0] += (g[m].y - gbar - glo) * t[m].y; s4[1] += v[0][m].y; s4[2] += t[m].y; }
    }
    surf_sums<4, NW>(s4, sh, r);
    const double rbar = cnt > 0.0 ? r[1] / cnt : 0.0, tbar = cnt > 0.0 ? r[2] / cnt : 0.0;
    double c1[1] = {0.0}, den[1];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      if (p[m].x > 0.0) c1[0] += (v[0][m].x - rbar) * (t[m].x - tbar);
      if (p[m].y > 0.0) c1[0] += (v[0][m].y - rbar) * (t[m].y - tbar);
    }
    surf_sums<1, NW>(c1, sh, den);
    const double tau = den[0] != 0.0 ? r[0] / den[0] : 0.0;
    const double tre = tau != 0.0 ? tau : tau0;
    double s2[2] = {0.0, 0.0}, n[2];
    cpx<double> pn[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) pn[m] = p[m];
    if (q.on) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        pn[m].x = pk_step(p[m].x, g[m].x - gbar - glo, t[m].x, tau, tre, s2[1]);
        pn[m].y = pk_step(p[m].y, g[m].y - gbar - glo, t[m].y, tau, tre, s2[1]);
        s2[0] += pn[m].x + pn[m].y;
      }
    }
    surf_sums<2, NW>(s2, sh, n);
    // load renormalised, a restart after re-admission, new gap (k_pk_gap)
    const double scale = n[0] > 0.0 ? W / (dA * n[0]) : 1.0;
    delta = n[1] > 0.0 ? 0.0 : 1.0;
    dp = 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      pn[m] = scl(pn[m], scale);
      dp += fabs(pn[m].x - p[m].x) + fabs(pn[m].y - p[m].y);
      p[m] = pn[m];
      v[0][m] = pn[m];
    }
    comply(v);
#pragma unroll
    for (int m = 0; m < 4; ++m) g[m] = sub(v[0][m], h[m]);
    gap_sums();
    err = dA * o[0] / W;
    stop = !(err >= tol && err <= 1.7976931348623157e308);     // converged or not finite
  }
  const double gbar = o[2] > 0.0 ? o[1] / o[2] : 0.0;
  if (stop || last) {
#pragma unroll
    for (int m = 0; m < 4; ++m) g[m] = mk(g[m].x - gbar, g[m].y - gbar);
  }
  store_pair<LX>(a.p, q, p);
  store_pair<LX>(a.g, q, g);
  store_pair<LX>(a.t, q, t);
  if (threadIdx.x == 0) {
    a.sc[S_DELTA] = delta;
    a.sc[S_GOLD] = gold;
    a.sc[S_GBAR] = gbar;
    a.sc[S_CNT] = o[2];
    a.sc[S_ERR] = a.mirror[S_ERR] = err;
    a.mirror[S_IT] = (double)it;
  }
}

hipError_t launch_columns(int nx, int ny, double lx, double ly, double estar, const cpx<double>* twy,
                          cpx<double>* X, const double* part, int ldp, int nb, const double* sc, hipStream_t st) {
  const double fac = 2.0 / estar / ((double)nx * ny);
  const int kxh = nx / 2 + 1;
#define CALL(L)                                                                                              \
  hipLaunchKernelGGL((k_columns<L>), dim3((unsigned)((kxh + Surf<L>::SEQ - 1) / Surf<L>::SEQ)),              \
                     dim3(Surf<L>::NTH), 0, st, X, nx, lx, ly, fac, twy, part, ldp, nb, sc)
  FVIM_SURF_SWITCH(surf_log2(ny), CALL)
#undef CALL
  return hipGetLastError();
}

}  // namespace

int pk_part_count(int nx, int ny) { return PROWS * pk_ldp(nx, ny); }

hipError_t launch_rows_fwd(int nx, int ny, const double* in, cpx<double>* X, const cpx<double>* twx, hipStream_t st) {
#define CALL(L) \
  hipLaunchKernelGGL((k_rows_fwd<L>), dim3(pk_row_blocks(nx, ny)), dim3(Surf<L>::NTH), 0, st, in, X, ny, twx)
  FVIM_SURF_SWITCH(surf_log2(nx), CALL)
#undef CALL
  return hipGetLastError();
}

hipError_t launch_rows_inv(int nx, int ny, const cpx<double>* X, double* out, const cpx<double>* twx, hipStream_t st) {
#define CALL(L) \
  hipLaunchKernelGGL((k_rows_inv<L>), dim3(pk_row_blocks(nx, ny)), dim3(Surf<L>::NTH), 0, st, X, out, ny, twx)
  FVIM_SURF_SWITCH(surf_log2(nx), CALL)
#undef CALL
  return hipGetLastError();
}

hipError_t launch_compliance(int nx, int ny, double lx, double ly, double estar, const cpx<double>* twx,
                             const cpx<double>* twy, const double* in, double* out, cpx<double>* X, hipStream_t st) {
  hipError_t e = launch_rows_fwd(nx, ny, in, X, twx, st);
  if (e == hipSuccess) e = launch_columns(nx, ny, lx, ly, estar, twy, X, nullptr, 0, 0, nullptr, st);
  return e == hipSuccess ? launch_rows_inv(nx, ny, X, out, twx, st) : e;
}

hipError_t launch_pk_first(const PkBufs& b, hipStream_t st) {
  const int ldp = pk_ldp(b.nx, b.ny), nbr = pk_row_blocks(b.nx, b.ny);
  hipError_t e = launch_rows_fwd(b.nx, b.ny, b.p, b.X, b.twx, st);
  if (e != hipSuccess) return e;
  e = launch_columns(b.nx, b.ny, b.lx, b.ly, b.estar, b.twy, b.X, nullptr, 0, 0, nullptr, st);
  if (e != hipSuccess) return e;
#define CALL(L)                                                                                               \
  hipLaunchKernelGGL((k_pk_gap<L, true>), dim3(nbr), dim3(Surf<L>::NTH), 0, st, b.X, b.h, b.p, b.pold, b.g, b.ny, \
                     b.twx, b.part, ldp, nbr, b.sc)
  FVIM_SURF_SWITCH(surf_log2(b.nx), CALL)
#undef CALL
  return hipGetLastError();
}

hipError_t launch_pk_gap_mean(const PkBufs& b, hipStream_t st) {
  const int n = b.nx * b.ny;
  hipLaunchKernelGGL(k_pk_gap_mean, dim3(std::min((n + GT - 1) / GT, GB)), dim3(GT), 0, st, b.g, n, b.part,
                     pk_ldp(b.nx, b.ny), pk_row_blocks(b.nx, b.ny), b.sc);
  return hipGetLastError();
}

hipError_t launch_pk_iteration(const PkBufs& b, hipStream_t st) {
  const int ldp = pk_ldp(b.nx, b.ny), nbr = pk_row_blocks(b.nx, b.ny);
  hipError_t e;
#define CALL(L)                                                                                                    \
  hipLaunchKernelGGL((k_pk_dir<L>), dim3(nbr), dim3(Surf<L>::NTH), 0, st, b.p, b.g, b.t, b.X, b.ny, b.twx, b.part, \
                     ldp, nbr, b.sc)
  FVIM_SURF_SWITCH(surf_log2(b.nx), CALL)
#undef CALL
  if ((e = launch_columns(b.nx, b.ny, b.lx, b.ly, b.estar, b.twy, b.X, nullptr, 0, 0, nullptr, st)) != hipSuccess)
    return e;
#define CALL(L)                                                                                                     \
  hipLaunchKernelGGL((k_pk_curv<L>), dim3(nbr), dim3(Surf<L>::NTH), 0, st, b.X, b.p, b.g, b.t, b.ny, b.twx, b.part, \
                     ldp, b.sc)
  FVIM_SURF_SWITCH(surf_log2(b.nx), CALL)
#undef CALL
#define CALL(L)                                                                                                   \
  hipLaunchKernelGGL((k_pk_update<L>), dim3(nbr), dim3(Surf<L>::NTH), 0, st, b.p, b.pold, b.g, b.t, b.X, b.ny,    \
                     b.twx, b.part, ldp, nbr, b.sc)
  FVIM_SURF_SWITCH(surf_log2(b.nx), CALL)
#undef CALL
  if ((e = launch_columns(b.nx, b.ny, b.lx, b.ly, b.estar, b.twy, b.X, b.part, ldp, nbr, b.sc, st)) != hipSuccess)
    return e;
#define CALL(L)                                                                                                \
  hipLaunchKernelGGL((k_pk_gap<L, false>), dim3(nbr), dim3(Surf<L>::NTH), 0, st, b.X, b.h, b.p, b.pold, b.g,   \
                     b.ny, b.twx, b.part, ldp, nbr, b.sc)
  FVIM_SURF_SWITCH(surf_log2(b.nx), CALL)
#undef CALL
  return hipGetLastError();
}

// 16: the threads of a shorter side would not fill a wave; 64: see k_pk_solo.  (Longer
// sides of as few points, 128 x 16, would fit too: not built, six launches.)
bool pk_solo_fits(int nx, int ny) { return nx >= 16 && nx <= 64 && ny >= 16 && ny <= 64; }

hipError_t launch_pk_solo(const PkBufs& b, int count, double tol, bool first, bool last, hipStream_t st) {
#define CASE(LX, LY)                                                                                            \
  case LX * 16 + LY:                                                                                            \
    hipLaunchKernelGGL((k_pk_solo<LX, LY>), dim3(1), dim3(Solo<LX, LY>::NTH), 0, st, b, count, tol, first, last); \
    break;
  switch (surf_log2(b.nx) * 16 + surf_log2(b.ny)) {
    CASE(4, 4) CASE(4, 5) CASE(4, 6) CASE(5, 4) CASE(5, 5) CASE(5, 6) CASE(6, 4) CASE(6, 5) CASE(6, 6)
    default: return hipErrorInvalidValue;
  }
#undef CASE
  return hipGetLastError();
}

hipError_t launch_pk_err(const PkBufs& b, hipStream_t st) {
  hipLaunchKernelGGL(k_pk_err, dim3(1), dim3(GT), 0, st, b.part, pk_ldp(b.nx, b.ny), pk_row_blocks(b.nx, b.ny), b.sc,
                     b.mirror);
  return hipGetLastError();
}

}  // namespace fvim
