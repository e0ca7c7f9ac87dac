// Tangential (Coulomb, partial-slip) contact under a given normal pressure:
// the friction Sec. 5.1 says the contact step can include.  Normal and
// tangential problems are uncoupled (Goodman's approximation); the
// tangential surface traction q = (q1, q2) minimises the complementary
// energy 1/2 <q, C q> over |q_i| <= mu_f p_i with the total tangential force
// dA sum q = Q prescribed, C the tangential block of the half-space surface
// compliance: per mode, (2 (1 + nu) / (E |k|)) (I - nu n n^T), n = k / |k|,
// k = 0 dropped, n1 n2 averaged to 0 over the sign replicas of a Nyquist
// line.  Its optimality conditions are the stick/slip conditions (one rigid
// shift of the stick zone; slip against the traction where it is on the
// friction limit).
//
// Accelerated projected gradient (FISTA) with gradient restart, step 1 / L,
// L the largest eigenvalue of C.  One iteration, all on the device with no
// host round trip, in the five launches its global sums allow:
//   columns   u = C y: column transforms of both components' row spectra, the
//             2x2 multiplier, inverse column transforms, in place
//   grad      rows transformed back, v = y - u / L;  sums of P(v + lam)
//   sums      Newton step on lam;                    sums of P(v + lam)
//   apply     Newton step on lam; q_new = P(v + lam); change, restart test
//   momentum  restart or momentum; y and q updated, the rows of y transformed
// P is the projection onto the disks |.| <= mu_f p_i, lam (2 values) the root
// of dA sum P(v + lam) = Q, found by two warm-started Newton steps (sums of P
// and of its 2x2 Jacobian); the restart test is <y - q_new, q_new - q> > 0.
// A row transform carries the two components of one row as one complex
// sequence.  Block sums are totalled, in one fixed order, by each block of the
// kernel that uses them.  The separate form (a 5-launch compliance, 7 more
// launches) was bound by launch latency: a solve at 512^2 132 ms against 75 (38 us
// per iteration).
// The host reads the change measure dA sum |q_new - q| / (mu_f W) every few
// iterations.
//
// Coupled form (frictional_contact_solve, coupled = 1): for nu < 1/2 the
// Boussinesq-Cerruti surface response has cross terms, per mode
// u_a = K_a t3 and u3 = sum_a conj(K_a) t_a with K_a = i (1 - 2 nu) n_a /
// (2 mu |k|) (0 at k = 0 and on the Nyquist line of axis a).  The pressure
// then solves the normal problem on h - u3[q] and q the tangential problem
// with the extra displacement u_t[p] (added to C y in the gradient step);
// the two solves alternate, each warm-started from the last, until
// dA sum |dp| / W + dA sum |dq| / (mu_f W) < tol.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "common.hpp"
#include "contact.hpp"
#include "solver.hpp"
#include "surf_dev.hpp"

namespace fvim {
namespace {

constexpr int NT = 256;
constexpr int RB = 1024;               // max reduction blocks
constexpr int PB = 256;                // most blocks of the pointwise iteration kernels
constexpr int WARM = 8;                // Newton steps of the projection of a warm start
constexpr int CHECK = 8;               // iterations between host checks

// device scalars
// (F_LAMA, F_LAMB: lam before and after an odd Newton step; F_TN: the next F_T)
enum { F_LAMA = 0, F_LAMB = 2, F_T = 4, F_TN, F_CHANGE, F_SUMP, F_STICK, F_CONTACT, F_CP, F_CQ, F_NSC = 16 };

template <int NS>
__device__ __forceinline__ void fblock_sums(double (&v)[NS], double* part) {
  __shared__ double sh[NS][NT / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    double x = v[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
    if (lane == 0) sh[k][w] = x;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      double s = 0.0;
      for (int i = 0; i < NT / 64; ++i) s += sh[k][i];
      part[k * RB + blockIdx.x] = s;
    }
  }
}

// total of the nb partials of row k, one block, fixed order
__device__ double ffinal(const double* part, int k, int nb) {
  __shared__ double sh[NT];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += NT) s += part[k * RB + i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = NT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  double r = sh[0];
  __syncthreads();
  return r;
}

// projection of w onto the disk |.| <= rho: P and its Jacobian (a, b, c) =
// [[a, b], [b, c]]
__device__ __forceinline__ void disk(double w0, double w1, double rho, double& p0, double& p1, double& ja,
                                     double& jb, double& jc) {
  const double r = sqrt(w0 * w0 + w1 * w1);
  if (r <= rho) {
    p0 = w0;
    p1 = w1;
    ja = 1.0;
    jb = 0.0;
    jc = 1.0;
    return;
  }
  const double s = rho / r, a = s / (r * r);
  p0 = s * w0;
  p1 = s * w1;
  ja = s - a * w0 * w0;
  jb = -a * w0 * w1;
  jc = s - a * w1 * w1;
}

// rho = mu_f p; block sums of p (negative pressures, which a contact
// solution does not hold, count as 0)
__global__ __launch_bounds__(NT) void k_f_rho(const double* __restrict__ p, double mu, double* __restrict__ rho,
                                             size_t n, double* part) {
  double v[1] = {0.0};
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT) {
    const double pi = fmax(p[i], 0.0);
    rho[i] = mu * pi;
    v[0] += pi;
  }
  fblock_sums<1>(v, part);
}

// q = y = (c0, c1) rho (the full-slip field scaled to the load)
__global__ __launch_bounds__(NT) void k_f_init(const double* __restrict__ rho, double* __restrict__ q,
                                              double* __restrict__ y, size_t n, double c0, double c1) {
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT) {
    const double r = rho[i];
    q[i] = y[i] = c0 * r;
    q[n + i] = y[n + i] = c1 * r;
  }
}

// one row of both components as one complex sequence
struct Row {
  int b, jj, y;
  bool on;
  size_t off;
};
template <int LOGN>
__device__ __forceinline__ Row one_row(int ny) {
  using S = Surf<LOGN>;
  Row q;
  q.b = threadIdx.x / S::M;
  q.jj = threadIdx.x & (S::M - 1);
  q.y = blockIdx.x * S::SEQ + q.b;
  q.on = q.y < ny;
  q.off = (size_t)q.y * S::N;
  return q;
}
// the components (f[0 .. n), f[n .. 2 n)) at x = jj + m M of the row
template <int LOGN>
__device__ __forceinline__ void load_row(const double* __restrict__ f, size_t n, const Row& q, cpx<double> (&v)[4]) {
  using S = Surf<LOGN>;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const size_t i = q.off + q.jj + m * S::M;
    v[m] = q.on ? mk(f[i], f[n + i]) : zero<double>();
  }
}
template <int LOGN>
__device__ __forceinline__ void store_row(double* __restrict__ f, size_t n, const Row& q, const cpx<double> (&v)[4]) {
  using S = Surf<LOGN>;
  if (!q.on) return;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const size_t i = q.off + q.jj + m * S::M;
    f[i] = v[m].x;
    f[n + i] = v[m].y;
  }
}
template <int LOGN>
__device__ __forceinline__ void row_out(cpx<double> (&v)[1][4], cpx<double>* buf, const Row& q, int ny,
                                        const SurfTw<LOGN>& t, cpx<double>* __restrict__ X) {
  using S = Surf<LOGN>;
  constexpr int kxh = S::N / 2 + 1;
  surf_fft<LOGN, false, 1>(v, buf, 0, q.b, q.jj, t);
  cpx<double>* Xa = X + (size_t)q.y * kxh;
  surf_store_spectra<LOGN>(v[0], buf + (surf_last<LOGN>(0) ^ 1) * S::TILE, q.b, q.jj, q.on, Xa,
                           Xa + (size_t)ny * kxh);
}
template <int LOGN>
__device__ __forceinline__ void row_in(cpx<double> (&v)[1][4], cpx<double>* buf, const Row& q, int ny,
                                       const SurfTw<LOGN>& t, const cpx<double>* __restrict__ X) {
  constexpr int kxh = Surf<LOGN>::N / 2 + 1;
  const cpx<double>* Xa = X + (size_t)q.y * kxh;
  surf_load_inverse<LOGN>(v, buf, q.b, q.jj, q.on, Xa, Xa + (size_t)ny * kxh, t);
}

// row spectra of both components of in, and back
template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_f_rows_fwd(const double* __restrict__ in,
                                                               cpx<double>* __restrict__ X, int ny,
                                                               const cpx<double>* __restrict__ tw) {
  __shared__ cpx<double> buf[2 * Surf<LOGN>::TILE];
  const Row q = one_row<LOGN>(ny);
  SurfTw<LOGN> t;
  cpx<double> v[1][4];
  load_row<LOGN>(in, (size_t)ny * Surf<LOGN>::N, q, v[0]);
  surf_load_tw<LOGN>(tw, q.jj, t);
  row_out<LOGN>(v, buf, q, ny, t, X);
}
template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_f_rows_inv(const cpx<double>* __restrict__ X,
                                                               double* __restrict__ out, int ny,
                                                               const cpx<double>* __restrict__ tw) {
  __shared__ cpx<double> buf[2 * Surf<LOGN>::TILE];
  const Row q = one_row<LOGN>(ny);
  SurfTw<LOGN> t;
  cpx<double> v[1][4];
  surf_load_tw<LOGN>(tw, q.jj, t);
  row_in<LOGN>(v, buf, q, ny, t, X);
  store_row<LOGN>(out, (size_t)ny * Surf<LOGN>::N, q, v[0]);
}

// Multipliers of a mode (a, b: planes 0 and 1), with the 1 / (nx ny) of the
// inverse transform:
// COMPLIANCE: the 2x2 tangential compliance;
// N2T: plane 0 (the pressure) -> planes 0, 1: u_a = K_a p;
// T2N: planes 0, 1 (the tangential traction) -> plane 0: u3 = sum conj(K_a) q_a.
// K_a = i c n_a, c = (1 - 2 nu) / (2 mu |k|); K_1 = 0 on the Nyquist line of
// x, K_2 = 0 on the one of y; mode 0 dropped.
enum { COMPLIANCE = 0, N2T = 1, T2N = 2 };
struct ModeMat {
  double lx, ly, fac, nu, mu;           // fac = 1 / (nx ny)
};
template <int OP>
__device__ __forceinline__ void mode_apply(cpx<double>& a, cpx<double>& b, int kx, int ky, int nx, int ny,
                                           const ModeMat& c) {
  const int k2 = (ky * 2 <= ny) ? ky : ky - ny;
  const double twopi = 6.283185307179586476925286766559;
  const double q1 = twopi * kx / c.lx, q2 = twopi * k2 / c.ly;
  const double q = sqrt(q1 * q1 + q2 * q2);
  const bool mean = kx == 0 && ky == 0;
  if (OP == COMPLIANCE) {
    const double f = mean ? 0.0 : c.fac / (c.mu * q), n1 = mean ? 0.0 : q1 / q, n2 = mean ? 0.0 : q2 / q;
    const bool nyq = (kx * 2 == nx) || (ky * 2 == ny);
    const double c11 = f * (1.0 - c.nu * n1 * n1), c22 = f * (1.0 - c.nu * n2 * n2);
    const double c12 = nyq ? 0.0 : -f * c.nu * n1 * n2;
    const cpx<double> x = a, y = b;
    a = mk(c11 * x.x + c12 * y.x, c11 * x.y + c12 * y.y);
    b = mk(c12 * x.x + c22 * y.x, c12 * x.y + c22 * y.y);
    return;
  }
  double c1 = 0.0, c2 = 0.0;            // c n_a, with the Nyquist zeros
  if (!mean) {
    const double cq = c.fac * (1.0 - 2.0 * c.nu) / (2.0 * c.mu * q * q);
    if (kx * 2 != nx) c1 = cq * q1;
    if (ky * 2 != ny) c2 = cq * q2;
  }
  if (OP == N2T) {
    const cpx<double> p = a;            // i c n_a p
    a = mk(-c1 * p.y, c1 * p.x);
    b = mk(-c2 * p.y, c2 * p.x);
  } else {                              // -i (c1 a + c2 b)
    const double zx = c1 * a.x + c2 * b.x, zy = c1 * a.y + c2 * b.y;
    a = mk(zy, -zx);
  }
}

// Column transforms of length ny = 2^LOGN of the planes of X, mode
// multiplier, inverse column transforms, in place; SEQ columns per block.  The
// two planes' transforms run in step where four LDS tiles fit (up to 2048),
// else one after the other.
template <int LOGN, int OP>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_f_columns(cpx<double>* __restrict__ X, int nx, ModeMat c,
                                                              const cpx<double>* __restrict__ tw) {
  using S = Surf<LOGN>;
  constexpr int PIN = OP == N2T ? 1 : 2, POUT = OP == T2N ? 1 : 2;
  constexpr bool STEP = 4 * S::TILE * sizeof(cpx<double>) <= 150 * 1024;
  __shared__ cpx<double> buf[(STEP ? 4 : 2) * S::TILE];
  const int kxh = nx / 2 + 1;
  const int b = threadIdx.x / S::M, jj = threadIdx.x & (S::M - 1);
  const int kx = xcd_block() * S::SEQ + b;
  const bool on = kx < kxh;
  const size_t plane = (size_t)S::N * kxh;
  SurfTw<LOGN> t;
  cpx<double> v[2][4];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int m = 0; m < 4; ++m)
      v[q][m] = on && q < PIN ? X[q * plane + (size_t)(jj + m * S::M) * kxh + kx] : zero<double>();
  surf_load_tw<LOGN>(tw, jj, t);
  constexpr int LAST = surf_last<LOGN>(0);
  int first = 0;
  auto transform = [&](auto inv, int planes) {
    constexpr bool INV = decltype(inv)::value;
    if constexpr (STEP) {
      if (planes == 2) {
        surf_fft<LOGN, INV, 2>(v, buf, first, b, jj, t);
      } else {
        cpx<double>(&w)[1][4] = reinterpret_cast<cpx<double>(&)[1][4]>(v);
        surf_fft<LOGN, INV, 1>(w, buf, first, b, jj, t);
      }
      first = first ^ LAST ^ 1;
    } else {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (q >= planes) break;
        cpx<double>(&w)[1][4] = reinterpret_cast<cpx<double>(&)[1][4]>(v[q]);
        surf_fft<LOGN, INV, 1>(w, buf, first, b, jj, t);
        first = first ^ LAST ^ 1;
      }
    }
  };
  transform(std::integral_constant<bool, false>{}, PIN);
#pragma unroll
  for (int m = 0; m < 4; ++m) mode_apply<OP>(v[0][m], v[1][m], kx, jj + m * S::M, nx, S::N, c);
  transform(std::integral_constant<bool, true>{}, POUT);
  if (!on) return;
#pragma unroll
  for (int q = 0; q < POUT; ++q)
#pragma unroll
    for (int m = 0; m < 4; ++m) X[q * plane + (size_t)(jj + m * S::M) * kxh + kx] = v[q][m];
}

// sums of P(v + lam) and of its Jacobian
struct ProjSums {
  double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  __device__ __forceinline__ void point(double w0, double w1, double rho) {
    double p0, p1, ja, jb, jc;
    disk(w0, w1, rho, p0, p1, ja, jb, jc);
    s[0] += p0;
    s[1] += p1;
    s[2] += ja;
    s[3] += jb;
    s[4] += jc;
  }
};

// one Newton step on lam from those sums: g = sum P - S, J = sum of the
// Jacobians (regularised); the same in every thread
template <int NW>
__device__ __forceinline__ void newton(const double* __restrict__ part, int ldp, int nb, double S0, double S1,
                                       double* sh, double& l0, double& l1) {
  double t[5];
  surf_totals<5, NW>(nb, sh, t, [&](int i, double (&x)[5]) {
#pragma unroll
    for (int k = 0; k < 5; ++k) x[k] += part[k * ldp + i];
  });
  const double g0 = t[0] - S0, g1 = t[1] - S1;
  double a = t[2], b = t[3], c = t[4];
  const double reg = 1e-14 * (a + c + 1.0);
  a += reg;
  c += reg;
  const double det = a * c - b * b;
  if (det > 0.0) {
    l0 -= (c * g0 - b * g1) / det;
    l1 -= (a * g1 - b * g0) / det;
  }
}

// v = y - (u + ue) / L from u's row spectra; projection sums at F_LAMA
template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_f_grad(const cpx<double>* __restrict__ X,
                                                           const double* __restrict__ y,
                                                           const double* __restrict__ ue, double invL,
                                                           const double* __restrict__ rho, double* __restrict__ v,
                                                           int ny, const cpx<double>* __restrict__ tw, double* sc,
                                                           double* __restrict__ part, int ldp) {
  using S = Surf<LOGN>;
  __shared__ cpx<double> buf[2 * S::TILE];
  __shared__ double sh[5 * S::NW];
  const Row q = one_row<LOGN>(ny);
  const size_t n = (size_t)ny * S::N;
  SurfTw<LOGN> t;
  cpx<double> u[1][4], yv[4], uev[4];
  double r[4];
  if (!S::TIGHT) {
    load_row<LOGN>(y, n, q, yv);
    if (ue) load_row<LOGN>(ue, n, q, uev);
#pragma unroll
    for (int m = 0; m < 4; ++m) r[m] = q.on ? rho[q.off + q.jj + m * S::M] : 0.0;
  }
  surf_load_tw<LOGN>(tw, q.jj, t);
  const double l0 = sc[F_LAMA], l1 = sc[F_LAMA + 1];
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[F_T] = sc[F_TN];   // of the last k_f_momentum
  row_in<LOGN>(u, buf, q, ny, t, X);
  if (S::TIGHT) {
    load_row<LOGN>(y, n, q, yv);
    if (ue) load_row<LOGN>(ue, n, q, uev);
#pragma unroll
    for (int m = 0; m < 4; ++m) r[m] = q.on ? rho[q.off + q.jj + m * S::M] : 0.0;
  }
  ProjSums p;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (ue) u[0][m] = add(u[0][m], uev[m]);
    u[0][m] = axpy(yv[m], -invL, u[0][m]);
    if (q.on) p.point(u[0][m].x + l0, u[0][m].y + l1, r[m]);
  }
  store_row<LOGN>(v, n, q, u[0]);
  double o[5];
  surf_sums<5, S::NW>(p.s, sh, o);
  surf_put<5>(part, ldp, o);
}

// Newton step lam = sc[in] -> sc[out] from the sums pin of an earlier kernel
// (pin NULL: lam = sc[in]), projection sums at the new lam
__global__ __launch_bounds__(NT) void k_f_sums(const double* __restrict__ v, const double* __restrict__ rho, size_t n,
                                              double S0, double S1, double* sc, int in, int out,
                                              const double* __restrict__ pin, int nbin, double* __restrict__ part,
                                              int ldp) {
  __shared__ double sh[5 * NT / 64];
  double l0 = sc[in], l1 = sc[in + 1];
  if (pin) {
    newton<NT / 64>(pin, ldp, nbin, S0, S1, sh, l0, l1);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      sc[out] = l0;
      sc[out + 1] = l1;
    }
  }
  ProjSums p;
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT)
    p.point(v[i] + l0, v[n + i] + l1, rho[i]);
  double o[5];
  surf_sums<5, NT / 64>(p.s, sh, o);
  surf_put<5>(part, ldp, o);
}

// Newton step lam = F_LAMB -> F_LAMA, q_new = P(v + lam); sums of
// |q_new - q| and <y - q_new, q_new - q>
__global__ __launch_bounds__(NT) void k_f_apply(const double* __restrict__ v, const double* __restrict__ y,
                                               const double* __restrict__ rho, const double* __restrict__ q,
                                               double* __restrict__ qn, size_t n, double S0, double S1, double* sc,
                                               const double* __restrict__ pin, int nbin, double* __restrict__ part,
                                               int ldp) {
  __shared__ double sh[5 * NT / 64];
  double l0 = sc[F_LAMB], l1 = sc[F_LAMB + 1];
  newton<NT / 64>(pin, ldp, nbin, S0, S1, sh, l0, l1);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc[F_LAMA] = l0;
    sc[F_LAMA + 1] = l1;
  }
  double s[2] = {0.0, 0.0}, o[2];
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT) {
    const double y0 = y[i], y1 = y[n + i], q0 = q[i], q1 = q[n + i];
    double p0, p1, ja, jb, jc;
    disk(v[i] + l0, v[n + i] + l1, rho[i], p0, p1, ja, jb, jc);
    qn[i] = p0;
    qn[n + i] = p1;
    const double d0 = p0 - q0, d1 = p1 - q1;
    s[0] += fabs(d0) + fabs(d1);
    s[1] += (y0 - p0) * d0 + (y1 - p1) * d1;
  }
  surf_sums<2, NT / 64>(s, sh, o);
  surf_put<2>(part, ldp, o);
}

// restart or momentum from the sums of k_f_apply, the change measure to the
// host mirror; y = q_new + beta (q_new - q), q = q_new, row spectra of y
template <int LOGN>
__global__ __launch_bounds__(Surf<LOGN>::NTH) void k_f_momentum(double* __restrict__ q, const double* __restrict__ qn,
                                                               double* __restrict__ y, cpx<double>* __restrict__ X,
                                                               int ny, const cpx<double>* __restrict__ tw,
                                                               const double* __restrict__ part, int ldp, int nb,
                                                               double* sc, double* mirror, double cscale) {
  using S = Surf<LOGN>;
  __shared__ cpx<double> buf[2 * S::TILE];
  __shared__ double sh[2 * S::NW];
  const Row r = one_row<LOGN>(ny);
  const size_t n = (size_t)ny * S::N;
  SurfTw<LOGN> w;
  cpx<double> v[1][4], qv[4], nv[4];
  load_row<LOGN>(q, n, r, qv);
  load_row<LOGN>(qn, n, r, nv);
  if (!S::TIGHT) surf_load_tw<LOGN>(tw, r.jj, w);
  const double t = sc[F_T];
  double s[2];
  surf_totals<2, S::NW>(nb, sh, s, [&](int i, double (&x)[2]) {
    x[0] += part[i];
    x[1] += part[ldp + i];
  });
  double beta = 0.0, tn = 1.0;
  if (!(s[1] > 0.0)) {
    tn = 0.5 * (1.0 + sqrt(1.0 + 4.0 * t * t));
    beta = (t - 1.0) / tn;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc[F_TN] = tn;
    mirror[F_CHANGE] = s[0] * cscale;
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) v[0][m] = axpy(nv[m], beta, sub(nv[m], qv[m]));
  store_row<LOGN>(y, n, r, v[0]);
  store_row<LOGN>(q, n, r, nv);
  if (S::TIGHT) surf_load_tw<LOGN>(tw, r.jj, w);
  row_out<LOGN>(v, buf, r, ny, w, X);
}

// block sums of stick points (|q| < rho (1 - 1e-9)) and contact points (rho > 0)
__global__ __launch_bounds__(NT) void k_f_stick(const double* __restrict__ q, const double* __restrict__ rho,
                                               size_t n, double* part) {
  double v[2] = {0.0, 0.0};
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT) {
    const double r = rho[i];
    if (r > 0.0) {
      v[1] += 1.0;
      const double a = sqrt(q[i] * q[i] + q[n + i] * q[n + i]);
      if (a < r * (1.0 - 1e-9)) v[0] += 1.0;
    }
  }
  fblock_sums<2>(v, part);
}

// out = a - b
__global__ __launch_bounds__(NT) void k_c_sub(const double* __restrict__ a, const double* __restrict__ b,
                                             double* __restrict__ out, size_t n) {
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT) out[i] = a[i] - b[i];
}

// block sums of |p - p_prev| and |q - q_prev| (both components); t = (q0,
// q1, p) and tp its previous value, [3][n] each
__global__ __launch_bounds__(NT) void k_c_change(const double* __restrict__ t, const double* __restrict__ tp,
                                                size_t n, double* part) {
  double v[2] = {0.0, 0.0};
  for (size_t i = (size_t)blockIdx.x * NT + threadIdx.x; i < n; i += (size_t)gridDim.x * NT) {
    v[0] += fabs(t[2 * n + i] - tp[2 * n + i]);
    v[1] += fabs(t[i] - tp[i]) + fabs(t[n + i] - tp[n + i]);
  }
  fblock_sums<2>(v, part);
}

__global__ __launch_bounds__(NT) void k_f_totals(const double* __restrict__ part, int nb, int k, double* sc,
                                                double* mirror, int slot) {
  double s[3];
  for (int j = 0; j < k; ++j) s[j] = ffinal(part, j, nb);
  if (threadIdx.x == 0)
    for (int j = 0; j < k; ++j) sc[slot + j] = mirror[slot + j] = s[j];
}

// blocks of the row kernels and of the pointwise iteration kernels
int row_blocks(int nx, int ny) {
  const int m = nx / 4, nth = m < 64 ? 64 : m, seq = nth / m;
  return (ny + seq - 1) / seq;
}
int point_blocks(size_t n) { return (int)std::min<size_t>((n + 2 * NT - 1) / (2 * NT), PB); }
int iter_blocks(int nx, int ny) { return std::max(row_blocks(nx, ny), point_blocks((size_t)nx * ny)); }

int fblocks(size_t n) { return (int)std::min<size_t>((n + NT - 1) / NT, RB); }

}  // namespace

struct FricWork {
  size_t n = 0;
  double* vec = nullptr;          // q, y, u, q_new (2 planes each), rho; then for the
                                  // coupled solve: u_t[p] (2), h - u3[q] (1), previous
                                  // traction (3)
  cpx<double>* spec = nullptr;    // row spectra [2][ny][kxh]
  double* part = nullptr;         // [3][RB] of the sums outside the iteration
  double* ipart = nullptr;        // [12][ldp]: projection sums (two sets), apply sums
  int ldp = 0;
  double* sc = nullptr;           // device scalars
  double* hmap = nullptr;         // mapped host mirror (host view)
  double* dmap = nullptr;         //   (device view)
};

void friction_release(fvim_ctx* c) {
  FricWork* w = c->fric;
  if (!w) return;
  std::lock_guard<std::recursive_mutex> lk(device_lock());
  if (w->vec) hipFree(w->vec);
  if (w->spec) hipFree(w->spec);
  if (w->part) hipFree(w->part);
  if (w->ipart) hipFree(w->ipart);
  if (w->sc) hipFree(w->sc);
  if (w->hmap) hipHostFree(w->hmap);
  delete w;
  c->fric = nullptr;
}

static int fric_ensure(fvim_ctx* c) {
  if (c->fric) return FVIM_OK;
  std::lock_guard<std::recursive_mutex> lk(device_lock());
  FricWork* w = new FricWork();
  c->fric = w;
  const int nx = c->grid.nx, ny = c->grid.ny, kxh = nx / 2 + 1;
  w->n = (size_t)nx * ny;
  w->ldp = iter_blocks(nx, ny);
  const bool ok = hipMalloc((void**)&w->vec, sizeof(double) * 15 * w->n) == hipSuccess &&
                  hipMalloc((void**)&w->spec, sizeof(cpx<double>) * 2 * kxh * ny) == hipSuccess &&
                  hipMalloc((void**)&w->part, sizeof(double) * 3 * RB) == hipSuccess &&
                  hipMalloc((void**)&w->ipart, sizeof(double) * 12 * w->ldp) == hipSuccess &&
                  hipMalloc((void**)&w->sc, sizeof(double) * F_NSC) == hipSuccess &&
                  hipHostMalloc((void**)&w->hmap, sizeof(double) * F_NSC,
                                hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess &&
                  hipHostGetDevicePointer((void**)&w->dmap, w->hmap, 0) == hipSuccess;
  if (!ok) {
    friction_release(c);
    return fail(FVIM_ENOMEM, "tangential contact workspace allocation failed");
  }
  return FVIM_OK;
}

int friction_reserve(fvim_ctx* c) { return fric_ensure(c); }

size_t friction_footprint(const fvim_grid* g) {
  const size_t n = (size_t)g->nx * g->ny, nm = (size_t)(g->nx / 2 + 1) * g->ny;
  return sizeof(double) * (15 * n + 3 * RB + 12 * (size_t)iter_blocks(g->nx, g->ny) + F_NSC) +
         sizeof(cpx<double>) * 2 * nm;
}

static double shear_modulus(const fvim_ctx* c) { return c->mat.E / (2.0 * (1.0 + c->mat.nu)); }

template <int OP>
static hipError_t launch_f_columns(fvim_ctx* c, hipStream_t st) {
  const int nx = c->grid.nx, ny = c->grid.ny, kxh = nx / 2 + 1;
  const ModeMat m = {c->grid.lx, c->grid.ly, 1.0 / ((double)nx * ny), c->mat.nu, shear_modulus(c)};
#define CALL(L)                                                                                                  \
  hipLaunchKernelGGL((k_f_columns<L, OP>), dim3((unsigned)((kxh + Surf<L>::SEQ - 1) / Surf<L>::SEQ)),            \
                     dim3(Surf<L>::NTH), 0, st, c->fric->spec, nx, m, (const cpx<double>*)c->twy64)
  FVIM_SURF_SWITCH(surf_log2(ny), CALL)
#undef CALL
  return hipGetLastError();
}

static hipError_t launch_f_rows(fvim_ctx* c, const double* in, double* out, hipStream_t st) {
  const int nx = c->grid.nx, ny = c->grid.ny, nb = row_blocks(nx, ny);
  cpx<double>* X = c->fric->spec;
  const cpx<double>* tw = (const cpx<double>*)c->twx64;
#define CALL(L)                                                                                             \
  if (in) hipLaunchKernelGGL((k_f_rows_fwd<L>), dim3(nb), dim3(Surf<L>::NTH), 0, st, in, X, ny, tw);        \
  else hipLaunchKernelGGL((k_f_rows_inv<L>), dim3(nb), dim3(Surf<L>::NTH), 0, st, X, out, ny, tw)
  FVIM_SURF_SWITCH(surf_log2(nx), CALL)
#undef CALL
  return hipGetLastError();
}

// Cerruti cross displacements.  n2t: ut (2 planes) = u_t of the pressure in
// (1 plane); else u3 (1 plane) = u3 of the tangential traction in (2 planes).
static int cerruti_cross(fvim_ctx* c, const double* in, double* out, bool n2t, hipStream_t st) {
  const int nx = c->grid.nx, ny = c->grid.ny;
  cpx<double>* X = c->fric->spec;
  const cpx<double>* tw = (const cpx<double>*)c->twx64;
  hipError_t e = n2t ? launch_rows_fwd(nx, ny, in, X, tw, st) : launch_f_rows(c, in, nullptr, st);
  if (e == hipSuccess) e = n2t ? launch_f_columns<N2T>(c, st) : launch_f_columns<T2N>(c, st);
  if (e == hipSuccess) e = n2t ? launch_f_rows(c, nullptr, out, st) : launch_rows_inv(nx, ny, X, out, tw, st);
  return e == hipSuccess ? FVIM_OK : fail_hip(e, "cross displacements");
}

// One iteration from the row spectra of y; leaves those of the next y.
struct FricIter {
  double *q, *y, *v, *qn, *rho;
  const double* ue;
  double invL, S0, S1, cscale;
};
static hipError_t launch_f_iteration(fvim_ctx* c, const FricIter& f, hipStream_t st) {
  FricWork* w = c->fric;
  const int nx = c->grid.nx, ny = c->grid.ny, nbr = row_blocks(nx, ny), nbp = point_blocks(w->n), ldp = w->ldp;
  double* pa = w->ipart;
  double* pb = pa + 5 * (size_t)ldp;
  double* pc = pb + 5 * (size_t)ldp;
  const cpx<double>* tw = (const cpx<double>*)c->twx64;
  hipError_t e = launch_f_columns<COMPLIANCE>(c, st);
  if (e != hipSuccess) return e;
#define CALL(L)                                                                                                      \
  hipLaunchKernelGGL((k_f_grad<L>), dim3(nbr), dim3(Surf<L>::NTH), 0, st, w->spec, f.y, f.ue, f.invL, f.rho, f.v,    \
                     ny, tw, w->sc, pa, ldp)
  FVIM_SURF_SWITCH(surf_log2(nx), CALL)
#undef CALL
  hipLaunchKernelGGL(k_f_sums, dim3(nbp), dim3(NT), 0, st, f.v, f.rho, w->n, f.S0, f.S1, w->sc, (int)F_LAMA,
                     (int)F_LAMB, pa, nbr, pb, ldp);
  hipLaunchKernelGGL(k_f_apply, dim3(nbp), dim3(NT), 0, st, f.v, f.y, f.rho, f.q, f.qn, w->n, f.S0, f.S1, w->sc, pb,
                     nbp, pc, ldp);
#define CALL(L)                                                                                                      \
  hipLaunchKernelGGL((k_f_momentum<L>), dim3(nbr), dim3(Surf<L>::NTH), 0, st, f.q, f.qn, f.y, w->spec, ny, tw, pc,   \
                     ldp, nbp, w->sc, w->dmap, f.cscale)
  FVIM_SURF_SWITCH(surf_log2(nx), CALL)
#undef CALL
  return hipGetLastError();
}

int friction_solve(fvim_ctx* c, const double* p, double mu_f, double Qx, double Qy, double tol, int max_iter,
                   double* q_out, fvim_tangential_info* info, bool warm, const double* ue) {
  if (!(mu_f > 0.0) || !std::isfinite(Qx) || !std::isfinite(Qy) || !(tol > 0.0) || max_iter < 1)
    return fail(FVIM_EINVAL, "tangential_solve: bad arguments");
  int rc = fric_ensure(c);
  if (rc) return rc;
  FricWork* w = c->fric;
  hipStream_t st = c->stream;
  const size_t n = w->n;
  double* q = w->vec;
  double* y = q + 2 * n;
  double* v = y + 2 * n;
  double* qn = v + 2 * n;
  double* rho = qn + 2 * n;
  const int nb = fblocks(n);
  const double dA = c->grid.lx * c->grid.ly / (double)n;
  hipLaunchKernelGGL(k_f_rho, dim3(nb), dim3(NT), 0, st, p, mu_f, rho, n, w->part);
  hipLaunchKernelGGL(k_f_totals, dim3(1), dim3(NT), 0, st, w->part, nb, 1, w->sc, w->dmap, (int)F_SUMP);
  hipError_t e = hipStreamSynchronize(st);
  if (e != hipSuccess) return fail_hip(e, "tangential_solve");
  const double W = dA * w->hmap[F_SUMP];
  if (!(std::hypot(Qx, Qy) < mu_f * W))
    return fail(FVIM_EINVAL, "tangential_solve: partial slip needs |Q| < mu_f W (full sliding: q = mu_f p Q/|Q|)");
  // largest eigenvalue of C: the lowest wavenumber, along the direction
  // where I - nu n n^T is 1 (the coupling only lowers it)
  const double G = shear_modulus(c);
  const double twopi = 6.283185307179586476925286766559;
  double kmin = INFINITY;
  if (c->grid.nx > 1) kmin = std::min(kmin, twopi / c->grid.lx);
  if (c->grid.ny > 1) kmin = std::min(kmin, twopi / c->grid.ly);
  const double L = 1.0 / (G * kmin);
  const double invL = 1.0 / L;
  const double S0 = Qx / dA, S1 = Qy / dA;
  hipLaunchKernelGGL(k_f_init, dim3(nb), dim3(NT), 0, st, rho, q, y, n, Qx / (mu_f * W), Qy / (mu_f * W));
  double init[F_NSC] = {};
  init[F_T] = init[F_TN] = 1.0;
  {
    std::lock_guard<std::recursive_mutex> lk(device_lock());     // pageable copy
    e = hipMemcpyAsync(w->sc, init, sizeof(init), hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
  }
  if (e != hipSuccess) return fail_hip(e, "tangential_solve");
  const double cscale = dA / (mu_f * W);
  if (warm) {
    // start from the projection of the caller's q (the previous solution
    // under a nearby pressure) onto the new constraint set: Newton steps on
    // lam with v = q (step length 0), then q = y = P(q + lam)
    e = hipMemcpyAsync(y, q_out, sizeof(double) * 2 * n, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return fail_hip(e, "tangential_solve");
    const int nbp = point_blocks(n), ldp = w->ldp;
    double* part[2] = {w->ipart, w->ipart + 5 * (size_t)ldp};
    static_assert(WARM % 2 == 0 && F_LAMB == F_LAMA + 2, "the last Newton step starts from F_LAMB");
    for (int j = 0; j < WARM; ++j)
      hipLaunchKernelGGL(k_f_sums, dim3(nbp), dim3(NT), 0, st, y, rho, n, S0, S1, w->sc,
                         (int)(j == 0 || j % 2 ? F_LAMA : F_LAMB), (int)(j % 2 ? F_LAMB : F_LAMA),
                         (const double*)(j ? part[(j - 1) % 2] : nullptr), nbp, part[j % 2], ldp);
    hipLaunchKernelGGL(k_f_apply, dim3(nbp), dim3(NT), 0, st, y, y, rho, q, qn, n, S0, S1, w->sc, part[1], nbp,
                       part[0], ldp);
    e = hipMemcpyAsync(q, qn, sizeof(double) * 2 * n, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = hipMemcpyAsync(y, qn, sizeof(double) * 2 * n, hipMemcpyDeviceToDevice, st);
    if (e != hipSuccess) return fail_hip(e, "tangential_solve");
  }
  const FricIter it = {q, y, v, qn, rho, ue, invL, S0, S1, cscale};
  if ((e = launch_f_rows(c, y, nullptr, st)) != hipSuccess) return fail_hip(e, "tangential_solve");
  int k = 0;
  double change = INFINITY;
  bool conv = false;
  while (k < max_iter) {
    if ((e = launch_f_iteration(c, it, st)) != hipSuccess) return fail_hip(e, "tangential_solve");
    ++k;
    if (k % CHECK == 0 || k == max_iter) {
      if ((e = hipStreamSynchronize(st)) != hipSuccess) return fail_hip(e, "tangential_solve");
      change = w->hmap[F_CHANGE];
      if (!std::isfinite(change)) return fail(FVIM_EINVAL, "tangential_solve: iterate is not finite");
      if (change < tol) {
        conv = true;
        break;
      }
    }
  }
  // outputs: q, stick fraction, the rigid shift L lam of the stick zone
  e = hipMemcpyAsync(q_out, q, sizeof(double) * 2 * n, hipMemcpyDeviceToDevice, st);
  if (e != hipSuccess) return fail_hip(e, "tangential_solve");
  hipLaunchKernelGGL(k_f_stick, dim3(nb), dim3(NT), 0, st, q, rho, n, w->part);
  hipLaunchKernelGGL(k_f_totals, dim3(1), dim3(NT), 0, st, w->part, nb, 2, w->sc, w->dmap, (int)F_STICK);
  double lam[2];
  {
    std::lock_guard<std::recursive_mutex> lk(device_lock());     // pageable copy
    e = hipMemcpyAsync(lam, w->sc + F_LAMA, sizeof(lam), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
  }
  if (e != hipSuccess) return fail_hip(e, "tangential_solve");
  if (info) {
    info->iters = k;
    info->rel_change = change;
    info->stick_fraction = w->hmap[F_CONTACT] > 0 ? w->hmap[F_STICK] / w->hmap[F_CONTACT] : 0.0;
    info->shift[0] = L * lam[0];
    info->shift[1] = L * lam[1];
  }
  if (!conv) return fail(FVIM_ENOCONV, "tangential_solve: iteration limit reached");
  return FVIM_OK;
}

int frictional_solve(fvim_ctx* c, const double* h, double W, double mu_f, double Qx, double Qy, int coupled,
                     double tol, double tol_contact, double tol_f, int max_contact, int max_iter, double* T,
                     bool warm, fvim_frictional_info* info) {
  if (!(mu_f > 0.0) || !(W > 0.0) || !std::isfinite(W) || !std::isfinite(Qx) || !std::isfinite(Qy) ||
      !(tol > 0.0) || !(tol_contact > 0.0) || !(tol_f > 0.0) || max_iter < 1 || max_contact < 1 ||
      (coupled != 0 && coupled != 1))
    return fail(FVIM_EINVAL, "frictional_contact_solve: bad arguments");
  if (!(std::hypot(Qx, Qy) < mu_f * W))
    return fail(FVIM_EINVAL, "frictional_contact_solve: partial slip needs |Q| < mu_f W");
  int rc = fric_ensure(c);
  if (rc) return rc;
  FricWork* w = c->fric;
  hipStream_t st = c->stream;
  const size_t n = w->n;
  const int nb = fblocks(n);
  const double dA = c->grid.lx * c->grid.ly / (double)n;
  double* q = T;
  double* p = T + 2 * n;
  double* ue = w->vec + 9 * n;        // u_t of the pressure [2][n]
  double* he = ue + 2 * n;            // h - u3 of the tangential traction
  double* prev = he + n;              // traction of the previous alternation [3][n]
  hipError_t e;
  int k = 0, cit = 0, tit = 0;
  double change = INFINITY;
  bool conv = !coupled;
  fvim_contact_info ci{};
  fvim_tangential_info fi{};
  const int kmax = coupled ? max_iter : 1;
  for (k = 1; k <= kmax; ++k) {
    const bool haveq = coupled && (k > 1 || warm);      // q holds a traction to start from
    const bool track = coupled && (k > 1 || warm);
    const double* hk = h;
    if (haveq) {
      if ((rc = cerruti_cross(c, q, he, false, st))) return rc;
      hipLaunchKernelGGL(k_c_sub, dim3(nb), dim3(NT), 0, st, h, he, he, n);
      hk = he;
    }
    if (track && (e = hipMemcpyAsync(prev, T, sizeof(double) * 3 * n, hipMemcpyDeviceToDevice, st)) != hipSuccess)
      return fail_hip(e, "frictional_contact_solve");
    if ((rc = pk_solve(c, hk, W, tol_contact, max_contact, p, nullptr, &ci))) return rc;
    cit += ci.iters;
    if (coupled && (rc = cerruti_cross(c, p, ue, true, st))) return rc;
    rc = friction_solve(c, p, mu_f, Qx, Qy, tol_f, max_contact, q, &fi, coupled ? haveq : warm,
                        coupled ? ue : nullptr);
    if (rc) return rc;
    tit += fi.iters;
    if (track) {
      hipLaunchKernelGGL(k_c_change, dim3(nb), dim3(NT), 0, st, T, prev, n, w->part);
      hipLaunchKernelGGL(k_f_totals, dim3(1), dim3(NT), 0, st, w->part, nb, 2, w->sc, w->dmap, (int)F_CP);
      if ((e = hipStreamSynchronize(st)) != hipSuccess) return fail_hip(e, "frictional_contact_solve");
      change = dA * w->hmap[F_CP] / W + dA * w->hmap[F_CQ] / (mu_f * W);
      if (!std::isfinite(change)) return fail(FVIM_EINVAL, "frictional_contact_solve: iterate is not finite");
      if (change < tol) {
        conv = true;
        break;
      }
    }
  }
  if (k > kmax) k = kmax;
  if (info) {
    info->iters = k;
    info->contact_iters = cit;
    info->tangential_iters = tit;
    info->rel_change = change;
    info->kkt_residual = ci.kkt_residual;
    info->stick_fraction = fi.stick_fraction;
    info->shift[0] = fi.shift[0];
    info->shift[1] = fi.shift[1];
  }
  if (!conv) return fail(FVIM_ENOCONV, "frictional_contact_solve: alternation limit reached");
  return FVIM_OK;
}

int frictional_reserve(fvim_ctx* c) {
  int rc = fric_ensure(c);
  return rc ? rc : solver_reserve(c);
}

}  // namespace fvim

int frictional_contact_solve(fvim_ctx* ctx, const double* h, double W, double mu_f, double Qx, double Qy,
                             int coupled, double tol, int max_iter, int warm, double* traction,
                             fvim_frictional_info* info) {
  if (!ctx || !h || !traction) return fvim::fail(FVIM_EINVAL, "frictional_contact_solve: NULL argument");
  if (info) *info = fvim_frictional_info{};
  // the normal solves to a tenth of the alternation's tolerance (not below
  // 1e-15), the tangential solves to it
  const double tc = std::max(0.1 * tol, 1e-15);
  return fvim::frictional_solve(ctx, h, W, mu_f, Qx, Qy, coupled, tol, tc, tol, 100000, max_iter, traction,
                                warm != 0, info);
}

int tangential_solve(fvim_ctx* ctx, const double* p, double mu_f, double Qx, double Qy, double tol, int max_iter,
                     double* q, fvim_tangential_info* info) {
  if (!ctx || !p || !q) return fvim::fail(FVIM_EINVAL, "tangential_solve: NULL argument");
  return fvim::friction_solve(ctx, p, mu_f, Qx, Qy, tol, max_iter, q, info);
}
