// Pointwise float64 kernels: the J2 radial return (Sec. 4.1) and the vector
// algebra of the iterative solvers.  All are HBM-streaming; each thread
// handles consecutive voxels of one component plane so every access is a
// contiguous run.
#include "common.hpp"
#include "kernels.hpp"

namespace fvim {
namespace {

constexpr int NT = 256;

// Backward-Euler radial return for linear isotropic hardening.  The plastic
// multiplier increment is exact for this law: with f = sigma_eq_trial -
// (sy0 + eh ep_n) > 0, the consistency condition
// sigma_eq_trial - 3 mu d_ep = sy0 + eh (ep_n + d_ep) gives
// d_ep = f / (3 mu + eh), and the flow direction is that of dev sigma_trial.
// The strain increment is de + cf F when F is given (a trial point of the
// plasticity iteration), and is then also stored in xt unless xt is NULL;
// d_ep and sigma_(n+1) are written only where dp and sn1 are given.
__global__ __launch_bounds__(NT) void k_return_map(const double* __restrict__ de, const double* __restrict__ F,
                                                  double cf, double* __restrict__ xt, const double* sn,
                                                  const double* __restrict__ epn, double* __restrict__ dep,
                                                  double* __restrict__ dp, double* sn1, size_t V, double lam,
                                                  double mu, double sy0, double eh, int* __restrict__ flags,
                                                  int lp, const int* __restrict__ zwrite) {
  size_t v = (size_t)blockIdx.x * NT + threadIdx.x;
  if (v >= V) return;
  double e[6], s[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    e[c] = de[c * V + v];
    s[c] = sn[c * V + v];
  }
  if (F) {
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      e[c] += cf * F[c * V + v];
      if (xt) xt[c * V + v] = e[c];
    }
  }
  const double tre = e[0] + e[1] + e[2];
#pragma unroll
  for (int c = 0; c < 6; ++c) s[c] += 2.0 * mu * e[c] + (c < 3 ? lam * tre : 0.0);
  const double m = (s[0] + s[1] + s[2]) * (1.0 / 3.0);
  double d[6] = {s[0] - m, s[1] - m, s[2] - m, s[3], s[4], s[5]};
  const double nn = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + 2.0 * (d[3] * d[3] + d[4] * d[4] + d[5] * d[5]);
  const double seq = sqrt(1.5 * nn);
  const double f = seq - (sy0 + eh * epn[v]);
  double dpv = 0.0, fac = 0.0;
  if (f > 0.0) {
    dpv = f / (3.0 * mu + eh);
    fac = 1.5 * dpv / seq;
  }
  if (dp) dp[v] = dpv;
  if (flags && fac != 0.0) flags[v >> lp] = 1;   // d_eps_p = fac dev(sigma_trial) is not zero
  // with zwrite, dep already holds zeros in the layers >= *zwrite: an elastic
  // voxel there needs no store
  if (zwrite && fac == 0.0 && (int)(v >> lp) >= *zwrite) return;
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const double x = fac * d[c];
    dep[c * V + v] = x;
    if (sn1) sn1[c * V + v] = s[c] - 2.0 * mu * x;
  }
}

// Consistent tangent T of the radial return above at the strain increment
// de: out = base - T (u1 - u2) (base, u2 may be NULL), for the voxels
// v < na of each component (component stride V).  With d = dev
// sigma_trial, seq = sqrt(3/2)|d|, d_ep = f / (3 mu + eh) and
// d_eps_p = (3 d_ep / (2 seq)) d, a change u of de changes d by
// dd = 2 mu dev(u), seq by (3/2) <d, dd> / seq and d_ep by that over
// (3 mu + eh); the product rule gives the rest.  The trial state is formed
// with the same operations as the return map, so T is nonzero exactly on
// the voxels the return map at de lets flow.
__global__ __launch_bounds__(NT) void k_plastic_tangent(const double* __restrict__ de, const double* u1,
                                                       const double* u2, const double* base,
                                                       const double* __restrict__ sn, const double* __restrict__ epn,
                                                       double* out, size_t na, size_t V, double lam, double mu,
                                                       double sy0, double eh) {
  size_t v = (size_t)blockIdx.x * NT + threadIdx.x;
  if (v >= na) return;
  double e[6], s[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    e[c] = de[c * V + v];
    s[c] = sn[c * V + v];
  }
  const double tre = e[0] + e[1] + e[2];
#pragma unroll
  for (int c = 0; c < 6; ++c) s[c] += 2.0 * mu * e[c] + (c < 3 ? lam * tre : 0.0);
  const double m = (s[0] + s[1] + s[2]) * (1.0 / 3.0);
  const double d[6] = {s[0] - m, s[1] - m, s[2] - m, s[3], s[4], s[5]};
  const double nn = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + 2.0 * (d[3] * d[3] + d[4] * d[4] + d[5] * d[5]);
  const double seq = sqrt(1.5 * nn);
  const double f = seq - (sy0 + eh * epn[v]);
  double b[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) b[c] = base ? base[c * V + v] : 0.0;
  if (!(f > 0.0)) {
#pragma unroll
    for (int c = 0; c < 6; ++c) out[c * V + v] = b[c];
    return;
  }
  double dd[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) dd[c] = u1[c * V + v] - (u2 ? u2[c * V + v] : 0.0);
  const double um = (dd[0] + dd[1] + dd[2]) * (1.0 / 3.0);
#pragma unroll
  for (int c = 0; c < 6; ++c) dd[c] = 2.0 * mu * (c < 3 ? dd[c] - um : dd[c]);
  const double dn = d[0] * dd[0] + d[1] * dd[1] + d[2] * dd[2] + 2.0 * (d[3] * dd[3] + d[4] * dd[4] + d[5] * dd[5]);
  const double dseq = 1.5 * dn / seq;
  const double h = 1.0 / (3.0 * mu + eh);
  const double dp = f * h, ddp = dseq * h;
  const double fac = 1.5 * dp / seq;
  const double dfac = 1.5 * (ddp * seq - dp * dseq) / (seq * seq);
#pragma unroll
  for (int c = 0; c < 6; ++c) out[c * V + v] = b[c] - (dfac * d[c] + fac * dd[c]);
}

// Mean-mode fields in float64 (precision FP32_REFINED).  G threads per depth
// node: sum the partials of the 6 eigenstrain planes of that node (and of the 3
// traction planes; nsum each) in a fixed order, form the laterally
// uniform response (sigma . e3 = -t_mean, eps13 = (w13 - t1)/(2 mu),
// eps23 = (w23 - t2)/(2 mu), eps33 = (w33 - t3)/(lambda + 2 mu), other
// strains 0, displacement 0) and write one constant per output plane.  Bound by
// the latency of the partials' loads: a thread per node, which reads them one after
// the other, takes 14.6 us with 64 partials (64 x 1024 x 64), 64 threads 6.1.
template <int G>
__device__ __forceinline__ void k0_fields(const double* __restrict__ wsum, const double* __restrict__ tsum, int nsum,
                                          double* __restrict__ out, const DepthParams& p, int z, int l) {
  const int nz = p.nz;
  if (z >= nz) return;
  const double inv = p.norm;                      // 1 / (nx ny)
  const double mu = p.mu, lam = p.kappa * p.mu;
  const bool with_t = p.has_t && p.k0_include;
  double e[6] = {0, 0, 0, 0, 0, 0};
  double w[6] = {0, 0, 0, 0, 0, 0};
  double v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int k = l; k < nsum; k += G) {
    if (p.has_w) {
#pragma unroll
      for (int c = 0; c < 6; ++c) v[c] += wsum[((size_t)c * nz + z) * nsum + k];
    }
    if (with_t) {
#pragma unroll
      for (int c = 0; c < 3; ++c) v[6 + c] += tsum[(size_t)c * nsum + k];
    }
  }
#pragma unroll
  for (int o = (G < 64 ? G : 64) / 2; o > 0; o >>= 1) {
#pragma unroll
    for (int c = 0; c < 9; ++c) v[c] += __shfl_xor(v[c], o, 64);
  }
  if constexpr (G > 64) {
    __shared__ double sh[9][NT / 64];
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int c = 0; c < 9; ++c) sh[c][threadIdx.x >> 6] = v[c];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 9; ++c) v[c] = (sh[c][0] + sh[c][1]) + (sh[c][2] + sh[c][3]);
  }
  if (l != 0) return;
  if (p.has_w) {
    double ep[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) ep[c] = v[c] * inv;
    const double tr = ep[0] + ep[1] + ep[2];
#pragma unroll
    for (int c = 0; c < 6; ++c) w[c] = 2.0 * mu * ep[c] + (c < 3 ? lam * tr : 0.0);
  }
  const double t[3] = {v[6] * inv, v[7] * inv, v[8] * inv};
  e[4] = (w[4] - t[0]) / (2.0 * mu);
  e[3] = (w[3] - t[1]) / (2.0 * mu);
  e[2] = (w[2] - t[2]) / (lam + 2.0 * mu);
  if (p.off_strain >= 0)
    for (int c = 0; c < 6; ++c) out[p.off_strain + c * nz + z] = e[c];
  if (p.off_stress >= 0) {
    const double tre = e[0] + e[1] + e[2];
    for (int c = 0; c < 6; ++c) out[p.off_stress + c * nz + z] = 2.0 * mu * e[c] + (c < 3 ? lam * tre : 0.0) - w[c];
  }
  if (p.off_disp >= 0)
    for (int c = 0; c < 3; ++c) out[p.off_disp + c * nz + z] = 0.0;
  if (p.off_u3 >= 0 && z == 0) out[p.off_u3] = 0.0;
}

template <int G>
__global__ __launch_bounds__(NT) void k_k0_fields(const double* __restrict__ wsum, const double* __restrict__ tsum,
                                                 int nsum, double* __restrict__ out, DepthParams p) {
  k0_fields<G>(wsum, tsum, nsum, out, p, (blockIdx.x * NT + threadIdx.x) / G, threadIdx.x % G);
}
// The grids of a batched depth pass, a block per node.  (The lanes' sums are
// combined in pairs, so with G at least nsum the result does not depend on G: these
// are the bits of the single launch.)
__global__ __launch_bounds__(NT) void k_k0_batch(const DepthBatch* __restrict__ b, K0Batch k) {
  const int c = blockIdx.y;
  k0_fields<NT>(k.wsum[c], k.tsum[c], k.nsum[c], k.out[c], b->prm[c], blockIdx.x, threadIdx.x);
}

}  // namespace

hipError_t launch_k0_fields(const double* wsum, const double* tsum, int nsum, double* out, const DepthParams& p,
                            hipStream_t st) {
#define CALL(G)                                                                                                    \
  hipLaunchKernelGGL(k_k0_fields<G>, dim3((unsigned)(((size_t)p.nz * G + NT - 1) / NT)), dim3(NT), 0, st, wsum, tsum, \
                     nsum, out, p)
  if (nsum <= 1) CALL(1);
  else if (nsum <= 4) CALL(4);
  else if (nsum <= 16) CALL(16);
  else if (nsum <= 64) CALL(64);
  else CALL(256);
#undef CALL
  return hipGetLastError();
}
hipError_t launch_k0_batch(const DepthBatch& host, const DepthBatch* dtab, const K0Batch& k, hipStream_t st) {
  int nz = 0;
  for (int c = 0; c < host.n; ++c) nz = nz > host.prm[c].nz ? nz : host.prm[c].nz;
  hipLaunchKernelGGL(k_k0_batch, dim3((unsigned)nz, (unsigned)host.n), dim3(NT), 0, st, dtab, k);
  return hipGetLastError();
}

hipError_t launch_return_map(const double* d_eps, const double* sig_n, const double* ep_n, double* d_eps_p,
                             double* d_ep, double* sig_np1, size_t nvox, double lam, double mu, double sy0,
                             double eh, hipStream_t st) {
  unsigned nb = (unsigned)((nvox + NT - 1) / NT);
  hipLaunchKernelGGL(k_return_map, dim3(nb), dim3(NT), 0, st, d_eps, nullptr, 0.0, nullptr, sig_n, ep_n, d_eps_p,
                     d_ep, sig_np1, nvox, lam, mu, sy0, eh, nullptr, 0, nullptr);
  return hipGetLastError();
}

hipError_t launch_trial_return_map(const double* x, const double* F, double cf, double* xt, const double* sig_n,
                                   const double* ep_n, double* d_eps_p, size_t nvox, double lam, double mu,
                                   double sy0, double eh, hipStream_t st, int* layer_flags, int lp,
                                   const int* zwrite) {
  unsigned nb = (unsigned)((nvox + NT - 1) / NT);
  hipLaunchKernelGGL(k_return_map, dim3(nb), dim3(NT), 0, st, x, F, cf, xt, sig_n, ep_n, d_eps_p, nullptr,
                     nullptr, nvox, lam, mu, sy0, eh, layer_flags, lp, zwrite);
  return hipGetLastError();
}

hipError_t launch_plastic_tangent(const double* d_eps, const double* u1, const double* u2, const double* base,
                                  const double* sig_n, const double* ep_n, double* out, size_t na, size_t nvox,
                                  double lam, double mu, double sy0, double eh, hipStream_t st) {
  if (na == 0) return hipSuccess;
  unsigned nb = (unsigned)((na + NT - 1) / NT);
  hipLaunchKernelGGL(k_plastic_tangent, dim3(nb), dim3(NT), 0, st, d_eps, u1, u2, base, sig_n, ep_n, out, na, nvox,
                     lam, mu, sy0, eh);
  return hipGetLastError();
}

}  // namespace fvim
