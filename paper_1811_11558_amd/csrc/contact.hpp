// Launches of the normal contact iteration (contact.hip) for the solvers.
#pragma once
#include "common.hpp"

namespace fvim {

// device scalar slots of the solvers
enum {
  S_GBAR = 0, S_G, S_GOLD, S_DELTA, S_ERR, S_CNT, S_W, S_DA,
  S_DOT0, S_DOT1, S_DOT2, S_KKT, S_TAU0, S_GLO, S_IT, NSCAL = 32
};

// One contact problem on an nx x ny surface: device fields of nx ny doubles
// (h, p: the caller's; pold, g, t: workspace), the row spectrum X of
// ny (nx / 2 + 1) complex, block sums, scalars and their host mirror.
struct PkBufs {
  int nx, ny;
  double lx, ly, estar;
  const cpx<double>* twx;
  const cpx<double>* twy;
  const double* h;
  double *p, *pold, *g, *t;
  cpx<double>* X;
  double* part;           // pk_part_count(nx, ny) doubles
  double* sc;
  double* mirror;
};

// doubles of block sums an nx x ny problem needs
int pk_part_count(int nx, int ny);

// Row transforms of one surface plane to and from its row spectrum X[y][kx].
hipError_t launch_rows_fwd(int nx, int ny, const double* in, cpx<double>* X, const cpx<double>* twx, hipStream_t st);
hipError_t launch_rows_inv(int nx, int ny, const cpx<double>* X, double* out, const cpx<double>* twx, hipStream_t st);

// out = M[in] . e3 at z = 0 of one surface plane (2 / (E* |q|) per mode, mode
// 0 dropped); X as in PkBufs.
hipError_t launch_compliance(int nx, int ny, double lx, double ly, double estar, const cpx<double>* twx,
                             const cpx<double>* twy, const double* in, double* out, cpx<double>* X, hipStream_t st);

// g = M[p] - h and its sums on the contact set for the pressure p, before the
// first iteration.
hipError_t launch_pk_first(const PkBufs& b, hipStream_t st);

// One Polonsky-Keer iteration from the state launch_pk_first or the previous
// iteration left: p is the new pressure, g = M[p] - h.
hipError_t launch_pk_iteration(const PkBufs& b, hipStream_t st);

// Whether an nx x ny surface is iterated by one workgroup (launch_pk_solo).
bool pk_solo_fits(int nx, int ny);

// Up to `count` iterations in one launch, fewer when sum |p - p_old| falls below
// tol or is not finite.  first: from the start pressure (launch_pk_first's g,
// no direction), else from the state the previous launch left.  mirror[S_ERR],
// mirror[S_IT]: the last iteration's measure and how many ran; after the last
// one (converged, or `last` and count done) g is left minus its mean on the contact
// set, with sc[S_GBAR] and sc[S_CNT].
hipError_t launch_pk_solo(const PkBufs& b, int count, double tol, bool first, bool last, hipStream_t st);

// sc[S_ERR] (and its mirror) = dA sum |p - p_old| / W of the last iteration.
hipError_t launch_pk_err(const PkBufs& b, hipStream_t st);

// g minus its mean on the contact set (sc[S_GBAR], sc[S_CNT]), after the
// last iteration.
hipError_t launch_pk_gap_mean(const PkBufs& b, hipStream_t st);

}  // namespace fvim
