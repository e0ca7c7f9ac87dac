// In-plane transforms of the layered fields (the DFT of Sec. 3.1, eqn dft),
// written for gfx950: every kernel holds a batch of 1D transforms in registers
// and runs a self-sorting (Stockham) FFT of radix 4 (one radix-2 stage when
// log2(n) is odd) or radix 8 (one radix-2 or radix-4 stage first), exchanging
// through LDS between passes of several stages.
// Global memory is touched once on the way in and once on the way out, with
// the layouts chosen so both sides are contiguous runs:
//
//   real field        [P][ny][nx]          (P planes = components x layers)
//   x-spectrum   X    [P][nx/2+1][ny]      written by x_r2c, read by y_fwd
//   mode-major   S    [nx/2+1][ny][P]      written by y_fwd, read by the
//                                          depth pass (all planes of one
//                                          mode are contiguous)
//
// and the mirror images for the inverse.  Real transforms of length nx are
// done two rows at a time as one complex transform (z = a + i b).
// Forward transforms are unnormalised; the depth pass applies 1/(nx ny).
//
// The tile (runs of half, default or twice the default length on the strided
// side) and the radix are choices of each launch (FftChoice), timed by the context's tuner for
// lengths 2^5 .. 2^10; other lengths use the default.  Kernels over several
// grids (XformBatch) have blocks of NT threads: rows in a tile of that size, columns
// in the default tile or half of it, radix 4.
#include <algorithm>

#include "common.hpp"
#include "fft_dev.hpp"
#include "kernels.hpp"

namespace fvim {

namespace {
// ---------------------------------------------------- single-grid kernels
template <typename T, int LOGN, bool NTL, int TILE, int RADIX>
__global__ __launch_bounds__((row_threads<T>(1 << LOGN, TILE)))
void k_x_r2c(InSegments seg, cpx<T>* __restrict__ out, int ny, int R, const cpx<T>* __restrict__ tw,
             double* __restrict__ bsum, LayerSkip skip) {
  __shared__ __align__(16) char tile[row_lds_bytes<T>(1 << LOGN, TILE)];
  x_r2c_body<T, LOGN, NTL, TILE, RADIX>(tile, blockIdx.x, seg, out, ny, R, tw, bsum, skip);
}

template <typename T, int LOGN, bool NTL, int TILE, int RADIX>
__global__ __launch_bounds__((col_threads<T>(1 << LOGN, TILE)))
void k_y_fwd(const cpx<T>* __restrict__ in, cpx<T>* __restrict__ out, int kxh, int NP, int ldp,
             const cpx<T>* __restrict__ tw, LayerSkip skip) {
  __shared__ __align__(16) char tile[col_lds_bytes<T>(1 << LOGN, TILE)];
  y_fwd_body<T, LOGN, NTL, TILE, RADIX>(tile, threadIdx.x, xcd_block(), true, in, out, kxh, NP, ldp, tw, skip);
}

template <typename T, int LOGN, bool NTL, int TILE, int RADIX>
__global__ __launch_bounds__((col_threads<T>(1 << LOGN, TILE)))
void k_y_inv(const cpx<T>* __restrict__ in, cpx<T>* __restrict__ out, int kxh, int NP, int ldp,
             const cpx<T>* __restrict__ tw) {
  __shared__ __align__(16) char tile[col_lds_bytes<T>(1 << LOGN, TILE)];
  y_inv_body<T, LOGN, NTL, TILE, RADIX>(tile, threadIdx.x, xcd_block(), true, in, out, kxh, NP, ldp, tw);
}

template <typename T, int LOGN, int TILE, int RADIX>
__global__ __launch_bounds__((row_threads<T>(1 << LOGN, TILE)))
void k_x_c2r(const cpx<T>* __restrict__ in, OutSegments seg, int ny, int R, double scale,
             const cpx<T>* __restrict__ tw, const double* __restrict__ padd, ResidEpilogue ep, int nts) {
  __shared__ __align__(16) char tile[row_lds_bytes<T>(1 << LOGN, TILE)];
  __shared__ double red[row_threads<T>(1 << LOGN, TILE) / 64];
  // the last planes first: the inverse column transform wrote them last
  x_c2r_body<T, LOGN, TILE, RADIX>(tile, red, (int)(gridDim.x - 1 - blockIdx.x), in, seg, ny, R, scale, tw, padd,
                                   ep, nts != 0);
}

template <typename T>
__global__ __launch_bounds__(NT) void k_x_r2c_batch(XformBatch b) {
  x_r2c_batch_block<T>(b, (int)blockIdx.x);
}

template <typename T>
__global__ __launch_bounds__(NT) void k_y_fwd_batch(XformBatch b) {
  y_fwd_batch_block<T>(b, xcd_block());
}

template <typename T>
__global__ __launch_bounds__(NT) void k_y_inv_batch(XformBatch b) {
  y_inv_batch_block<T>(b, xcd_block());
}

template <typename T>
__global__ __launch_bounds__(NT) void k_x_c2r_batch(XformBatch b) {
  __shared__ double red[NT / 64];
  x_c2r_batch_block<T>(b, (int)blockIdx.x, red);
}

// -------------------------------------------------------------- launches
// R of a row kernel launch: 2 SEQ rows, or the whole plane when it is shorter
int rows_per_block(int seq, int ny) { return 2 * seq < ny ? 2 * seq : ny; }

int ilog2(int n) { return 31 - __builtin_clz((unsigned)n); }

bool fft_tunable(int logn) { return logn >= FFT_TUNE_MIN_LOGN && logn <= FFT_TUNE_MAX_LOGN; }

#define FVIM_LOGN_SWITCH(logn, CALL) \
  switch (logn) {                    \
    case 2: CALL(2); break;          \
    case 3: CALL(3); break;          \
    case 4: CALL(4); break;          \
    case 5: CALL(5); break;          \
    case 6: CALL(6); break;          \
    case 7: CALL(7); break;          \
    case 8: CALL(8); break;          \
    case 9: CALL(9); break;          \
    case 10: CALL(10); break;        \
    case 11: CALL(11); break;        \
    case 12: CALL(12); break;        \
    default: return hipErrorInvalidValue; \
  }

// Calls GO<TILE, RADIX>() of the launcher struct for the effective choice:
// the six (tile, radix) variants exist for tunable lengths only.
template <int L, typename F>
hipError_t with_choice(FftChoice ch, F& f) {
  if constexpr (L >= FFT_TUNE_MIN_LOGN && L <= FFT_TUNE_MAX_LOGN) {
    if (ch.radix == 8) {
      if (ch.tile == 0) return f.template go<L, 0, 8>();
      if (ch.tile == 2) return f.template go<L, 2, 8>();
      return f.template go<L, 1, 8>();
    }
    if (ch.tile == 0) return f.template go<L, 0, 4>();
    if (ch.tile == 2) return f.template go<L, 2, 4>();
  }
  return f.template go<L, 1, 4>();
}

// Planes of at most SEQ rows fill half a default row block or less: the half-sized
// block then, which still holds the whole plane (the same sums, bit for bit; float32
// x_fwd / x_inv 14.6 / 13.2 -> 11.3 / 11.0 us at 512 x 4 x 100).
template <typename T>
constexpr bool row_halves(int n, int tile) { return tile == 1 && row_seq<T>(n, 0) < row_seq<T>(n, 1); }

template <typename T>
struct R2CLaunch {
  const InSegments& seg;
  cpx<T>* out;
  int ny;
  size_t nplanes;
  const cpx<T>* tw;
  hipStream_t st;
  double* bsum;
  bool stream_in;
  const LayerSkip& skip;
  template <int L, int TILE, int RADIX>
  hipError_t go() {
    if constexpr (row_halves<T>(1 << L, TILE))
      if (ny <= row_seq<T>(1 << L, TILE)) return go<L, 0, RADIX>();
    const int R = rows_per_block(row_seq<T>(1 << L, TILE), ny);
    const dim3 grid((unsigned)(nplanes * (size_t)ny / R)), blk(row_threads<T>(1 << L, TILE));
    if (stream_in)
      hipLaunchKernelGGL((k_x_r2c<T, L, true, TILE, RADIX>), grid, blk, 0, st, seg, out, ny, R, tw, bsum, skip);
    else
      hipLaunchKernelGGL((k_x_r2c<T, L, false, TILE, RADIX>), grid, blk, 0, st, seg, out, ny, R, tw, bsum, skip);
    return hipGetLastError();
  }
};

template <typename T, bool FWD>
struct ColLaunch {
  const cpx<T>* in;
  cpx<T>* out;
  int kxh, NP, ldp;
  const cpx<T>* tw;
  hipStream_t st;
  bool stream_in;
  const LayerSkip& skip;
  template <int L, int TILE, int RADIX>
  hipError_t go() {
    constexpr int B = col_batch<T>(1 << L, TILE);
    if constexpr (TILE == 1 && col_batch<T>(1 << L, THIN) < B)
      if (NP <= 4) return go<L, THIN, RADIX>();
    const dim3 grid((unsigned)(kxh * ((NP + B - 1) / B))), blk(col_threads<T>(1 << L, TILE));
    if (FWD) {
      if (stream_in)
        hipLaunchKernelGGL((k_y_fwd<T, L, true, TILE, RADIX>), grid, blk, 0, st, in, out, kxh, NP, ldp, tw, skip);
      else
        hipLaunchKernelGGL((k_y_fwd<T, L, false, TILE, RADIX>), grid, blk, 0, st, in, out, kxh, NP, ldp, tw,
                           skip);
    } else {
      if (stream_in)
        hipLaunchKernelGGL((k_y_inv<T, L, true, TILE, RADIX>), grid, blk, 0, st, in, out, kxh, NP, ldp, tw);
      else
        hipLaunchKernelGGL((k_y_inv<T, L, false, TILE, RADIX>), grid, blk, 0, st, in, out, kxh, NP, ldp, tw);
    }
    return hipGetLastError();
  }
};

template <typename T>
struct C2RLaunch {
  const cpx<T>* in;
  const OutSegments& seg;
  int ny;
  size_t nplanes;
  double scale;
  const cpx<T>* tw;
  hipStream_t st;
  const double* padd;
  const ResidEpilogue& ep;
  bool stream_out;
  template <int L, int TILE, int RADIX>
  hipError_t go() {
    if constexpr (row_halves<T>(1 << L, TILE))
      if (ny <= row_seq<T>(1 << L, TILE)) return go<L, 0, RADIX>();
    const int R = rows_per_block(row_seq<T>(1 << L, TILE), ny);
    const dim3 grid((unsigned)(nplanes * (size_t)ny / R)), blk(row_threads<T>(1 << L, TILE));
    hipLaunchKernelGGL((k_x_c2r<T, L, TILE, RADIX>), grid, blk, 0, st, in, seg, ny, R, scale, tw, padd, ep,
                       stream_out ? 1 : 0);
    return hipGetLastError();
  }
};

}  // namespace

FftChoice fft_effective(int logn, FftChoice ch) {
  if (!fft_tunable(logn) || (ch.radix != 4 && ch.radix != 8) || ch.tile < 0 || ch.tile > 2) return FftChoice{};
  return ch;
}

int x_r2c_sums_per_plane(int nx, int ny) { return row_sums(nx, ny); }

template <typename T>
hipError_t launch_x_r2c(const InSegments& seg, cpx<T>* out, int nx, int ny, size_t nplanes, const cpx<T>* tw,
                        hipStream_t st, double* bsum, bool stream_in, const LayerSkip& skip, FftChoice ch) {
  if (seg.n < 1 || seg.n > 2 || seg.first[0] != 0) return hipErrorInvalidValue;
  R2CLaunch<T> f{seg, out, ny, nplanes, tw, st, bsum, stream_in, skip};
  ch = fft_effective(ilog2(nx), ch);
#define CALL(L) return with_choice<L>(ch, f)
  FVIM_LOGN_SWITCH(ilog2(nx), CALL)
#undef CALL
}

template <typename T>
hipError_t launch_y_fwd(const cpx<T>* in, cpx<T>* out, int ny, int kxh, int NP, int ldp, const cpx<T>* tw,
                        hipStream_t st, bool stream_in, const LayerSkip& skip, FftChoice ch) {
  if (ldp < NP) return hipErrorInvalidValue;
  ColLaunch<T, true> f{in, out, kxh, NP, ldp, tw, st, stream_in, skip};
  ch = fft_effective(ilog2(ny), ch);
#define CALL(L) return with_choice<L>(ch, f)
  FVIM_LOGN_SWITCH(ilog2(ny), CALL)
#undef CALL
}

template <typename T>
hipError_t launch_y_inv(const cpx<T>* in, cpx<T>* out, int ny, int kxh, int NP, int ldp, const cpx<T>* tw,
                        hipStream_t st, bool stream_in, FftChoice ch) {
  if (ldp < NP) return hipErrorInvalidValue;
  const LayerSkip none{};
  ColLaunch<T, false> f{in, out, kxh, NP, ldp, tw, st, stream_in, none};
  ch = fft_effective(ilog2(ny), ch);
#define CALL(L) return with_choice<L>(ch, f)
  FVIM_LOGN_SWITCH(ilog2(ny), CALL)
#undef CALL
}

template <typename T>
hipError_t launch_x_c2r(const cpx<T>* in, const OutSegments& seg, int nx, int ny, size_t nplanes,
                        double scale, const cpx<T>* tw, hipStream_t st, const double* padd,
                        const ResidEpilogue& ep, bool stream_out, FftChoice ch) {
  // the epilogue reads its fields at the output's own offsets: one segment
  // holding the 6 nz strain planes from plane 0
  if (ep.x && (seg.n != 1 || seg.first[0] != 0 || !ep.part || ep.nz < 1 || nplanes != (size_t)6 * ep.nz))
    return hipErrorInvalidValue;
  C2RLaunch<T> f{in, seg, ny, nplanes, scale, tw, st, padd, ep, stream_out};
  ch = fft_effective(ilog2(nx), ch);
#define CALL(L) return with_choice<L>(ch, f)
  FVIM_LOGN_SWITCH(ilog2(nx), CALL)
#undef CALL
}

template <typename T>
int x_c2r_blocks(int nx, int ny, size_t nplanes, FftChoice ch) {
  return (int)(nplanes * (size_t)ny / rows_per_block(row_seq<T>(nx, fft_effective(ilog2(nx), ch).tile), ny));
}

template <typename T>
int x_c2r_max_blocks(int nx, int ny, size_t nplanes) {
  int m = 0;
  for (int t = 0; t < 3; ++t) m = std::max(m, x_c2r_blocks<T>(nx, ny, nplanes, FftChoice{t, 4}));
  return m;
}

// ------------------------------------------------- launches over grids
namespace {

// block count and LDS bytes of one grid's part of a batched launch, and its rows
// per block (row kernels)
template <typename T>
struct BatchGeom {
  int blocks = 0, R = 0;
  size_t lds = 0;
};

template <typename T>
BatchGeom<T> geom_row(int logn, int ny, int nplanes) {
  BatchGeom<T> g;
  const int n = 1 << logn;
  g.R = rows_per_block(row_seq<T>(n, 3), ny);
  g.blocks = nplanes * ny / g.R;
  g.lds = (size_t)row_lds_bytes<T>(n, 3);
  return g;
}
template <typename T>
BatchGeom<T> geom_col(int logn, int kxh, int NP) {
  BatchGeom<T> g;
  const int n = 1 << logn;
  const int tile = col_shared_tile<T>(n);
  const int B = col_batch<T>(n, tile), G = NT / col_threads<T>(n, tile);
  g.blocks = (kxh * ((NP + B - 1) / B) + G - 1) / G;
  g.lds = (size_t)G * col_lds_bytes<T>(n, tile);
  return g;
}

}  // namespace

// kind: 0 x_r2c, 1 y_fwd, 2 y_inv, 3 x_c2r.  The host fills every grid's
// fields but first[]; logn is the transform length of the kernel (nx for
// the row kernels, ny for the column kernels), nplanes[c] its plane count.
template <typename T>
size_t xform_batch_prepare(int kind, XformBatch& b) {
  if (b.n < 1 || b.n > XFORM_BATCH_MAX || kind < 0 || kind > 3) return 0;
  size_t lds = 0;
  b.first[0] = 0;
  for (int c = 0; c < b.n; ++c) {
    if (b.logn[c] < 2 || b.logn[c] > XFORM_BATCH_MAX_LOGN) return 0;
    BatchGeom<T> g = kind == 0 || kind == 3 ? geom_row<T>(b.logn[c], b.ny[c], b.NP[c])
                                            : geom_col<T>(b.logn[c], b.kxh[c], b.NP[c]);
    b.R[c] = g.R;
    b.first[c + 1] = b.first[c] + g.blocks;
    lds = std::max(lds, g.lds);
  }
  return lds;
}

template <typename T>
hipError_t launch_xform_batch(int kind, XformBatch& b, hipStream_t st) {
  if (b.n < 1 || b.n > XFORM_BATCH_MAX) return hipErrorInvalidValue;
  size_t lds = 0;
  b.first[0] = 0;
  for (int c = 0; c < b.n; ++c) {
    if (b.logn[c] < 2 || b.logn[c] > XFORM_BATCH_MAX_LOGN) return hipErrorInvalidValue;
    BatchGeom<T> g = kind == 0 || kind == 3 ? geom_row<T>(b.logn[c], b.ny[c], b.NP[c])
                                            : geom_col<T>(b.logn[c], b.kxh[c], b.NP[c]);
    b.R[c] = g.R;
    b.first[c + 1] = b.first[c] + g.blocks;
    lds = std::max(lds, g.lds);
  }
  const dim3 grid((unsigned)b.first[b.n]);
  switch (kind) {
    case 0: hipLaunchKernelGGL(k_x_r2c_batch<T>, grid, dim3(NT), lds, st, b); break;
    case 1: hipLaunchKernelGGL(k_y_fwd_batch<T>, grid, dim3(NT), lds, st, b); break;
    case 2: hipLaunchKernelGGL(k_y_inv_batch<T>, grid, dim3(NT), lds, st, b); break;
    case 3: hipLaunchKernelGGL(k_x_c2r_batch<T>, grid, dim3(NT), lds, st, b); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

#define FVIM_INST(T)                                                                                            \
  template hipError_t launch_x_r2c<T>(const InSegments&, cpx<T>*, int, int, size_t, const cpx<T>*, hipStream_t, \
                                      double*, bool, const LayerSkip&, FftChoice);                              \
  template hipError_t launch_y_fwd<T>(const cpx<T>*, cpx<T>*, int, int, int, int, const cpx<T>*, hipStream_t,   \
                                      bool, const LayerSkip&, FftChoice);                                       \
  template hipError_t launch_y_inv<T>(const cpx<T>*, cpx<T>*, int, int, int, int, const cpx<T>*, hipStream_t,   \
                                      bool, FftChoice);                                                         \
  template hipError_t launch_x_c2r<T>(const cpx<T>*, const OutSegments&, int, int, size_t, double,              \
                                      const cpx<T>*, hipStream_t, const double*, const ResidEpilogue&, bool,    \
                                      FftChoice);                                                               \
  template int x_c2r_blocks<T>(int, int, size_t, FftChoice);                                                    \
  template int x_c2r_max_blocks<T>(int, int, size_t);                                                           \
  template hipError_t launch_xform_batch<T>(int, XformBatch&, hipStream_t);                                      \
  template size_t xform_batch_prepare<T>(int, XformBatch&);
FVIM_INST(double)
FVIM_INST(float)
#undef FVIM_INST

}  // namespace fvim
