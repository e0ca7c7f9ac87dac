// Device code of the in-plane transforms (constants, LDS Stockham stages and
// the row/column bodies, single-grid and batched).  Included by fft.hip and
// persist.hip; everything is in an anonymous namespace (one copy per
// translation unit).
#pragma once
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace fvim {
namespace {


#ifndef FVIM_NT_DEFINED
#define FVIM_NT_DEFINED
constexpr int NT = 256;   // threads per block (the transforms of one grid: tile_threads)
#endif

// a times the twiddle w (its conjugate for INV), with its fused operations
// spelled out: left to the compiler, which product of a sum is fused depends on
// the code around it, and results would differ in their last bits between a
// kernel's variants.
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <bool INV, typename T>
__device__ __forceinline__ cpx<T> turn(cpx<T> a, cpx<T> w) {
  const T p = a.y * w.y, q = a.x * w.y;
  return mk(fma_t(a.x, w.x, INV ? p : -p), fma_t(a.y, w.x, INV ? -q : q));
}

// Complex elements of one block's LDS tile in the row kernels.  TILE picks
// half (0), the default (1) or twice (2) the default, which was chosen per
// kernel and precision by measurement on 256^2 x 64: a smaller tile lets
// more blocks share a CU (the forward transform gains: 16 KiB in float64),
// a larger one gives the inverse transform's strided reads longer runs
// (32 KiB in float64; 16 KiB in float32).  The tuner times the three.
__host__ __device__ constexpr int tile_scale(int base, int tile) {
  return tile == 0 ? base / 2 : (tile == 2 ? base * 2 : base);
}
template <typename T>
__host__ __device__ constexpr int r2c_tile_elems(int tile) { return tile_scale(sizeof(T) == 8 ? 1024 : 2048, tile); }
template <typename T>
__host__ __device__ constexpr int c2r_tile_elems(int tile) { return tile_scale(2048, tile); }
// Row pairs per block of a row kernel (R = 2 SEQ rows of length n).  The
// X[p][kx][y] side is touched in runs of R elements of one kx, so SEQ is the
// tile's share but at least what gives runs of ROW_RUN bytes, as far as the
// 160 KiB of LDS a block may use and a tile of 8192 elements (the loads of a
// whole tile are staged in registers) allow.  (At nx = 1024 in float64 a 16 KiB
// tile alone gives 2-row blocks, 32-byte runs and 1.5 TB/s.)
constexpr int ROW_RUN = 128;
__host__ __device__ constexpr int row_seq(int n, int csize, int tile) {
  int seq = tile / n;
  if (seq < 1) seq = 1;
  const int minseq = ROW_RUN / (2 * csize);
  if (seq < minseq) seq = minseq;
  while (seq > 1 && (seq * (n + 1) * csize > 160 * 1024 || seq * n > 8192)) seq /= 2;
  return seq;
}
template <typename T>
__host__ __device__ constexpr int r2c_seq(int n, int tile) {
  return row_seq(n, (int)sizeof(cpx<T>), r2c_tile_elems<T>(tile));
}
template <typename T>
__host__ __device__ constexpr int c2r_seq(int n, int tile) {
  return row_seq(n, (int)sizeof(cpx<T>), c2r_tile_elems<T>(tile));
}
// Elements of a transform per thread of a column kernel: 64 registers of
// float64 values.  In float32 32 values from length 1024 on (512 threads per
// tile instead of 1024: y_fwd 833 -> 787 us at 1024^2 x 64) and 16 below (with 32
// the passes of length 256 and 512 take 150 to 170 registers, two waves per SIMD:
// y_inv 541 against 460 us at 512^2 x 128).
template <typename T>
__host__ __device__ constexpr int reg_elems(int n) {
  const int v = sizeof(T) == 4 && n >= 1024 ? 32 : 16;
  return n < v ? n : v;
}

// Columns (planes) per block of the column (y) kernels.  The mode-major side
// S[kx][ky][p] is touched in runs of B consecutive planes: 128 bytes, whole
// lines, by default (half or twice that with TILE 0 or 2), as far as a block of
// 1024 threads with reg_elems values each allows.  64-byte runs: y_inv 104
// against 71 us at 256^2 x 64 in float64, 1925 against 1360 at 1024^2 x 64.
template <typename T>
__host__ __device__ constexpr int col_batch(int n, int tile) {
  int b = tile_scale(128, tile) / (int)sizeof(cpx<T>);
  const int m = n / reg_elems<T>(n);
  while (b > 1 && b * m > 1024) b /= 2;
  while (b * m < 64) b *= 2;            // at least one wave
  return b;
}
template <typename T>
__host__ __device__ constexpr int col_threads(int n, int tile) {
  return col_batch<T>(n, tile) * (n / reg_elems<T>(n));
}
// Exchange the parts one after the other where the whole tile is over 32 KiB:
// at 64 KiB only two blocks share a CU (splitting a 32 KiB tile too gains
// nothing: y_inv 72.9 against 70.6 us at 256^2 x 64).
template <typename T>
__host__ __device__ constexpr bool col_split(int n, int tile) {
  return col_batch<T>(n, tile) * n * (int)sizeof(cpx<T>) > 32 * 1024;
}
template <typename T>
__host__ __device__ constexpr int col_lds_bytes(int n, int tile) {
  return col_batch<T>(n, tile) * n * (int)sizeof(cpx<T>) / (col_split<T>(n, tile) ? 2 : 1);
}

// Threads per block of a tile of `bytes` of LDS: 8 float64 elements per thread
// up to 1024 threads, so that a larger tile does not mean fewer waves per CU
// (64 KiB tiles on 256 threads left 8 waves per CU and ran at 3 to 3.7 TB/s).
__host__ __device__ constexpr int tile_threads(int bytes) {
  return bytes > 64 * 1024 ? 1024 : (bytes > 32 * 1024 ? 512 : 256);
}
template <typename T>
__host__ __device__ constexpr int r2c_threads(int n, int tile) {
  return tile_threads(r2c_seq<T>(n, tile) * n * (int)sizeof(cpx<T>));
}
template <typename T>
__host__ __device__ constexpr int c2r_threads(int n, int tile) {
  return tile_threads(c2r_seq<T>(n, tile) * n * (int)sizeof(cpx<T>));
}
__host__ __device__ constexpr int ilog2c(int n) { return n <= 1 ? 0 : 1 + ilog2c(n / 2); }

// Radix-R butterfly (R = 2, 4, 8) of the DFT with kernel exp(-2 pi i / R)
// (its conjugate for INV), in place on a[0 .. R).
template <typename T, int R, bool INV>
__device__ __forceinline__ void butterfly(cpx<T>* a) {
  if constexpr (R == 2) {
    const cpx<T> a0 = a[0], a1 = a[1];
    a[0] = add(a0, a1);
    a[1] = sub(a0, a1);
  } else if constexpr (R == 4) {
    const cpx<T> s02 = add(a[0], a[2]), d02 = sub(a[0], a[2]);
    const cpx<T> s13 = add(a[1], a[3]), d13 = sub(a[1], a[3]);
    // forward: y1 = d02 - i d13, y3 = d02 + i d13 (conjugate for inverse)
    const cpx<T> id13 = INV ? mul_i(d13) : mul_mi(d13);
    a[0] = add(s02, s13);
    a[1] = add(d02, id13);
    a[2] = sub(s02, s13);
    a[3] = sub(d02, id13);
  } else {
    static_assert(R == 8, "radix 2, 4 or 8");
    // two length-4 transforms (even and odd inputs), then the odd ones
    // turned by w^p, w = exp(-+ 2 pi i / 8), and combined
    cpx<T> e[4] = {a[0], a[2], a[4], a[6]};
    cpx<T> o[4] = {a[1], a[3], a[5], a[7]};
    butterfly<T, 4, INV>(e);
    butterfly<T, 4, INV>(o);
    const T c = T(0.70710678118654752440084436210485);
    cpx<T> t1, t3;
    if (INV) {
      t1 = mk((o[1].x - o[1].y) * c, (o[1].x + o[1].y) * c);      // (1 + i)/sqrt2
      t3 = mk(-(o[3].x + o[3].y) * c, (o[3].x - o[3].y) * c);     // (-1 + i)/sqrt2
    } else {
      t1 = mk((o[1].x + o[1].y) * c, (o[1].y - o[1].x) * c);      // (1 - i)/sqrt2
      t3 = mk((o[3].y - o[3].x) * c, -(o[3].x + o[3].y) * c);     // (-1 - i)/sqrt2
    }
    const cpx<T> t2 = INV ? mul_i(o[2]) : mul_mi(o[2]);
    a[0] = add(e[0], o[0]);
    a[4] = sub(e[0], o[0]);
    a[1] = add(e[1], t1);
    a[5] = sub(e[1], t1);
    a[2] = add(e[2], t2);
    a[6] = sub(e[2], t2);
    a[3] = add(e[3], t3);
    a[7] = sub(e[3], t3);
  }
}

// One self-sorting (Stockham) radix-R stage of NB transforms of length
// N = 2^LOGN held at buf[b * ld + k] (NB <= NBMAX), for sub-transforms of
// length ns = 2^LS: butterfly j of a transform takes elements j + m N/R,
// turned by w^(m k N/(R ns)) with k = j mod ns, and writes them to
// (j / ns) ns R + k + m ns.  Called by all NTH threads.
template <typename T, int LOGN, int NBMAX, bool INV, int R, int LS, int NTH>
__device__ __forceinline__ void stockham_stage(cpx<T>* buf, int ld, int NB, const cpx<T>* __restrict__ tw) {
  constexpr int N = 1 << LOGN;
  constexpr int LR = ilog2c(R);
  constexpr int M = N / R;
  constexpr int ns = 1 << LS;
  constexpr int tstep = M >> LS;
  constexpr int MB = (NBMAX * M + NTH - 1) / NTH;
  const int tid = threadIdx.x;
  const int nb = NB * M;
  cpx<T> v[MB][R];
#pragma unroll
  for (int u = 0; u < MB; ++u) {
    const int j = tid + u * NTH;
    if (j < nb) {
      const int b = j >> (LOGN - LR), jj = j & (M - 1);
      const cpx<T>* src = buf + b * ld + jj;
#pragma unroll
      for (int m = 0; m < R; ++m) v[u][m] = src[m * M];
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < MB; ++u) {
    const int j = tid + u * NTH;
    if (j < nb) {
      const int b = j >> (LOGN - LR), jj = j & (M - 1);
      const int k = jj & (ns - 1);
      if constexpr (LS > 0) {
#pragma unroll
        for (int m = 1; m < R; ++m) v[u][m] = turn<INV>(v[u][m], tw[m * k * tstep]);
      }
      butterfly<T, R, INV>(v[u]);
      const int o = b * ld + ((jj >> LS) << (LS + LR)) + k;
#pragma unroll
      for (int m = 0; m < R; ++m) buf[o + m * ns] = v[u][m];
    }
  }
  __syncthreads();
}

template <typename T, int LOGN, int NBMAX, bool INV, int R, int LS, int NTH>
__device__ __forceinline__ void stockham_from(cpx<T>* buf, int ld, int NB, const cpx<T>* __restrict__ tw) {
  if constexpr (LS < LOGN) {
    stockham_stage<T, LOGN, NBMAX, INV, R, LS, NTH>(buf, ld, NB, tw);
    stockham_from<T, LOGN, NBMAX, INV, R, LS + ilog2c(R), NTH>(buf, ld, NB, tw);
  }
}

// NB transforms of length N = 2^LOGN held at buf[b * ld + k] (NB <= NBMAX),
// Stockham autosort.  RADIX 4: one radix-2 stage first when LOGN is odd,
// then radix-4 stages; RADIX 8: one radix-2 or radix-4 stage first when
// LOGN mod 3 is 1 or 2, then radix-8 stages.  All index arithmetic is shifts
// and masks.  Called by all NTH threads.
template <typename T, int LOGN, int NBMAX, bool INV, int RADIX, int NTH>
__device__ __forceinline__ void lds_fft(cpx<T>* buf, int ld, int NB, const cpx<T>* __restrict__ tw) {
  if constexpr (RADIX == 4) {
    if constexpr (LOGN & 1) {
      stockham_stage<T, LOGN, NBMAX, INV, 2, 0, NTH>(buf, ld, NB, tw);
      stockham_from<T, LOGN, NBMAX, INV, 4, 1, NTH>(buf, ld, NB, tw);
    } else {
      stockham_from<T, LOGN, NBMAX, INV, 4, 0, NTH>(buf, ld, NB, tw);
    }
  } else {
    static_assert(RADIX == 8, "radix 4 or 8");
    if constexpr (LOGN % 3 == 1) {
      stockham_stage<T, LOGN, NBMAX, INV, 2, 0, NTH>(buf, ld, NB, tw);
      stockham_from<T, LOGN, NBMAX, INV, 8, 1, NTH>(buf, ld, NB, tw);
    } else if constexpr (LOGN % 3 == 2) {
      stockham_stage<T, LOGN, NBMAX, INV, 4, 0, NTH>(buf, ld, NB, tw);
      stockham_from<T, LOGN, NBMAX, INV, 8, 2, NTH>(buf, ld, NB, tw);
    } else {
      stockham_from<T, LOGN, NBMAX, INV, 8, 0, NTH>(buf, ld, NB, tw);
    }
  }
}

// Sum of v over the block (fixed order: waves by shuffles, then the waves in
// turn); red: NTH / 64 doubles of LDS.  Every thread gets the total.
template <int NTH>
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NTH / 64; ++w) s += red[w];
  __syncthreads();
  return s;
}

// ------------------------------------------------------- register passes
// A transform as few passes over registers: a thread holds V elements of its
// sequence, positions t + e M (M = N / V threads per sequence), and runs as many
// consecutive Stockham stages on them as their radices' product (at most V)
// allows, so that only the passes, not the stages, exchange through LDS.  Each
// stage does the same operations on the same values as stockham_stage.
//
// Stages of radices R1, Rest... from sub-transforms of length 2^LS on: the Rg
// values at positions tt + c N / Rg give outputs idx at positions
// (tt / ns) Rg ns + k + idx ns, k = tt mod ns, ns = 2^LS.  The first stage's
// butterfly over m of v[m2 + m S] (S = Rg / R1) yields the inputs of R1
// independent groups of the other stages, with k + m1 ns for their k.  ZERO: k is
// 0 (the transform's first pass), the twiddles are the same for every thread.
template <int... R>
struct Radices {};

template <typename T, bool INV, int N, int LS, bool ZERO, int R1, int... Rest>
__device__ __forceinline__ void group_stages(cpx<T>* v, int k, const cpx<T>* __restrict__ tw, Radices<R1, Rest...>) {
  constexpr int S = (1 * ... * Rest);
  if constexpr (LS > 0) {
    if (!(ZERO && k == 0)) {
      constexpr int step = N / (R1 << LS);
#pragma unroll
      for (int m = 1; m < R1; ++m) {
        const cpx<T> w = tw[m * k * step];
#pragma unroll
        for (int m2 = 0; m2 < S; ++m2) v[m2 + m * S] = turn<INV>(v[m2 + m * S], w);
      }
    }
  }
#pragma unroll
  for (int m2 = 0; m2 < S; ++m2) {
    cpx<T> a[R1];
#pragma unroll
    for (int m = 0; m < R1; ++m) a[m] = v[m2 + m * S];
    butterfly<T, R1, INV>(a);
#pragma unroll
    for (int m = 0; m < R1; ++m) v[m2 + m * S] = a[m];
  }
  if constexpr (sizeof...(Rest) > 0) {
#pragma unroll
    for (int m1 = 0; m1 < R1; ++m1)
      group_stages<T, INV, N, LS + ilog2c(R1), ZERO>(v + m1 * S, k + (m1 << LS), tw, Radices<Rest...>{});
  }
}
// register index of a group's values -> its output index idx
template <int R1, int... Rest>
__host__ __device__ constexpr int group_index(int reg, Radices<R1, Rest...>) {
  constexpr int S = (1 * ... * Rest);
  if constexpr (sizeof...(Rest) == 0) return reg;
  else return reg / S + R1 * group_index(reg % S, Radices<Rest...>{});
}

// The stages of a length-2^LOGN transform in lds_fft's order, from the one at
// sub-length 2^LS on.
template <int LOGN, int RADIX>
__host__ __device__ constexpr int stage_radix(int ls) {
  if (ls > 0) return RADIX;
  if (RADIX == 4) return LOGN & 1 ? 2 : 4;
  return LOGN % 3 == 1 ? 2 : (LOGN % 3 == 2 ? 4 : 8);
}
// The pass that starts at 2^LS: as many stages as fit into V.
template <int LOGN, int RADIX, int LS, int V, int... R>
__host__ __device__ constexpr auto pass_radices(Radices<R...> r) {
  constexpr int prod = (1 * ... * R);
  constexpr int at = LS + ilog2c(prod);
  if constexpr (at >= LOGN) {
    return r;
  } else if constexpr (prod * stage_radix<LOGN, RADIX>(at) > V) {
    return r;
  } else {
    return pass_radices<LOGN, RADIX, LS, V>(Radices<R..., stage_radix<LOGN, RADIX>(at)>{});
  }
}
template <int... R>
__host__ __device__ constexpr int radix_product(Radices<R...>) { return (1 * ... * R); }

// One transform: v[e] = element t + e M of the thread's sequence.  The first
// pass runs with the threads' places (t0, lds0), the passes after it with (t1,
// lds1): the exchange between them may hand a sequence to other threads, so
// that both the loads before and the stores after are in their best order.
// lds(pos) is the LDS place of the sequence's element pos.  SPLIT: the real and
// the imaginary parts are exchanged one after the other, in half the LDS.
template <typename T, int LOGN, bool INV, int RADIX, int V, int LS, bool SPLIT, typename L0, typename L1>
__device__ __forceinline__ void reg_fft(cpx<T> (&v)[V], int t0, L0 lds0, int t1, L1 lds1,
                                        const cpx<T>* __restrict__ tw) {
  constexpr int N = 1 << LOGN, M = N / V;
  using P = decltype(pass_radices<LOGN, RADIX, LS, V>(Radices<>{}));
  constexpr int Rg = radix_product(P{}), U = V / Rg, ns = 1 << LS;
  cpx<T> o[V];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    cpx<T> w[Rg];
#pragma unroll
    for (int c = 0; c < Rg; ++c) w[c] = v[u + c * U];
    const int k = LS == 0 ? 0 : ((t0 + u * M) & (ns - 1));
    group_stages<T, INV, N, LS, LS == 0>(w, k, tw, P{});
#pragma unroll
    for (int c = 0; c < Rg; ++c) o[u + group_index(c, P{}) * U] = w[c];
  }
  if constexpr (ns * Rg >= N) {
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = o[e];
  } else {
    // output idx of butterfly tt = t + u M is at (tt / ns) Rg ns + tt mod ns + idx ns
    int base[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tt = t0 + u * M;
      base[u] = (tt >> LS) * (Rg * ns) + (tt & (ns - 1));
    }
    if constexpr (LS > 0) __syncthreads();          // the last exchange has been read
    if constexpr (SPLIT) {
#pragma unroll
      for (int e = 0; e < V; ++e) *lds0(base[e % U] + (e / U) * ns) = o[e].x;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < V; ++e) v[e].x = *lds1(t1 + e * M);
      __syncthreads();
#pragma unroll
      for (int e = 0; e < V; ++e) *lds0(base[e % U] + (e / U) * ns) = o[e].y;
      __syncthreads();
#pragma unroll
      for (int e = 0; e < V; ++e) v[e].y = *lds1(t1 + e * M);
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e) *lds0(base[e % U] + (e / U) * ns) = o[e];
      __syncthreads();
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = *lds1(t1 + e * M);
    }
    reg_fft<T, LOGN, INV, RADIX, V, LS + ilog2c(Rg), SPLIT>(v, t1, lds1, t1, lds1, tw);
  }
}

// ------------------------------------------------------------------ bodies
// Each transform is a device body over one block's tile (logical block lb of
// one grid) using the LDS tile buf (and red, NTH/64 doubles), shared by the
// single-grid kernels and by the kernels that serve several grids in one
// launch.

// Rows of nx = 2^LOGN reals -> half spectra.  Block = R consecutive rows of
// one plane (R even, R | ny), two rows per complex sequence.  Output
// X[(plane * kxh + k) * ny + y].
// If bsum is not NULL, block lb also writes the float64 sum of its R rows to
// bsum[lb] (the plane means of the mean mode are then formed in float64).
template <typename T, int LOGN, bool NTL, int TILE, int RADIX, int NTH>
__device__ __forceinline__ void x_r2c_body(cpx<T>* buf, double* red, int lb, const InSegments& seg,
                                           cpx<T>* __restrict__ out, int ny, int R,
                                           const cpx<T>* __restrict__ tw, double* __restrict__ bsum,
                                           const LayerSkip& skip) {
  constexpr int N = 1 << LOGN;
  constexpr int SEQ = r2c_seq<T>(N, TILE);
  constexpr int ld = N + 1;
  constexpr int kxh = N / 2 + 1;
  const size_t row0 = (size_t)lb * R;
  const size_t plane = row0 / ny;
  const int y0 = (int)(row0 - plane * ny);
  // a layer without plastic strain: its rows sum to zero, nothing to transform
  if (skip.zact && (int)plane < skip.nw && (int)(plane % skip.nz) >= *skip.zact) {
    if (bsum && threadIdx.x == 0) bsum[lb] = 0.0;
    return;
  }
  const int sg = (seg.n > 1 && (int)plane >= seg.first[1]) ? 1 : 0;
  const double* in = seg.ptr[sg] + ((plane - seg.first[sg]) * ny + y0) * (size_t)N;
  // 16-byte loads: two consecutive x of one row
  constexpr int MV = (2 * SEQ * N / 2 + NTH - 1) / NTH;
  const int tot = R * N / 2;
  const double2* src = reinterpret_cast<const double2*>(in);
  double2 v[MV];
#pragma unroll
  for (int u = 0; u < MV; ++u) {
    int i = threadIdx.x + u * NTH;
    if (i < tot) v[u] = ld_in<NTL>(src + i);
  }
#pragma unroll
  for (int u = 0; u < MV; ++u) {
    int i = threadIdx.x + u * NTH;
    if (i < tot) {
      int r = (2 * i) >> LOGN, x = (2 * i) & (N - 1);
      cpx<T>* d = buf + (r >> 1) * ld + x;
      if (r & 1) { d[0].y = (T)v[u].x; d[1].y = (T)v[u].y; }
      else { d[0].x = (T)v[u].x; d[1].x = (T)v[u].y; }
    }
  }
  if (bsum) {
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < MV; ++u) {
      int i = threadIdx.x + u * NTH;
      if (i < tot) acc += v[u].x + v[u].y;
    }
    acc = block_sum<NTH>(acc, red);
    if (threadIdx.x == 0) bsum[lb] = acc;
  }
  __syncthreads();
  lds_fft<T, LOGN, SEQ, false, RADIX, NTH>(buf, ld, R / 2, tw);
  const int tot2 = kxh * R;
  for (int i = threadIdx.x; i < tot2; i += NTH) {
    int k = i / R, yl = i - k * R;
    int p = yl >> 1;
    cpx<T> Z = buf[p * ld + k];
    cpx<T> Zc = buf[p * ld + ((N - k) & (N - 1))];
    cpx<T> X;
    if ((yl & 1) == 0) X = mk(T(0.5) * (Z.x + Zc.x), T(0.5) * (Z.y - Zc.y));
    else X = mk(T(0.5) * (Z.y + Zc.y), T(0.5) * (Zc.x - Z.x));
    out[(plane * kxh + k) * ny + y0 + yl] = X;
  }
}

// Logical block index such that the blocks dispatched to one XCD (physical
// blocks b, b + 8, b + 16, ...) take consecutive logical indices.
__device__ __forceinline__ int xcd_block() {
  const int b = blockIdx.x, n = gridDim.x;
  const int x = b & 7, slot = b >> 3, per = n >> 3, rem = n & 7;
  return x * per + (x < rem ? x : rem) + slot;
}

// Threads of a column tile in two orders: y fastest (t consecutive, for the
// X side, contiguous in y) and plane fastest (b consecutive, for the mode-major
// side, runs of B planes).  The exchange tile [pos][b] has the planes of each
// position permuted by the position's bits, so that both orders, and the passes'
// strided positions, spread over the banks.
template <typename T, int LOGN, int TILE>
struct ColOrder {
  static constexpr int N = 1 << LOGN, B = col_batch<T>(N, TILE), V = reg_elems<T>(N), M = N / V;
  int b, t;
  template <bool Y_FIRST>
  static __device__ __forceinline__ ColOrder of(int tid) {
    return Y_FIRST ? ColOrder{tid / M, tid % M} : ColOrder{tid % B, tid / B};
  }
};
template <typename T, int LOGN, int TILE, bool INV, int RADIX, int V>
__device__ __forceinline__ void col_fft(cpx<T> (&v)[V], char* tile, ColOrder<T, LOGN, TILE> c0,
                                        ColOrder<T, LOGN, TILE> c1, const cpx<T>* __restrict__ tw) {
  constexpr int N = 1 << LOGN, B = col_batch<T>(N, TILE);
  constexpr bool SPLIT = col_split<T>(N, TILE);
  using E = std::conditional_t<SPLIT, T, cpx<T>>;
  E* lds = reinterpret_cast<E*>(tile);
  auto place = [lds](int b) {
    return [lds, b](int pos) { return lds + pos * B + (b ^ ((pos ^ (pos >> 3) ^ (pos >> 4)) & (B - 1))); };
  };
  reg_fft<T, LOGN, INV, RADIX, V, 0, SPLIT>(v, c0.t, place(c0.b), c1.t, place(c1.b), tw);
}

// Forward column transform: X[p][kx][y] -> S[kx][ky][p] of tile lb, up to B
// planes of one kx, by threads tid = 0 .. col_threads - 1 (a shared launch puts
// several tiles in one block: live = false for a tile past the last, which
// only keeps the barriers).  Lanes past the last plane repeat it (never
// stored), so every load is unconditional.
template <typename T, int LOGN, bool NTL, int TILE, int RADIX>
__device__ __forceinline__ void y_fwd_body(char* tile, int tid, int lb, bool live, const cpx<T>* __restrict__ in,
                                           cpx<T>* __restrict__ out, int kxh, int NP, int ldp,
                                           const cpx<T>* __restrict__ tw, const LayerSkip& skip) {
  using C = ColOrder<T, LOGN, TILE>;
  constexpr int N = C::N, B = C::B, V = C::V, M = C::M;
  const int npb = (NP + B - 1) / B;
  const int kx = lb / npb;
  const int p0 = (lb - kx * npb) * B;
  const int nb = min(B, NP - p0);
  if (skip.zact) {                     // every plane of the group in a layer without plastic strain
    const int za = *skip.zact;
    bool any = false;
    for (int b = 0; b < nb; ++b) {
      const int p = p0 + b;
      any = any || p >= skip.nw || p % skip.nz < za;
    }
    if (!any) return;
  }
  // (one pass only, M = 1: no exchange, one order)
  const C ci = C::template of<(M > 1)>(tid), co = C::template of<false>(tid);
  const cpx<T>* src = in + ((size_t)(p0 + min(ci.b, nb - 1)) * kxh + kx) * N + ci.t;
  cpx<T> v[V];
#pragma unroll
  for (int e = 0; e < V; ++e) v[e] = ld_in<NTL>(src + e * M);
  col_fft<T, LOGN, TILE, false, RADIX, V>(v, tile, ci, co, tw);
  if (co.b >= nb || !live) return;
  cpx<T>* dst = out + ((size_t)kx * N + co.t) * ldp + p0 + co.b;
#pragma unroll
  for (int e = 0; e < V; ++e) dst[(size_t)e * M * ldp] = v[e];
}

// Inverse column transform: S[kx][ky][p] -> X[p][kx][y].
template <typename T, int LOGN, bool NTL, int TILE, int RADIX>
__device__ __forceinline__ void y_inv_body(char* tile, int tid, int lb, bool live, const cpx<T>* __restrict__ in,
                                           cpx<T>* __restrict__ out, int kxh, int NP, int ldp,
                                           const cpx<T>* __restrict__ tw) {
  using C = ColOrder<T, LOGN, TILE>;
  constexpr int N = C::N, B = C::B, V = C::V, M = C::M;
  // blocks run plane group by plane group (kx fastest), so the inverse row
  // transform, which runs its blocks from the last plane back, finds the
  // planes written last still in the last-level cache
  const int kx = lb % kxh;
  const int p0 = (lb / kxh) * B;
  const int nb = min(B, NP - p0);
  const C ci = C::template of<false>(tid), co = C::template of<(M > 1)>(tid);
  const cpx<T>* src = in + ((size_t)kx * N + ci.t) * ldp + p0 + min(ci.b, nb - 1);
  cpx<T> v[V];
#pragma unroll
  for (int e = 0; e < V; ++e) v[e] = ld_in<NTL>(src + (size_t)e * M * ldp);
  col_fft<T, LOGN, TILE, true, RADIX, V>(v, tile, ci, co, tw);
  if (co.b >= nb || !live) return;
  cpx<T>* dst = out + ((size_t)(p0 + co.b) * kxh + kx) * N + co.t;
#pragma unroll
  for (int e = 0; e < V; ++e) dst[e * M] = v[e];
}

// Half spectra -> rows of nx = 2^LOGN reals, two rows per complex transform.
// Plane p of the input goes to the output segment that contains it.
// If padd is not NULL, padd[plane] (float64) is added to every output value
// of that plane (the mean mode computed in float64).  nts: the outputs
// (without the epilogue) are stored as streaming writes.
template <typename T, int LOGN, int TILE, int RADIX, int NTH>
__device__ __forceinline__ void x_c2r_body(cpx<T>* buf, double* red, int lb, const cpx<T>* __restrict__ in,
                                           const OutSegments& seg, int ny, int R, double scale,
                                           const cpx<T>* __restrict__ tw, const double* __restrict__ padd,
                                           const ResidEpilogue& ep, bool nts) {
  constexpr int N = 1 << LOGN;
  constexpr int SEQ = c2r_seq<T>(N, TILE);
  constexpr int ld = N + 1;
  constexpr int kxh = N / 2 + 1;
  constexpr int nyq = N / 2;
  const int hp = R / 2;                  // a power of two (R = ny or 2 SEQ)
  const int lr = __builtin_ctz(R);
  // one element per lane, consecutive lanes on consecutive rows y of one kx
  // (runs of R elements); slots past the end repeat the last row pair, which
  // writes the same values again.  The rows 2 pr, 2 pr + 1 of a pair sit in
  // lanes 2 j, 2 j + 1 and are exchanged by a DPP lane swap.
  const int totr = kxh * R;
  const bool odd = threadIdx.x & 1;
  const int last = totr - (odd ? 1 : 2);
  constexpr int MV = (kxh * 2 * SEQ + NTH - 1) / NTH;
  const size_t row0 = (size_t)lb * R;
  const int plane = (int)(row0 / ny);
  const int y0 = (int)(row0 - (size_t)plane * ny);
  cpx<T> v[MV];
  {
    const cpx<T>* src = in + (size_t)plane * kxh * ny + y0;
#pragma unroll
    for (int u = 0; u < MV; ++u) {
      const int i = min((int)threadIdx.x + u * NTH, last);
      const int k = i >> lr, y = i & (R - 1);
      v[u] = src[(size_t)k * ny + y];
    }
  }
  {
#pragma unroll
    for (int u = 0; u < MV; ++u) {
      const int i = min((int)threadIdx.x + u * NTH, last);
      const int k = i >> lr, pr = (i & (R - 1)) >> 1;
      const cpx<T> o = dpp_move<DPP_SWAP1>(v[u]);
      const cpx<T> X0 = odd ? o : v[u], X1 = odd ? v[u] : o;
      if (k == 0 || k == nyq) {
        if (!odd) buf[pr * ld + k] = mk(X0.x, X1.x);
      } else if (!odd) {
        buf[pr * ld + k] = mk(X0.x - X1.y, X0.y + X1.x);
      } else {
        buf[pr * ld + N - k] = mk(X0.x + X1.y, X1.x - X0.y);
      }
    }
    __syncthreads();
    lds_fft<T, LOGN, SEQ, true, RADIX, NTH>(buf, ld, hp, tw);
    int s = 0;
    while (s + 1 < seg.n && plane >= seg.first[s + 1]) ++s;
    double* dst = seg.ptr[s] + ((size_t)(plane - seg.first[s]) * ny + y0) * N;
    const double add = padd ? padd[plane] : 0.0;
    typedef double v2d __attribute__((ext_vector_type(2)));
    if (!ep.x) {
      // Each thread stores one x pair of a row pair: the real parts of the
      // two LDS elements it reads go to row 2 pr, their imaginary parts to
      // row 2 pr + 1.  The operator's outputs are not read again by the
      // operator, so they are stored as streaming (non-temporal) writes,
      // which do not displace the spectrum buffers from the last-level
      // cache.
      const int tot4 = hp * (N / 2);
      for (int i = threadIdx.x; i < tot4; i += NTH) {
        const int pr = (2 * i) >> LOGN, x = (2 * i) & (N - 1);
        const cpx<T>* b = buf + pr * ld + x;
        const cpx<T> b0 = b[0], b1 = b[1];
        v2d o0, o1;
        o0.x = (double)b0.x * scale + add;
        o0.y = (double)b1.x * scale + add;
        o1.x = (double)b0.y * scale + add;
        o1.y = (double)b1.y * scale + add;
        v2d* q0 = reinterpret_cast<v2d*>(dst) + (size_t)(2 * pr) * (N / 2) + (x >> 1);
        v2d* q1 = q0 + (N / 2);
        if (nts) {
          __builtin_nontemporal_store(o0, q0);
          __builtin_nontemporal_store(o1, q1);
        } else {
          *q0 = o0;
          *q1 = o1;
        }
      }
    } else {
      // residual epilogue (the residual is the first and only segment)
      const int tot2 = R * N / 2;
      double2* d2 = reinterpret_cast<double2*>(dst);
      const size_t off = ((size_t)plane * ny + y0) * N;
      const double2* x2 = reinterpret_cast<const double2*>(ep.x + off);
      const double2* f2 = ep.Fo ? reinterpret_cast<const double2*>(ep.Fo + off) : nullptr;
      double s0 = 0.0, s1 = 0.0;
      for (int i = threadIdx.x; i < tot2; i += NTH) {
        int r = (2 * i) >> LOGN, x = (2 * i) & (N - 1);
        const cpx<T>* b = buf + (r >> 1) * ld + x;
        double2 o;
        if (r & 1) { o.x = (double)b[0].y * scale + add; o.y = (double)b[1].y * scale + add; }
        else { o.x = (double)b[0].x * scale + add; o.y = (double)b[1].x * scale + add; }
        const double2 xv = x2[i];
        const double2 rr = make_double2(xv.x - o.x, xv.y - o.y);
        d2[i] = rr;
        s0 += rr.x * rr.x + rr.y * rr.y;
        if (f2) {
          const double2 f = f2[i];
          s1 += f.x * (rr.x - f.x) + f.y * (rr.y - f.y);
        }
      }
      const double a = block_sum<NTH>(s0, red);
      const double c = block_sum<NTH>(s1, red);
      if (threadIdx.x == 0) {
        const int cp = plane / ep.nz, z = plane - cp * ep.nz;
        const double wt = (cp < 3 ? 1.0 : 2.0) * (ep.wz ? ep.wz[z] : ((z == 0 || z == ep.nz - 1) ? 0.5 : 1.0));
        ep.part[2 * lb] = wt * a;
        ep.part[2 * lb + 1] = wt * c;
      }
    }
  }
}

// --------------------------------------------- kernels over several grids
// One launch serves the grids of an XformBatch (transform lengths up to
// 2^XFORM_BATCH_MAX_LOGN, default tile and radix 4): block b belongs to grid
// c with first[c] <= b < first[c + 1] and runs that grid's body with the
// block index b - first[c]; the tile lives in dynamic LDS sized by the host
// for the largest grid.  A grid's results are those of its own launch.
extern __shared__ double2 fvim_dyn_lds[];

__device__ __forceinline__ int batch_grid(const XformBatch& b, int blk) {
  int c = 0;
  while (c + 1 < b.n && blk >= b.first[c + 1]) ++c;
  return c;
}

#define FVIM_BATCH_LOGN_SWITCH(logn, CALL) \
  switch (logn) {                          \
    case 2: CALL(2); break;                \
    case 3: CALL(3); break;                \
    case 4: CALL(4); break;                \
    case 5: CALL(5); break;                \
    case 6: CALL(6); break;                \
    case 7: CALL(7); break;                \
    case 8: CALL(8); break;                \
    case 9: CALL(9); break;                \
  }

// Tile of a thread in a column launch over several grids: blocks of NT threads
// hold NT / col_threads tiles each, of the default choice or, where that takes
// more threads, half of it.
struct ColTile {
  char* lds;
  int tid, lb;
  bool live;
};
template <typename T>
__host__ __device__ constexpr int col_shared_tile(int n) { return col_threads<T>(n, 1) > NT ? 0 : 1; }
template <typename T, int LOGN>
__device__ __forceinline__ ColTile col_tile(int blk, int kxh, int NP) {
  constexpr int N = 1 << LOGN, TILE = col_shared_tile<T>(N);
  constexpr int TH = col_threads<T>(N, TILE), G = NT / TH, B = col_batch<T>(N, TILE);
  static_assert(TH <= NT && NT % TH == 0, "tiles of a shared launch");
  const int g = threadIdx.x / TH, tiles = kxh * ((NP + B - 1) / B);
  ColTile q;
  q.lds = reinterpret_cast<char*>(fvim_dyn_lds) + (size_t)g * col_lds_bytes<T>(N, TILE);
  q.tid = threadIdx.x - g * TH;
  q.lb = blk * G + g;
  q.live = q.lb < tiles;
  if (!q.live) q.lb = tiles - 1;
  return q;
}

// One block of each batched transform (block blk of the launch over the
// table b); the kernels below and the persistent batched operator run them.
template <typename T>
__device__ __forceinline__ void x_r2c_batch_block(const XformBatch& b, int blk, double* red) {
  const int c = batch_grid(b, blk);
  const int lb = blk - b.first[c];
  cpx<T>* buf = reinterpret_cast<cpx<T>*>(fvim_dyn_lds);
  cpx<T>* out = static_cast<cpx<T>*>(b.out[c]);
  const cpx<T>* tw = static_cast<const cpx<T>*>(b.tw[c]);
#define CALL(L) x_r2c_body<T, L, false, 1, 4, NT>(buf, red, lb, b.iseg[c], out, b.ny[c], b.R[c], tw, b.bsum[c], LayerSkip{})
  FVIM_BATCH_LOGN_SWITCH(b.logn[c], CALL)
#undef CALL
}

template <typename T>
__device__ __forceinline__ void y_fwd_batch_block(const XformBatch& b, int blk) {
  const int c = batch_grid(b, blk);
  const int lb = blk - b.first[c];
  const cpx<T>* in = static_cast<const cpx<T>*>(b.in[c]);
  cpx<T>* out = static_cast<cpx<T>*>(b.out[c]);
  const cpx<T>* tw = static_cast<const cpx<T>*>(b.tw[c]);
#define CALL(L)                                                                                                \
  {                                                                                                            \
    const ColTile q = col_tile<T, L>(lb, b.kxh[c], b.NP[c]);                                                   \
    y_fwd_body<T, L, false, col_shared_tile<T>(1 << L), 4>(q.lds, q.tid, q.lb, q.live, in, out, b.kxh[c], b.NP[c],       \
                                  b.ldp[c], tw, LayerSkip{});                                                  \
  }
  FVIM_BATCH_LOGN_SWITCH(b.logn[c], CALL)
#undef CALL
}

template <typename T>
__device__ __forceinline__ void y_inv_batch_block(const XformBatch& b, int blk) {
  const int c = batch_grid(b, blk);
  const int lb = blk - b.first[c];
  const cpx<T>* in = static_cast<const cpx<T>*>(b.in[c]);
  cpx<T>* out = static_cast<cpx<T>*>(b.out[c]);
  const cpx<T>* tw = static_cast<const cpx<T>*>(b.tw[c]);
#define CALL(L)                                                                                                \
  {                                                                                                            \
    const ColTile q = col_tile<T, L>(lb, b.kxh[c], b.NP[c]);                                                   \
    y_inv_body<T, L, false, col_shared_tile<T>(1 << L), 4>(q.lds, q.tid, q.lb, q.live, in, out, b.kxh[c], b.NP[c],       \
                                  b.ldp[c], tw);                                                               \
  }
  FVIM_BATCH_LOGN_SWITCH(b.logn[c], CALL)
#undef CALL
}

template <typename T>
__device__ __forceinline__ void x_c2r_batch_block(const XformBatch& b, int blk, double* red) {
  const int c = batch_grid(b, blk);
  const int lb = blk - b.first[c];
  cpx<T>* buf = reinterpret_cast<cpx<T>*>(fvim_dyn_lds);
  const cpx<T>* in = static_cast<const cpx<T>*>(b.in[c]);
  const cpx<T>* tw = static_cast<const cpx<T>*>(b.tw[c]);
#define CALL(L) \
  x_c2r_body<T, L, 1, 4, NT>(buf, red, lb, in, b.oseg[c], b.ny[c], b.R[c], 1.0, tw, b.padd[c], ResidEpilogue{}, \
                         b.nts[c] != 0)
  FVIM_BATCH_LOGN_SWITCH(b.logn[c], CALL)
#undef CALL
}

}  // namespace
}  // namespace fvim
