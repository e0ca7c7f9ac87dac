// Device code of the in-plane transforms (constants, register passes and the
// row/column bodies, single-grid and batched).  Included by fft.hip and
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
constexpr int NT = 256;   // threads per block of the launches over several grids
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

// TILE picks half (0), the default (1) or twice (2) the default run of a
// transform kernel on its strided side; the tuner times the three.
__host__ __device__ constexpr int tile_scale(int base, int tile) {
  return tile == 0 ? base / 2 : (tile == 2 ? base * 2 : base);
}
// Elements of a transform per thread.  16: 64 registers of float64 values.  8 up
// to length 128: short grids are bound by the chain of one thread's loads, passes
// and stores (64 x 64 x 16 float64 27.6 -> 25.4 us, 32 x 32 x 16 21.6 -> 19.8 us; at
// 256 no gain).  In rows of 16 4: with 8 two threads share a row and a load touches
// 16 bytes of every line (x_fwd / x_inv 48.6 / 29.6 -> 33.1 / 23.5 us at 16 x 2048 x 40).
// In the columns 32 in float32 from length 1024 on (512 threads per
// tile instead of 1024: y_fwd 833 -> 787 us at 1024^2 x 64), but not below (at 256 and
// 512 the passes take 150 to 170 registers, two waves per SIMD: y_inv 541 against
// 460 us at 512^2 x 128), and not in the rows (the packing has as many values again:
// 165 to 212 registers).
__host__ __device__ constexpr int row_elems(int n) {
  const int v = n <= 16 ? 4 : (n <= 128 ? 8 : 16);
  return n < v ? n : v;
}
template <typename T>
__host__ __device__ constexpr int reg_elems(int n) {
  const int v = sizeof(T) == 4 && n >= 1024 ? 32 : (n <= 128 ? 8 : 16);
  return n < v ? n : v;
}

// Columns (planes) per block of the column (y) kernels.  The mode-major side
// S[kx][ky][p] is touched in runs of B consecutive planes: 128 bytes, whole
// lines, by default (half or twice that with TILE 0 or 2), as far as a block of
// 1024 threads with reg_elems values each allows.  64-byte runs: y_inv 104
// against 71 us at 256^2 x 64 in float64, 1925 against 1360 at 1024^2 x 64.  THIN:
// 4 planes, for a traction's 3 or the surface displacement's 1, where most of a
// default tile's threads only repeat the others' loads (y_fwd of 3 planes 32.6 ->
// 16.8 us at 1024^2 in float64, 40.5 -> 14.9 in float32, y_inv of 1 plane 31.7 -> 21.4
// and 33.6 -> 18.7).
constexpr int THIN = 3;
template <typename T>
__host__ __device__ constexpr int col_batch(int n, int tile) {
  int b = tile == THIN ? 4 : tile_scale(128, tile) / (int)sizeof(cpx<T>);
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

// Row pairs (two rows of reals are one complex transform) per block of the row
// (x) kernels.  The X[p][kx][y] side is touched in runs of 2 row_seq elements
// of one kx: 128 bytes by default, as far as a block of 1024 threads allows (half
// that: 1662 / 1619 us against 1364 / 1381 for x_fwd / x_inv at 1024^2 x 64 float64);
// of 512 at 4096 in float64, where 1024 threads of 128 registers spill: x_fwd 91 -> 75
// us at 4096 x 32 x 16, 332 -> 259 at 4096 x 256 x 8 (x_inv 81 -> 76, 306 -> 299).
// TILE 3: a block of the launches over several grids, NT threads.
template <typename T>
__host__ __device__ constexpr int row_seq(int n, int tile) {
  const int m = n / row_elems(n);
  if (tile == 3) return NT / m;
  int s = tile_scale(128, tile) / (2 * (int)sizeof(cpx<T>));
  while (s > 1 && s * m > (sizeof(T) == 8 && n >= 4096 ? 512 : 1024)) s /= 2;
  while (s * m < 64) s *= 2;            // at least one wave
  return s;
}
template <typename T>
__host__ __device__ constexpr int row_threads(int n, int tile) {
  return row_seq<T>(n, tile) * (n / row_elems(n));
}
template <typename T>
__host__ __device__ constexpr bool row_split(int n, int tile) {
  return row_seq<T>(n, tile) * n * (int)sizeof(cpx<T>) > 32 * 1024;
}
// Row of the exchange tile: element pos at pos + pos / 16, so that the first
// pass's writes (16 apart) spread over the banks, and row pairs so far apart that
// the unpacking, rows fastest, does too (w elements are 256 bytes).
template <typename T>
__host__ __device__ constexpr int row_ld(int n, int tile) {
  const int esz = row_split<T>(n, tile) ? (int)sizeof(T) : (int)sizeof(cpx<T>);
  const int w = 256 / esz, len = n + n / 16, s = row_seq<T>(n, tile);
  if (n < 4 * w) return len | 1;
  return (len + w - 1) / w * w + (s < w ? w / s : 1);
}
template <typename T>
__host__ __device__ constexpr int row_lds_bytes(int n, int tile) {
  return row_seq<T>(n, tile) * row_ld<T>(n, tile) * (int)(row_split<T>(n, tile) ? sizeof(T) : sizeof(cpx<T>));
}
// Partial sums of a plane of nx x ny reals: one for each wave that holds its row
// pairs, two rows per nx / row_elems(nx) threads, whatever the block's size.
__host__ __device__ constexpr int row_sums(int nx, int ny) {
  const int w = (ny / 2) * (nx / row_elems(nx)) / 64;
  return w > 1 ? w : 1;
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
    butterfly4<INV>(a);
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
// allows, so that only the passes, not the stages, exchange through LDS.
//
// A Stockham stage of radix R for sub-transforms of length ns takes elements
// j + m N/R (m < R), turned by w^(m k N/(R ns)) with k = j mod ns, and writes its
// butterfly's results to (j / ns) ns R + k + m ns.
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
    for (int m1 = 0; m1 < R1; ++m1) {
      // Float64 columns of 4096, 1024 threads of 128 registers: the groups one after
      // the other, or their twiddles, loaded all at once, spill (y_fwd / y_inv 275 / 368
      // -> 256 / 317 us at 256 x 4096 x 8).
      if constexpr (sizeof(T) == 8 && N >= 4096) __builtin_amdgcn_sched_barrier(0);
      group_stages<T, INV, N, LS + ilog2c(R1), ZERO>(v + m1 * S, k + (m1 << LS), tw, Radices<Rest...>{});
    }
  }
}
// register index of a group's values -> its output index idx
template <int R1, int... Rest>
__host__ __device__ constexpr int group_index(int reg, Radices<R1, Rest...>) {
  constexpr int S = (1 * ... * Rest);
  if constexpr (sizeof...(Rest) == 0) return reg;
  else return reg / S + R1 * group_index(reg % S, Radices<Rest...>{});
}

// The stages of a length-2^LOGN transform from sub-length 2^LS on.  RADIX 4: one
// radix-2 stage first when LOGN is odd, then radix 4; RADIX 8: one radix-2 or
// radix-4 stage first when LOGN mod 3 is 1 or 2, then radix 8.
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
// one grid) using the LDS tile (and, x_c2r, red, a double per wave), shared by the
// single-grid kernels and by the kernels that serve several grids in one
// launch.

// Rows of nx = 2^LOGN reals -> half spectra.  Block = R consecutive rows of
// one plane (R even, R | ny), two rows per complex sequence.  Output
// X[(plane * kxh + k) * ny + y].
// If bsum is not NULL (float32), every wave also writes the float64 sum of its rows there
// (the plane means of the mean mode are then formed in float64): the waves of a
// plane hold the same rows with every tile, so that the sums do not depend on it.
template <typename T, int LOGN, bool NTL, int TILE, int RADIX>
__device__ __forceinline__ void x_r2c_body(char* tile, int lb, const InSegments& seg,
                                           cpx<T>* __restrict__ out, int ny, int R,
                                           const cpx<T>* __restrict__ tw, double* __restrict__ bsum,
                                           const LayerSkip& skip) {
  constexpr int N = 1 << LOGN, V = row_elems(N), M = N / V;
  constexpr int SEQ = row_seq<T>(N, TILE), NTH = row_threads<T>(N, TILE), ld = row_ld<T>(N, TILE);
  constexpr bool SPLIT = row_split<T>(N, TILE);
  constexpr int kxh = N / 2 + 1;
  using E = std::conditional_t<SPLIT, T, cpx<T>>;
  const size_t row0 = (size_t)lb * R;
  const size_t plane = row0 / ny;
  const int y0 = (int)(row0 - plane * ny);
  const int s = (int)threadIdx.x / M, t = (int)threadIdx.x % M, hp = R / 2;
  constexpr bool SUMS = sizeof(T) == 4;  // (float64 has its mean mode in the depth pass)
  auto put_sum = [&](double v) {         // of the wave (one that holds rows)
    if ((threadIdx.x & 63) == 0 && s < hp)
      bsum[plane * row_sums(N, ny) + ((size_t)(y0 / 2) * M + threadIdx.x) / 64] = v;
  };
  // a layer without plastic strain: its rows sum to zero, nothing to transform
  if (skip.zact && (int)plane < skip.nw && (int)(plane % skip.nz) >= *skip.zact) {
    if (SUMS && bsum) put_sum(0.0);
    return;
  }
  const int sg = (seg.n > 1 && (int)plane >= seg.first[1]) ? 1 : 0;
  const double* in = seg.ptr[sg] + ((plane - seg.first[sg]) * ny + y0) * (size_t)N;
  // threads of a row pair in x order; those past the last pair repeat it (never
  // stored), so every load is unconditional
  const double* r0 = in + (size_t)(2 * min(s, hp - 1)) * N + t;
  double a[V], b[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    a[e] = ld_in<NTL>(r0 + e * M);
    b[e] = ld_in<NTL>(r0 + N + e * M);
  }
  cpx<T> v[V];
#pragma unroll
  for (int e = 0; e < V; ++e) v[e] = mk((T)a[e], (T)b[e]);
  if (SUMS && bsum) {
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < V; ++e) acc += a[e] + b[e];
    if (s >= hp) acc = 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    put_sum(acc);
  }
  E* lds = reinterpret_cast<E*>(tile);
  auto at = [lds](int q, int pos) { return lds + q * ld + pos + (pos >> 4); };
  auto mine = [at, s](int pos) { return at(s, pos); };
  reg_fft<T, LOGN, false, RADIX, V, 0, SPLIT>(v, t, mine, t, mine, tw);
  // X of the two rows from Z[k] and Z[N - k], rows fastest
  const int lr = __builtin_ctz(R), tot = kxh * R;
  cpx<T>* dst = out + plane * kxh * ny + y0;
  constexpr int MO = (kxh * 2 * SEQ + NTH - 1) / NTH;
  if constexpr (M > 1) __syncthreads();              // the last exchange has been read
  if constexpr (SPLIT) {
    T zx[MO], cx[MO];
#pragma unroll
    for (int e = 0; e < V; ++e) *mine(t + e * M) = v[e].x;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < MO; ++u) {
      const int i = min((int)threadIdx.x + u * NTH, tot - 1);
      const int k = i >> lr, p = (i & (R - 1)) >> 1;
      zx[u] = *at(p, k);
      cx[u] = *at(p, (N - k) & (N - 1));
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < V; ++e) *mine(t + e * M) = v[e].y;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < MO; ++u) {
      const int i = (int)threadIdx.x + u * NTH;
      if (i < tot) {
        const int k = i >> lr, y = i & (R - 1);
        const T zy = *at(y >> 1, k), cy = *at(y >> 1, (N - k) & (N - 1));
        dst[(size_t)k * ny + y] = (y & 1) == 0 ? mk(T(0.5) * (zx[u] + cx[u]), T(0.5) * (zy - cy))
                                               : mk(T(0.5) * (zy + cy), T(0.5) * (cx[u] - zx[u]));
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < V; ++e) *mine(t + e * M) = v[e];
    __syncthreads();
    for (int i = threadIdx.x; i < tot; i += NTH) {
      const int k = i >> lr, y = i & (R - 1);
      const cpx<T> Z = *at(y >> 1, k), Zc = *at(y >> 1, (N - k) & (N - 1));
      dst[(size_t)k * ny + y] = (y & 1) == 0 ? mk(T(0.5) * (Z.x + Zc.x), T(0.5) * (Z.y - Zc.y))
                                             : mk(T(0.5) * (Z.y + Zc.y), T(0.5) * (Zc.x - Z.x));
    }
  }
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
template <typename T, int LOGN, int TILE, int RADIX>
__device__ __forceinline__ void x_c2r_body(char* tile, double* red, int lb, const cpx<T>* __restrict__ in,
                                           const OutSegments& seg, int ny, int R, double scale,
                                           const cpx<T>* __restrict__ tw, const double* __restrict__ padd,
                                           const ResidEpilogue& ep, bool nts) {
  constexpr int N = 1 << LOGN, V = row_elems(N), M = N / V;
  constexpr int SEQ = row_seq<T>(N, TILE), NTH = row_threads<T>(N, TILE), ld = row_ld<T>(N, TILE);
  constexpr bool SPLIT = row_split<T>(N, TILE);
  constexpr int kxh = N / 2 + 1;
  constexpr int nyq = N / 2;
  using E = std::conditional_t<SPLIT, T, cpx<T>>;
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
  cpx<T> w[MV];
  {
    const cpx<T>* src = in + (size_t)plane * kxh * ny + y0;
#pragma unroll
    for (int u = 0; u < MV; ++u) {
      const int i = min((int)threadIdx.x + u * NTH, last);
      const int k = i >> lr, y = i & (R - 1);
      w[u] = src[(size_t)k * ny + y];
    }
  }
  E* lds = reinterpret_cast<E*>(tile);
  auto at = [lds](int q, int pos) { return lds + q * ld + pos + (pos >> 4); };
  const int s = (int)threadIdx.x / M, t = (int)threadIdx.x % M;
  auto mine = [at, s](int pos) { return at(s, pos); };
  // Z = X0 + i X1 at k (even lanes) and N - k (odd lanes)
#pragma unroll
  for (int u = 0; u < MV; ++u) {
    const int k = min((int)threadIdx.x + u * NTH, last) >> lr;
    const cpx<T> o = dpp_move<DPP_SWAP1>(w[u]);
    const cpx<T> X0 = odd ? o : w[u], X1 = odd ? w[u] : o;
    if (k == 0 || k == nyq) w[u] = mk(X0.x, X1.x);
    else if (!odd) w[u] = mk(X0.x - X1.y, X0.y + X1.x);
    else w[u] = mk(X0.x + X1.y, X1.x - X0.y);
  }
  auto place = [&](int u) {              // (both lanes write a pair's k = 0, nx/2: the same value)
    const int i = min((int)threadIdx.x + u * NTH, last);
    const int k = i >> lr;
    return at((i & (R - 1)) >> 1, odd ? (N - k) & (N - 1) : k);
  };
  cpx<T> v[V];
  if constexpr (SPLIT) {
#pragma unroll
    for (int u = 0; u < MV; ++u) *place(u) = w[u].x;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < V; ++e) v[e].x = *mine(t + e * M);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < MV; ++u) *place(u) = w[u].y;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < V; ++e) v[e].y = *mine(t + e * M);
  } else {
#pragma unroll
    for (int u = 0; u < MV; ++u) *place(u) = w[u];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = *mine(t + e * M);
  }
  if constexpr (M > 1) __syncthreads();
  reg_fft<T, LOGN, true, RADIX, V, 0, SPLIT>(v, t, mine, t, mine, tw);
  int sg = 0;
  while (sg + 1 < seg.n && plane >= seg.first[sg + 1]) ++sg;
  const bool live = s < hp;
  const size_t at0 = (size_t)(2 * min(s, hp - 1)) * N + t;
  double* dst = seg.ptr[sg] + ((size_t)(plane - seg.first[sg]) * ny + y0) * N + at0;
  const double add = padd ? padd[plane] : 0.0;
  if (!ep.x) {
    // the real parts are row 2 s, the imaginary parts row 2 s + 1.  The
    // operator's outputs are not read again by the operator, so they are stored
    // as streaming (non-temporal) writes, which do not displace the spectrum
    // buffers from the last-level cache -- where a wave writes whole lines.
    if (live) {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const double o0 = (double)v[e].x * scale + add, o1 = (double)v[e].y * scale + add;
        if (M >= 16 && nts) {
          __builtin_nontemporal_store(o0, dst + e * M);
          __builtin_nontemporal_store(o1, dst + N + e * M);
        } else {
          dst[e * M] = o0;
          dst[N + e * M] = o1;
        }
      }
    }
  } else {
    // residual epilogue (the residual is the first and only segment)
    const size_t off = ((size_t)plane * ny + y0) * N + at0;
    double s0 = 0.0, s1 = 0.0;
    if (live) {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const size_t i0 = off + e * M, i1 = i0 + N;
        const double ra = ep.x[i0] - ((double)v[e].x * scale + add);
        const double rb = ep.x[i1] - ((double)v[e].y * scale + add);
        dst[e * M] = ra;
        dst[N + e * M] = rb;
        s0 += ra * ra + rb * rb;
        if (ep.Fo) {
          const double fa = ep.Fo[i0], fb = ep.Fo[i1];
          s1 += fa * (ra - fa) + fb * (rb - fb);
        }
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

// --------------------------------------------- kernels over several grids
// One launch serves the grids of an XformBatch (transform lengths up to
// 2^XFORM_BATCH_MAX_LOGN; rows in blocks of NT threads, columns in the default tile or,
// where it takes more, half of it; radix 4): block b belongs to grid
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
__device__ __forceinline__ void x_r2c_batch_block(const XformBatch& b, int blk) {
  const int c = batch_grid(b, blk);
  const int lb = blk - b.first[c];
  char* tile = reinterpret_cast<char*>(fvim_dyn_lds);
  cpx<T>* out = static_cast<cpx<T>*>(b.out[c]);
  const cpx<T>* tw = static_cast<const cpx<T>*>(b.tw[c]);
#define CALL(L) \
  x_r2c_body<T, L, false, 3, 4>(tile, lb, b.iseg[c], out, b.ny[c], b.R[c], tw, b.bsum[c], LayerSkip{})
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
    y_fwd_body<T, L, false, col_shared_tile<T>(1 << L), 4>(q.lds, q.tid, q.lb, q.live, in, out, b.kxh[c],  \
                                                          b.NP[c], b.ldp[c], tw, LayerSkip{});                       \
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
    y_inv_body<T, L, false, col_shared_tile<T>(1 << L), 4>(q.lds, q.tid, q.lb, q.live, in, out, b.kxh[c],  \
                                                          b.NP[c], b.ldp[c], tw);                                    \
  }
  FVIM_BATCH_LOGN_SWITCH(b.logn[c], CALL)
#undef CALL
}

template <typename T>
__device__ __forceinline__ void x_c2r_batch_block(const XformBatch& b, int blk, double* red) {
  const int c = batch_grid(b, blk);
  const int lb = blk - b.first[c];
  char* tile = reinterpret_cast<char*>(fvim_dyn_lds);
  const cpx<T>* in = static_cast<const cpx<T>*>(b.in[c]);
  const cpx<T>* tw = static_cast<const cpx<T>*>(b.tw[c]);
#define CALL(L) \
  x_c2r_body<T, L, 3, 4>(tile, red, lb, in, b.oseg[c], b.ny[c], b.R[c], 1.0, tw, b.padd[c], ResidEpilogue{}, \
                         b.nts[c] != 0)
  FVIM_BATCH_LOGN_SWITCH(b.logn[c], CALL)
#undef CALL
}

}  // namespace
}  // namespace fvim
