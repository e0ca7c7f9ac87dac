// Transforms of single surface planes (float64) for the contact iterations:
// the building blocks of their fused kernels.  Included by contact.hip and
// friction.hip; everything is in an anonymous namespace (one copy per
// translation unit).
//
// A surface transform is small (1 MB at 256^2), so it is bound by the latency
// of its kernels, not by bandwidth.  Blocks are therefore as small as one
// wave (as many blocks as possible share the work), a thread holds exactly one
// radix-4 butterfly, its twiddles are loaded once, beside its data, instead of
// between the stages, and the stages exchange through two LDS tiles in turn,
// one barrier each.  The spectrum keeps rows together,
//   X[plane][y][kx], kx <= nx / 2,
// so the row kernels write and read whole rows; the column kernel reads one
// 16-byte element per row, and neighbouring columns run on one XCD, whose L2
// holds the lines they share.
#pragma once
#include "common.hpp"

namespace fvim {
namespace {

// Geometry of the length-2^LOGN transforms of one block: SEQ sequences, M
// threads each, thread (b, jj) holding the elements jj + m M, m < 4, of
// sequence b.
template <int LOGN>
struct Surf {
  static constexpr int N = 1 << LOGN;
  static constexpr int M = N / 4;
  static constexpr int NTH = M < 64 ? 64 : M;
  static constexpr int SEQ = NTH / M;
  static constexpr int LD = N + 1;
  static constexpr int TILE = SEQ * LD;              // elements of one LDS tile
  static constexpr int L0 = (LOGN & 1) ? 1 : 2;      // log2 of the first stage's radix
  static constexpr int NST = (LOGN - L0) / 2;        // radix-4 stages after it
  static constexpr int NW = NTH / 64;                // waves
  // Blocks of 1024 threads (length 4096) have 128 registers a thread: with the
  // twiddles (60) loaded beside the fields, or three fields beside a transform, 12
  // to 468 bytes a thread lay in scratch memory.  They load the twiddles after the
  // pointwise work that precedes a transform, the fields after a transform: us per
  // iteration of the contact at 4096^2 1840 -> 1262 and 4096 x 64 128 -> 84, of the
  // tangential contact 1765 -> 1479 and 66 -> 56.
  static constexpr bool TIGHT = NTH >= 1024;
};

// twiddles of the thread's butterfly in the stages after the first
template <int LOGN>
struct SurfTw {
  cpx<double> w[Surf<LOGN>::NST > 0 ? Surf<LOGN>::NST : 1][3];
};

template <int LOGN>
__device__ __forceinline__ void surf_load_tw(const cpx<double>* __restrict__ tw, int jj, SurfTw<LOGN>& t) {
  using S = Surf<LOGN>;
#pragma unroll
  for (int s = 0; s < S::NST; ++s) {
    const int ls = S::L0 + 2 * s;
    const int k = jj & ((1 << ls) - 1);
#pragma unroll
    for (int m = 1; m < 4; ++m) t.w[s][m - 1] = tw[m * k * (S::M >> ls)];
  }
}

// Stockham transform (radix 4, one radix-2 stage first when LOGN is odd) of
// the block's sequences, NPL of them per thread (PL planes in step): on entry
// v[q][m] is element jj + m M of the thread's sequence of plane q, on return
// the same element of its transform.  The first stage needs no exchange
// before it and the last none after it.  buf: NPL pairs of tiles, used in
// turn; a caller that has just read the tile `first` starts with the other.
template <int LOGN, bool INV, int NPL>
__device__ __forceinline__ void surf_fft(cpx<double> (&v)[NPL][4], cpx<double>* buf, int first, int b, int jj,
                                         const SurfTw<LOGN>& t) {
  using S = Surf<LOGN>;
  int cur = first;
#pragma unroll
  for (int q = 0; q < NPL; ++q) {
    cpx<double>* a = v[q];
    if constexpr (S::L0 == 2) {
      butterfly4<INV>(a);
      if constexpr (S::NST > 0) {
        cpx<double>* d = buf + (2 * q + cur) * S::TILE + b * S::LD + 4 * jj;
#pragma unroll
        for (int m = 0; m < 4; ++m) d[m] = a[m];
      }
    } else {
      const cpx<double> e0 = add(a[0], a[2]), o0 = sub(a[0], a[2]), e1 = add(a[1], a[3]), o1 = sub(a[1], a[3]);
      cpx<double>* d = buf + (2 * q + cur) * S::TILE + b * S::LD + 2 * jj;
      d[0] = e0;
      d[1] = o0;
      d[2 * S::M] = e1;
      d[2 * S::M + 1] = o1;
    }
  }
#pragma unroll
  for (int s = 0; s < S::NST; ++s) {
    __syncthreads();
    const int ls = S::L0 + 2 * s, ns = 1 << ls;
    const int k = jj & (ns - 1);
#pragma unroll
    for (int q = 0; q < NPL; ++q) {
      cpx<double>* a = v[q];
      const cpx<double>* src = buf + (2 * q + cur) * S::TILE + b * S::LD + jj;
      a[0] = src[0];
#pragma unroll
      for (int m = 1; m < 4; ++m) {
        const cpx<double> w = t.w[s][m - 1];
        a[m] = INV ? mulc(src[m * S::M], w) : mul(src[m * S::M], w);
      }
      butterfly4<INV>(a);
      if (s + 1 < S::NST) {
        cpx<double>* d = buf + (2 * q + (cur ^ 1)) * S::TILE + b * S::LD + ((jj >> ls) << (ls + 2)) + k;
#pragma unroll
        for (int m = 0; m < 4; ++m) d[m * ns] = a[m];
      }
    }
    cur ^= 1;
  }
}

// the tile surf_fft wrote last when it started with `first` (its caller may
// write the other one at once)
template <int LOGN>
__device__ constexpr int surf_last(int first) {
  using S = Surf<LOGN>;
  // NST tiles are written in turn from `first` (none when NST = 0 and the
  // first stage is the only one)
  return S::NST > 0 ? (first + S::NST - 1) & 1 : first ^ (S::L0 == 2 ? 1 : 0);
}

// Half spectra of the two real rows packed in the thread's sequence (v on
// return of the forward transform): row a of the pair goes to Xa[k], row b
// to Xb[k], k <= N / 2.  tile: an LDS tile no thread reads any more.
template <int LOGN>
__device__ __forceinline__ void surf_store_spectra(const cpx<double> (&v)[4], cpx<double>* tile, int b, int jj,
                                                   bool on, cpx<double>* __restrict__ Xa,
                                                   cpx<double>* __restrict__ Xb) {
  using S = Surf<LOGN>;
  cpx<double>* z = tile + b * S::LD;
#pragma unroll
  for (int m = 0; m < 4; ++m) z[jj + m * S::M] = v[m];
  __syncthreads();
  if (!on) return;
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int k = jj + u * S::M;
    if (u == 2 && jj != 0) break;
    const cpx<double> Z = z[k], Zc = z[(S::N - k) & (S::N - 1)];
    Xa[k] = mk(0.5 * (Z.x + Zc.x), 0.5 * (Z.y - Zc.y));
    Xb[k] = mk(0.5 * (Z.y + Zc.y), 0.5 * (Zc.x - Z.x));
  }
}

// The inverse of the above: the rows' half spectra packed into one complex
// sequence and transformed back; v[m] = (row a, row b) at x = jj + m M.
template <int LOGN>
__device__ __forceinline__ void surf_load_inverse(cpx<double> (&v)[1][4], cpx<double>* buf, int b, int jj, bool on,
                                                  const cpx<double>* __restrict__ Xa,
                                                  const cpx<double>* __restrict__ Xb, const SurfTw<LOGN>& t) {
  using S = Surf<LOGN>;
  cpx<double>* z = buf + b * S::LD;
  cpx<double> xa[3], xb[3];
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int k = jj + u * S::M;
    const bool ld = on && (u < 2 || jj == 0);
    xa[u] = ld ? Xa[k] : zero<double>();
    xb[u] = ld ? Xb[k] : zero<double>();
  }
#pragma unroll
  for (int u = 0; u < 3; ++u) {
    const int k = jj + u * S::M;
    if (k == 0 || u == 2) {
      if (jj == 0) z[k] = mk(xa[u].x, xb[u].x);
    } else {
      z[k] = mk(xa[u].x - xb[u].y, xa[u].y + xb[u].x);
      z[S::N - k] = mk(xa[u].x + xb[u].y, xb[u].x - xa[u].y);
    }
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 4; ++m) v[0][m] = z[jj + m * S::M];
  surf_fft<LOGN, true, 1>(v, buf, 1, b, jj, t);
}

// ---------------------------------------------------------------- reductions
// Sum over the wave, the same in every lane: DPP adds within each row of 16
// lanes, then the four rows by lane broadcasts (no LDS round trips, which made
// the totals of a one-wave block as long as its transform).
__device__ __forceinline__ double surf_wave_sum(double x) {
  x += dpp_move<DPP_ROW_DOWN + 1>(x);
  x += dpp_move<DPP_ROW_DOWN + 2>(x);
  x += dpp_move<DPP_ROW_DOWN + 4>(x);
  x += dpp_move<DPP_ROW_DOWN + 8>(x);
  return (lane_value(x, 0) + lane_value(x, 16)) + (lane_value(x, 32) + lane_value(x, 48));
}

// Sums of K quantities over the block's NW waves, in a fixed order; every
// thread gets them.  sh: K * NW doubles, free again on return.
template <int K, int NW>
__device__ __forceinline__ void surf_sums(const double (&v)[K], double* sh, double (&out)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) out[k] = surf_wave_sum(v[k]);
  if constexpr (NW > 1) {
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) sh[k * NW + (threadIdx.x >> 6)] = out[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double t = 0.0;
#pragma unroll NW > 8 ? 4 : NW         // (16 waves: not all K * NW values in registers)
      for (int i = 0; i < NW; ++i) t += sh[k * NW + i];
      out[k] = t;
    }
    __syncthreads();
  }
}

// Totals of K quantities over the nb blocks of an earlier kernel, formed by
// every block of the kernel that uses them (a launch of its own would cost
// more than the sums); f(i, s) adds block i's share to s[0 .. K).  Fixed order:
// every block gets the same bits (of one kernel: another wave count adds in another
// order).
template <int K, int NW, typename F>
__device__ __forceinline__ void surf_totals(int nb, double* sh, double (&out)[K], F f) {
  double s[K];
#pragma unroll
  for (int k = 0; k < K; ++k) s[k] = 0.0;
  for (int i = threadIdx.x; i < nb; i += NW * 64) f(i, s);
  surf_sums<K, NW>(s, sh, out);
}

// K block sums to part[k * ldp + blockIdx.x]
template <int K>
__device__ __forceinline__ void surf_put(double* __restrict__ part, int ldp, const double (&v)[K]) {
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) part[k * ldp + blockIdx.x] = v[k];
  }
}

#define FVIM_SURF_SWITCH(logn, CALL)       \
  switch (logn) {                          \
    case 2: CALL(2); break;                \
    case 3: CALL(3); break;                \
    case 4: CALL(4); break;                \
    case 5: CALL(5); break;                \
    case 6: CALL(6); break;                \
    case 7: CALL(7); break;                \
    case 8: CALL(8); break;                \
    case 9: CALL(9); break;                \
    case 10: CALL(10); break;              \
    case 11: CALL(11); break;              \
    case 12: CALL(12); break;              \
    default: return hipErrorInvalidValue;  \
  }

inline int surf_log2(int n) { return 31 - __builtin_clz((unsigned)n); }

}  // namespace
}  // namespace fvim
