// Products at any N beyond one workgroup's LDS (gfx950): each DCT-I of a pair of components
// as a chirp convolution on even sequences.
//
// With w_n = exp(-i pi n^2 / (2N)) (even, of period 2N) the DFT values of the even extension
// of z = a + i b (two components) are Y_k = w_k sum_{|n| <= N} u_n conj(w_{k-n}),
// u_n = z_|n| w_n with half weight at n = +-N.  The lags k - n reach 2N, so a circular
// length M >= 4N holds the filter conj(w_m), |m| <= 2N, unwrapped; input, filter and
// output are then all even in n, and so are their spectra: of M = M1 M2 points
// (n = M2 n1 + n2, k = k1 + M1 k2) only the columns n2 = 0..M2/2 and the rows
// k1 = 0..M1/2 are ever formed.  Column M2 - n2 is column n2 reversed, and row k1 of the
// two-step transform, G[k1][n2] = W_M^(n2 k1) F_n2[k1] with k1 signed, continues past
// n2 = M2/2 as G[k1][M2 - n2] = G[-k1][n2].  That is M/2 >= 2N points per pass where a
// convolution that is not even needs M >= 3N.
//
// M is the smallest of 4, 5, 6, 8 times a power of two that is >= 4N: M1 = R 2^A with
// R = 1, 3, 5, the factor R taken as R interleaved transforms of length 2^A and one
// butterfly at the output (short double-float convolutions leave R = 5 out, see blu_length).
//
//   columns:   even input (components, or the stencil of the first DCT's Y) x chirp,
//              FFT over n1, twiddle                                   -> G
//   rows:      FFT over n2, x filter spectrum, inverse FFT, inverse twiddle, in place
//   icolumns:  inverse FFT over k1, x chirp                           -> Y, or out
// The second DCT's columns form the stencil from Y where they read it, the first one's
// icolumns leave partial sums of c^_0, and the second one's add c^_0 (T_0 = 1: a constant)
// and write the components, so a product is these three launches twice.  The rows of G are
// kept a few elements longer than their M2/2 + 1, off a power of two: a column tile's
// accesses, one run per row, would otherwise all meet in the same cache sets.
//
// Traffic per pair and DCT in elements of N: read 1, write 2, read 2, write 2, read 2,
// write 1 and the tables, 10 against 15 for the three passes of a convolution of length 3N
// (whose power of two is also the coarser step).  Bound: at many pairs memory (64 uneven
// instances of 7.25 M values, double: rows 3.8 TB/s, columns 2.5 TB/s on their own bytes),
// at few the chain of a workgroup's loads, LDS stages and stores, six launches of 8 to 19
// us.  Measured per product in double, length-3N convolutions with separate stencil and
// unpacking launches before, this after: N = 100002 six components 122 -> 79 us, sixty
// (new only) 335; 64 uneven instances 775 -> 510; N = 999999 six components 1182 -> 386;
// N = 4999 six components 59 -> 50.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "birk_fft.h"
#include "birk_internal.h"
#include "birk_mid.h"

namespace birk {
namespace {

constexpr int kPPT = fast::kPPT;

// log2 of the 2^A W points per residue of a column tile: 8 NT = R 2^A W points, NT threads.
// Tiles of W = 8 columns (128-byte runs of G in double) where they fit 512 threads, no
// smaller than about 2048 points: wider tiles of short columns left fewer workgroups than
// CUs, narrower ones of long columns read partial cache lines (N = 999999 x 6 in double:
// 497 us a product with one column a tile, 417 with two).
__host__ __device__ constexpr int log_sub(int R, int A) {
  const int lo = R == 1 ? 11 : 9, hi = R == 1 ? 12 : R == 3 ? 10 : 9;
  const int s = A + 3 < lo ? lo : A + 3 > hi ? hi : A + 3;
  return s > A ? s : A;
}
// Row stride of G for columns 0..h.
__host__ __device__ constexpr int row_stride(int h) { return h + 8; }
constexpr int kLogRows = 11;   // points of a row tile (one row of 2^12 where rows are longer)

// W_M^t (t >= 0), or its conjugate, from the two-level table.
template <typename T>
__device__ __forceinline__ cplx<T> tw_at(const cplx<T>* __restrict__ hi, const cplx<T>* __restrict__ lo, int shift,
                                         int64_t t, bool conj) {
  const cplx<T> w = fast::cmul<T>(hi[t >> shift], lo[t & ((1 << shift) - 1)]);
  return conj ? fast::conjg<T>(w) : w;
}

template <typename T, int LOGL>
__device__ __forceinline__ void put(T* sm, int t, int n, cplx<T> v) {
  constexpr int LD = fast::padded_ld(1 << LOGL);
  sm[2 * t * LD + fast::pad(n)] = v.x;
  sm[(2 * t + 1) * LD + fast::pad(n)] = v.y;
}
template <typename T, int LOGL>
__device__ __forceinline__ cplx<T> get(const T* sm, int t, int n) {
  constexpr int LD = fast::padded_ld(1 << LOGL);
  return fast::mk<T>(sm[2 * t * LD + fast::pad(n)], sm[(2 * t + 1) * LD + fast::pad(n)]);
}

// X_j = sum_s g_s exp(-2 pi i s j / R) in place.  Double-floats form each product once (R = 5 from
// cos(2 pi / 5), cos(4 pi / 5) = -1/4 +- sqrt(5)/4); the others fuse them with the sums.
template <typename T, int R>
__device__ __forceinline__ void dft_odd(cplx<T> (&g)[R]) {
  auto add = [](cplx<T> a, cplx<T> b) { return fast::mk<T>(a.x + b.x, a.y + b.y); };
  auto sub = [](cplx<T> a, cplx<T> b) { return fast::mk<T>(a.x - b.x, a.y - b.y); };
  constexpr bool kFused = std::is_floating_point<T>::value;
  if constexpr (R == 3) {
    const T s = T(0.86602540378443864676);
    const cplx<T> t = add(g[1], g[2]), u = sub(g[1], g[2]);
    const cplx<T> m = fast::mk<T>(g[0].x - pow2_times(0.5f, t.x), g[0].y - pow2_times(0.5f, t.y));
    g[0] = add(g[0], t);
    if constexpr (kFused) {
      g[1] = fast::mk<T>(m.x + s * u.y, m.y - s * u.x);
      g[2] = fast::mk<T>(m.x - s * u.y, m.y + s * u.x);
    } else {
      const cplx<T> su = fast::mk<T>(s * u.x, s * u.y);
      g[1] = fast::mk<T>(m.x + su.y, m.y - su.x);
      g[2] = fast::mk<T>(m.x - su.y, m.y + su.x);
    }
  } else if constexpr (R == 5) {
    const T s1 = T(0.95105651629515357212), s2 = T(0.58778525229247312917);
    const cplx<T> t1 = add(g[1], g[4]), t2 = add(g[2], g[3]), u1 = sub(g[1], g[4]), u2 = sub(g[2], g[3]);
    cplx<T> m1, m2;
    if constexpr (kFused) {
      const T c1 = T(0.30901699437494742410), c2 = T(-0.80901699437494742410);
      m1 = fast::mk<T>(g[0].x + c1 * t1.x + c2 * t2.x, g[0].y + c1 * t1.y + c2 * t2.y);
      m2 = fast::mk<T>(g[0].x + c2 * t1.x + c1 * t2.x, g[0].y + c2 * t1.y + c1 * t2.y);
    } else {
      const T q = T(0.55901699437494742410);   // sqrt(5)/4
      const cplx<T> t = add(t1, t2), v = sub(t1, t2);
      const cplx<T> m = fast::mk<T>(g[0].x - pow2_times(0.25f, t.x), g[0].y - pow2_times(0.25f, t.y));
      const cplx<T> qv = fast::mk<T>(q * v.x, q * v.y);
      m1 = add(m, qv);
      m2 = sub(m, qv);
    }
    const cplx<T> n1 = fast::mk<T>(s1 * u1.x + s2 * u2.x, s1 * u1.y + s2 * u2.y);
    const cplx<T> n2 = fast::mk<T>(s2 * u1.x - s1 * u2.x, s2 * u1.y - s1 * u2.y);
    g[0] = add(g[0], add(t1, t2));
    g[1] = fast::mk<T>(m1.x + n1.y, m1.y - n1.x);
    g[4] = fast::mk<T>(m1.x - n1.y, m1.y + n1.x);
    g[2] = fast::mk<T>(m2.x + n2.y, m2.y - n2.x);
    g[3] = fast::mk<T>(m2.x - n2.y, m2.y + n2.x);
  }
}

// Workgroups are dealt to the 8 XCDs in turn: give each a contiguous range of the tile
// list, so that neighbouring tiles, which share cache lines, meet in one L2.
__device__ __forceinline__ int2 xcd_tile(const int2* __restrict__ tiles) {
  const int total = (int)gridDim.x, lid = (int)blockIdx.x;
  const int xcd = lid & 7, q = total >> 3, r = total & 7;
  return tiles[xcd * q + min(xcd, r) + (lid >> 3)];
}

// What the columns pass transforms.
enum { kSrcV = 0, kSrcVT = 1, kSrcFwd = 2, kSrcTr = 3, kSrcFilter = 4 };

// The tile's columns n2 = c0 + w, w < W, into LDS: residue s = n1 mod R, position n1 / R.
// All loads of a batch come from valid addresses (entries outside the input read |n| = 0)
// and none waits for another: under a branch per entry each would be waited for alone.
template <typename T, int R, int A>
__device__ __forceinline__ void load_cols(const PairDesc& d, const T* __restrict__ x, const cplx<T>* __restrict__ Y,
                                          int src, int c0, int nw, T* sm) {
  constexpr int pi = prec_index<T>();
  constexpr int LOGW = log_sub(R, A) - A, W = 1 << LOGW, NT = (R << log_sub(R, A)) / kPPT;
  const cplx<T>* chirp = (const cplx<T>*)d.chirp[pi];
  const int N = (int)d.N, M = (int)d.M, b = d.logM2;
  auto where = [&](int i, int& w, int& n1) {
    const int e = (int)threadIdx.x + i * NT;
    w = e & (W - 1);
    n1 = e >> LOGW;
  };
  // |n| of entry i, or -1 outside the columns and the input
  auto entry = [&](int i) {
    int w, n1;
    where(i, w, n1);
    const int n = (n1 << b) + c0 + w, k = min(n, M - n);
    return (w < nw && k <= N) ? k : -1;
  };
  auto store = [&](int i, cplx<T> v) {
    int w, n1;
    where(i, w, n1);
    put<T, A>(sm, w * R + n1 % R, n1 / R, v);
  };
  // x chirp, half weight at n = +-N (both are in the sum), zero outside
  auto finish = [&](int k, cplx<T> v, cplx<T> c) {
    const float h = k == N ? 0.5f : 1.0f;
    const cplx<T> r = fast::cmul<T>(fast::mk<T>(pow2_times(h, v.x), pow2_times(h, v.y)), c);
    return k >= 0 ? r : fast::mk<T>(T(0), T(0));
  };
  if (src <= kSrcVT) {
    const T* xa = x + d.src;
    const T* xb = xa + (d.has2 ? d.Nn : 0);   // a lone component is read twice
    T va[kPPT], vb[kPPT];
    cplx<T> c[kPPT];
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int k = max(entry(i), 0);
      va[i] = xa[k];
      vb[i] = xb[k];
      c[i] = chirp[k];
    }
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int k = entry(i);
      // E^{-1} of the transpose: ends doubled
      const float e = (src == kSrcVT && (k == 0 || k == N)) ? 2.0f : 1.0f;
      store(i, finish(k, fast::mk<T>(pow2_times(e, va[i]), d.has2 ? pow2_times(e, vb[i]) : T(0)), c[i]));
    }
  } else if (src != kSrcFilter) {
    constexpr int HB = kPPT / 2;
    const bool fwd = src == kSrcFwd;
    const T invN = T(1) / T(N), inv4N1 = T(1) / T(4 * N + 4), inv2N1 = T(1) / T(2 * N + 2);
    const cplx<T> Y0 = Y[0];
#pragma unroll
    for (int i0 = 0; i0 < kPPT; i0 += HB) {
      cplx<T> ym[HB], yp[HB], c[HB];
#pragma unroll
      for (int i = 0; i < HB; ++i) {
        const int k = max(entry(i0 + i), 0);
        ym[i] = Y[max(k - 1, 0)];
        yp[i] = Y[min(k + 1, N)];
        c[i] = chirp[k];
      }
#pragma unroll
      for (int i = 0; i < HB; ++i) {
        const int k = entry(i0 + i), kc = max(k, 0);
        cplx<T> v;
        if (fwd) {
          v = kc > 0 ? mid_fwd<T>(kc, N, ym[i], yp[i], invN, inv4N1) : fast::mk<T>(T(0), T(0));
        } else {
          v = mid_tr<T>(kc, N, Y0, ym[i], yp[i], inv2N1);
        }
        store(i0 + i, finish(k, v, c[i]));
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      int w, n1;
      where(i, w, n1);
      const int n = (n1 << b) + c0 + w, k = min(n, M - n);
      const bool in = w < nw && k <= 2 * N;
      const cplx<T> c = chirp[in ? (k <= N ? k : 2 * N - k) : 0];
      store(i, in ? fast::conjg<T>(c) : fast::mk<T>(T(0), T(0)));
    }
  }
}

// Twiddles are stepped in double (a tenth of the operations of a double-float product) and
// rounded to T where they are used; the powers that join the residues are formed in T, or in
// double for double-floats.
template <typename T>
using Pow = std::conditional_t<std::is_floating_point<T>::value, T, double>;
template <typename T, typename C>
__device__ __forceinline__ cplx<T> to(C a) {
  return fast::mk<T>((T)a.x, (T)a.y);
}

// The R outputs k + j 2^A of item (w, k): residues x W_M1^(s k), one R-point butterfly.
template <typename T, int R, int A>
__device__ __forceinline__ void join_residues(const T* sm, int w, int k, cplx<Pow<T>> q, cplx<T> (&g)[R]) {
  cplx<Pow<T>> p = q;
#pragma unroll
  for (int s = 0; s < R; ++s) {
    g[s] = get<T, A>(sm, w * R + s, k);
    if (s > 0) {
      g[s] = fast::cmul<T>(g[s], to<T>(p));
      if (s + 1 < R) p = fast::cmul<Pow<T>>(p, q);
    }
  }
  if constexpr (R > 1) dft_odd<T, R>(g);
}

// Columns pass of one tile.  Outputs k1 > M1/2 are kept with k1 - M1 in their twiddle.
template <typename T, int R, int A>
__device__ __forceinline__ void cols_body(const T* __restrict__ x, const cplx<T>* __restrict__ Y, cplx<T>* __restrict__ G, const PairDesc& d, int ty, int src,
                                          const cplx<T>* __restrict__ tw, T* sm) {
  constexpr int LOGW = log_sub(R, A) - A, W = 1 << LOGW, NT = (R << log_sub(R, A)) / kPPT;
  constexpr int M1 = R << A, NI = ((1 << log_sub(R, A)) + NT - 1) / NT, S = NT >> LOGW;
  const int t = (int)threadIdx.x;
  const bool on = t < NT;
  const int b = d.logM2, h = 1 << (b - 1);
  const bool last = ty * W >= h;   // the tile of column M2/2
  const int c0 = last ? h : ty * W;
  const int nw = last ? 1 : min(W, h - c0);
  const int w = t & (W - 1), k0 = t >> LOGW, n2 = c0 + w;
  // phase = W_M^(n2 k), stepped from item to item; stp = W_M^(n2 2^A); wrap = W_M2^(-n2)
  // (k1 - M1 for k1); q = W_M1^k
  using P = double;
  const cplx<P>* thi = (const cplx<P>*)d.thi[0];
  const cplx<P>* tlo = (const cplx<P>*)d.tlo[0];
  const int sh = d.tw_shift;
  cplx<P> phase, dphase, stp, wrap, q, dq;
  if (on) {
    load_cols<T, R, A>(d, x, Y, src, c0, nw, sm);
    phase = tw_at<P>(thi, tlo, sh, (int64_t)n2 * k0, false);
    dphase = tw_at<P>(thi, tlo, sh, (int64_t)n2 * S, false);
    wrap = tw_at<P>(thi, tlo, sh, (int64_t)n2 * M1, true);
    if constexpr (R > 1) {
      stp = tw_at<P>(thi, tlo, sh, (int64_t)n2 << A, false);
      q = tw_at<P>(thi, tlo, sh, (int64_t)k0 << b, false);
      dq = tw_at<P>(thi, tlo, sh, (int64_t)S << b, false);
    }
  }
  __syncthreads();
  fast::fft_ct<T, A, R * W, true>(sm, tw);
  if (!on) return;
  auto store = [&](int k1, cplx<T> v) { G[k1 * row_stride(h) + n2] = v; };
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int k = k0 + it * S;
    if (k < (1 << A) && w < nw) {
      cplx<T> g[R];
      cplx<Pow<T>> qt = to<Pow<T>>(fast::mk<P>(0.0, 0.0));
      if constexpr (R > 1) qt = to<Pow<T>>(q);
      join_residues<T, R, A>(sm, w, k, qt, g);
      cplx<P> p = phase;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int k1 = k + (j << A);
        const cplx<P> f = 2 * k1 > M1 ? fast::cmul<P>(p, wrap) : p;
        store(k1, fast::cmul<T>(g[j], to<T>(f)));
        if (j + 1 < R) p = fast::cmul<P>(p, stp);
      }
    }
    phase = fast::cmul<P>(phase, dphase);
    if constexpr (R > 1) q = fast::cmul<P>(q, dq);
  }
}

// Inverse columns pass of one tile: Y_k for the outputs n = k or M - k of its columns
// (columns 0 and M2/2 hold both: n <= N only).  FIN: the components, with c^_0 added or the
// transpose's scale; else Y, and the tile's part of the c^_0 sums in part[2 ty].
template <typename T, int R, int A, bool FIN>
__device__ __forceinline__ void icols_body(const cplx<T>* __restrict__ G,
                                           cplx<T>* __restrict__ Y, T* __restrict__ out, double* __restrict__ part,
                                           const PairDesc& d, int ty, int trans, const cplx<T>* __restrict__ tw, T* sm,
                                           double* red) {
  constexpr int pi = prec_index<T>();
  constexpr int LOGW = log_sub(R, A) - A, W = 1 << LOGW, NT = (R << log_sub(R, A)) / kPPT;
  constexpr int NI = ((1 << log_sub(R, A)) + NT - 1) / NT, S = NT >> LOGW;
  const int t = (int)threadIdx.x;
  const bool on = t < NT;
  const int N = (int)d.N, M = (int)d.M, b = d.logM2, h = 1 << (b - 1);
  const bool last = ty * W >= h;
  const int c0 = last ? h : ty * W;
  const int nw = last ? 1 : min(W, h - c0);
  const int w = t & (W - 1), k0 = t >> LOGW, n2 = c0 + w;
  const cplx<T>* chirp = (const cplx<T>*)d.chirp[pi];
  using P = double;
  const cplx<P>* thi = (const cplx<P>*)d.thi[0];
  const cplx<P>* tlo = (const cplx<P>*)d.tlo[0];
  const int sh = d.tw_shift;
  cplx<P> q, dq;
  auto index = [&](int n1) {   // output k of position n1, or -1
    const int n = (n1 << b) + n2;
    if (w >= nw) return -1;
    if (n <= N) return n;
    return (M - n <= N && n2 != 0 && n2 != h) ? M - n : -1;
  };
  cplx<T> v[kPPT], cv[R * NI];
  if (on) {
    // lanes beyond the tile's columns read its last one; their outputs are not stored
    const cplx<T>* g = G + c0 + min(w, nw - 1);
#pragma unroll
    for (int i = 0; i < kPPT; ++i) v[i] = g[(k0 + i * S) * row_stride(h)];   // k1 = (t + i NT) >> LOGW
#pragma unroll
    for (int it = 0; it < NI; ++it)
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int k = k0 + it * S;
        cv[it * R + j] = chirp[k < (1 << A) ? max(index(k + (j << A)), 0) : 0];
      }
    if constexpr (R > 1) {
      q = tw_at<P>(thi, tlo, sh, (int64_t)k0 << b, false);
      dq = tw_at<P>(thi, tlo, sh, (int64_t)S << b, false);
    }
  }
  if (FIN && !trans && t < 64) {
    // c^_0 of both components from the tiles' sums, in an order fixed by the pair alone
    const int np = ((h + W - 1) >> LOGW) + 1;
    double s0 = 0.0, s1 = 0.0;
    for (int p = t; p < np; p += 64) {
      s0 += part[2 * p];
      s1 += part[2 * p + 1];
    }
    s0 = wave_sum_last(s0);
    s1 = wave_sum_last(s1);
    if (t == 63) {
      red[0] = s0 / (double)N;
      red[1] = s1 / (double)N;
    }
  }
  if (on) {
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int k1 = k0 + i * S;
      put<T, A>(sm, w * R + k1 % R, k1 / R, fast::conjg<T>(v[i]));
    }
  }
  __syncthreads();
  fast::fft_ct<T, A, R * W, true>(sm, tw);
  double s0 = 0.0, s1 = 0.0;
  T ca = T(0), cb = T(0), sc = T(0.5);
  if (FIN) {
    if (trans) {
      sc = T(1) / T(N);
    } else {
      ca = (T)red[0];
      cb = (T)red[1];
    }
  }
  if (on) {
    T* o = out + (FIN ? d.src : 0);
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = k0 + it * S;
      if (k < (1 << A) && w < nw) {
        cplx<T> g[R];
        cplx<Pow<T>> qt = to<Pow<T>>(fast::mk<P>(0.0, 0.0));
        if constexpr (R > 1) qt = to<Pow<T>>(q);
        join_residues<T, R, A>(sm, w, k, qt, g);
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const int kk = index(k + (j << A));
          if (kk < 0) continue;
          const cplx<T> y = fast::cmul<T>(fast::conjg<T>(g[j]), cv[it * R + j]);
          if constexpr (FIN) {
            const T f = (trans && (kk == 0 || kk == N)) ? T(0.5) * sc : sc;
            o[kk] = f * y.x + ca;
            if (d.has2) o[d.Nn + kk] = f * y.y + cb;
          } else {
            Y[kk] = y;
            if (!trans) {
              const double c = c0_weight(kk, N);
              s0 += c * (double)y.x;
              s1 += c * (double)y.y;
            }
          }
        }
      }
      if constexpr (R > 1) q = fast::cmul<P>(q, dq);
    }
  }
  if (!FIN && !trans) {
    s0 = wave_sum_last(s0);
    s1 = wave_sum_last(s1);
    if ((t & 63) == 63) {
      red[2 * (t >> 6)] = s0;
      red[2 * (t >> 6) + 1] = s1;
    }
    __syncthreads();
    if (t == 0) {
      double a = 0.0, c = 0.0;
      for (int i = 0; i < NT / 64; ++i) {
        a += red[2 * i];
        c += red[2 * i + 1];
      }
      part[2 * ty] = a;
      part[2 * ty + 1] = c;
    }
  }
}

// Rows pass of one tile: rows k1 = r0 + w (k1 <= M1/2) with their continuation from row
// -k1.  SPEC: the filter's own transform, spectrum / M to `spec` in the order the product
// reads it.
template <typename T, int B, bool SPEC>
__device__ __forceinline__ void rows_body(cplx<T>* __restrict__ G, cplx<T>* __restrict__ spec,
                                          const PairDesc& d, int ty, const cplx<T>* __restrict__ tw, T* sm) {
  constexpr int pi = prec_index<T>();
  constexpr int LOGP = B > kLogRows ? B : kLogRows;
  constexpr int M2 = 1 << B, h = M2 / 2, hs = row_stride(h), W = 1 << (LOGP - B), NT = (1 << LOGP) / kPPT;
  const int t = (int)threadIdx.x;
  const bool on = t < NT;
  const int M1 = (int)d.M >> B, h1 = M1 / 2, r0 = ty * W;
  const cplx<T>* filt = (const cplx<T>*)d.filt[pi];
  cplx<T> v[kPPT], fv[kPPT];
  fast::StageTw<T, B> st;
  if (on) {
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int e = t + i * NT;
      // rows past M1/2 read row M1/2; they are not stored
      const int k1 = min(r0 + (e >> B), h1), n2 = e & (M2 - 1);
      const int km = (k1 == 0 || k1 == h1) ? k1 : M1 - k1;
      v[i] = G[n2 <= h ? k1 * hs + n2 : km * hs + (M2 - n2)];
      if constexpr (SPEC) fv[i] = v[i];
      else fv[i] = filt[(int64_t)k1 * M2 + n2];
    }
    st.load(tw);
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int e = t + i * NT;
      const int w = e >> B, n2 = e & (M2 - 1);
      // row M1/2 is its own mirror with k1 and k1 - M1 apart by W_M^(n2 M1)
      if (min(r0 + w, h1) == h1 && n2 > h) v[i] = fast::cmul<T>(v[i], fast::conjg<T>(tw[(M2 - n2) << (kLdsMaxLog - B)]));
      put<T, B>(sm, w, n2, v[i]);
    }
  }
  __syncthreads();
  fast::fft_ct<T, B, W, true>(sm, st);
  if constexpr (SPEC) {
    if (!on) return;
    const double inv = 1.0 / (double)d.M;
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int e = t + i * NT;
      const int w = e >> B, n2 = e & (M2 - 1);
      const cplx<T> g = get<T, B>(sm, w, n2);
      if (r0 + w <= h1) spec[(int64_t)(r0 + w) * M2 + n2] = fast::mk<T>(g.x * T(inv), g.y * T(inv));
    }
    return;
  }
  // twiddles W_M^(mu k1) of the outputs, mu = -n2 up to M2/2 and M2 - n2 above: a thread's
  // outputs step through k1 (rows of at most NT points) or through n2 (longer rows: a base
  // for each half)
  using P = double;
  const cplx<P>* thi = (const cplx<P>*)d.thi[0];
  const cplx<P>* tlo = (const cplx<P>*)d.tlo[0];
  const int sh = d.tw_shift;
  auto twid = [&](int64_t mu, int64_t k1) {
    const int64_t p = mu * k1;
    return tw_at<P>(thi, tlo, sh, p < 0 ? -p : p, p < 0);
  };
  if (on) {
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int e = t + i * NT;
      const int w = e >> B, n2 = e & (M2 - 1);
      put<T, B>(sm, w, n2, fast::conjg<T>(fast::cmul<T>(get<T, B>(sm, w, n2), fv[i])));
    }
  }
  __syncthreads();
  fast::fft_ct<T, B, W, true>(sm, st);
  if (!on) return;
  // row k1 up to M2/2; row -k1 from there on, and its column 0
  auto store = [&](int k1, int n2, cplx<P> f) {
    const cplx<T> z = fast::conjg<T>(get<T, B>(sm, k1 - r0, n2));
    const cplx<T> r = fast::cmul<T>(z, to<T>(f));
    const bool twin = k1 > 0 && k1 < h1;
    if (n2 <= h) G[k1 * hs + n2] = r;
    if (!twin) return;
    if (n2 > h) G[(M1 - k1) * hs + (M2 - n2)] = r;
    else if (n2 == h) G[(M1 - k1) * hs + h] = fast::cmul<T>(z, to<T>(fast::conjg<P>(f)));
    else if (n2 == 0) G[(M1 - k1) * hs] = r;   // no twiddle
  };
  if constexpr (M2 <= NT) {
    constexpr int S = NT / M2;   // rows between a thread's elements
    const int n2 = t & (M2 - 1), w0 = t >> B;
    const int mu = n2 <= h ? -n2 : M2 - n2;
    cplx<P> f = twid(mu, r0 + w0);
    const cplx<P> df = twid(mu, S);
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      const int k1 = r0 + w0 + i * S;
      if (k1 <= h1) store(k1, n2, f);
      f = fast::cmul<P>(f, df);
    }
  } else {
    constexpr int EPR = M2 / NT;   // elements of a thread in one row
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int k1 = r0 + w;
      if (k1 > h1) break;
      cplx<P> lo = twid(-t, k1), up = twid(h - t, k1);
      const cplx<P> df = twid(-NT, k1);
#pragma unroll
      for (int i = 0; i < EPR / 2; ++i) {
        store(k1, t + i * NT, lo);
        const int n2 = t + i * NT + h;
        store(k1, n2, n2 == h ? fast::conjg<P>(up) : up);
        if (i + 1 < EPR / 2) {
          lo = fast::cmul<P>(lo, df);
          up = fast::cmul<P>(up, df);
        }
      }
    }
  }
}

#define BLU_COL_SWITCH(d, CALL)                                   \
  switch ((d).R * 16 + (d).logM1) {                               \
    case 1 * 16 + 7: { constexpr int RR = 1, AA = 7; CALL; } break; \
    case 1 * 16 + 8: { constexpr int RR = 1, AA = 8; CALL; } break; \
    case 1 * 16 + 9: { constexpr int RR = 1, AA = 9; CALL; } break; \
    case 1 * 16 + 10: { constexpr int RR = 1, AA = 10; CALL; } break;\
    case 1 * 16 + 11: { constexpr int RR = 1, AA = 11; CALL; } break;\
    case 1 * 16 + 12: { constexpr int RR = 1, AA = 12; CALL; } break;\
    case 3 * 16 + 5: { constexpr int RR = 3, AA = 5; CALL; } break; \
    case 3 * 16 + 6: { constexpr int RR = 3, AA = 6; CALL; } break; \
    case 3 * 16 + 7: { constexpr int RR = 3, AA = 7; CALL; } break; \
    case 3 * 16 + 8: { constexpr int RR = 3, AA = 8; CALL; } break; \
    case 3 * 16 + 9: { constexpr int RR = 3, AA = 9; CALL; } break; \
    case 3 * 16 + 10: { constexpr int RR = 3, AA = 10; CALL; } break;\
    case 5 * 16 + 4: { constexpr int RR = 5, AA = 4; CALL; } break; \
    case 5 * 16 + 5: { constexpr int RR = 5, AA = 5; CALL; } break; \
    case 5 * 16 + 6: { constexpr int RR = 5, AA = 6; CALL; } break; \
    case 5 * 16 + 7: { constexpr int RR = 5, AA = 7; CALL; } break; \
    case 5 * 16 + 8: { constexpr int RR = 5, AA = 8; CALL; } break; \
    case 5 * 16 + 9: { constexpr int RR = 5, AA = 9; CALL; } break; \
    default: break;                                                 \
  }

template <typename T>
__global__ __launch_bounds__(512) void k_blu_cols(const T* __restrict__ x, const cplx<T>* __restrict__ Y,
                                                 cplx<T>* __restrict__ G,
                                                 const PairDesc* __restrict__ pd, const int2* __restrict__ tiles,
                                                 const cplx<T>* __restrict__ tw, int src) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int2 tile = xcd_tile(tiles);
  const PairDesc& d = pd[tile.x];
  BLU_COL_SWITCH(d, (cols_body<T, RR, AA>(x, Y + d.work, G + d.work, d, tile.y, src, tw, sm)))
}

template <typename T, bool FIN>
__global__ __launch_bounds__(512) void k_blu_icols(const cplx<T>* __restrict__ G,
                                                  cplx<T>* __restrict__ Y, T* __restrict__ out,
                                                  const PairDesc* __restrict__ pd, const int2* __restrict__ tiles,
                                                  const cplx<T>* __restrict__ tw, int trans) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[16];
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int2 tile = xcd_tile(tiles);
  const PairDesc& d = pd[tile.x];
  // the c^_0 sums follow the N + 1 values of Y in the pair's slot
  cplx<T>* Yp = Y + d.work;
  double* part = reinterpret_cast<double*>(Yp + d.Nn);
  BLU_COL_SWITCH(d, (icols_body<T, RR, AA, FIN>(G + d.work, Yp, out, part, d, tile.y, trans, tw, sm, red)))
}
#undef BLU_COL_SWITCH

template <typename T, bool SPEC>
__global__ __launch_bounds__(512) void k_blu_rows(cplx<T>* __restrict__ G,
                                                 const PairDesc* __restrict__ pd, const int2* __restrict__ tiles,
                                                 const cplx<T>* __restrict__ tw) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int2 tile = xcd_tile(tiles);
  const PairDesc& d = pd[tile.x];
  cplx<T>* g = G + d.work;
  cplx<T>* spec = SPEC ? (cplx<T>*)d.filt[prec_index<T>()] : nullptr;
  switch (d.logM2) {
    case 6: rows_body<T, 6, SPEC>(g, spec, d, tile.y, tw, sm); break;
    case 7: rows_body<T, 7, SPEC>(g, spec, d, tile.y, tw, sm); break;
    case 8: rows_body<T, 8, SPEC>(g, spec, d, tile.y, tw, sm); break;
    case 9: rows_body<T, 9, SPEC>(g, spec, d, tile.y, tw, sm); break;
    case 10: rows_body<T, 10, SPEC>(g, spec, d, tile.y, tw, sm); break;
    case 11: rows_body<T, 11, SPEC>(g, spec, d, tile.y, tw, sm); break;
    case 12: rows_body<T, 12, SPEC>(g, spec, d, tile.y, tw, sm); break;
    default: break;
  }
}

// dst = src in another precision
template <typename T>
__global__ void k_convert(const cplx<double>* __restrict__ src, cplx<T>* __restrict__ dst, int64_t n) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m < n) dst[m] = fast::mk<T>((T)src[m].x, (T)src[m].y);
}

// LDS reals of a column tile (2^A R points a column) and of a row tile.
constexpr int lds_cols(int R, int A) { return 2 * R * (1 << (log_sub(R, A) - A)) * fast::padded_ld(1 << A); }
constexpr int lds_rows(int B) { return 2 * (1 << (std::max(B, kLogRows) - B)) * fast::padded_ld(1 << B); }
// The most of them over the lengths that the kernels cover.
constexpr int lds_cols_most() {
  int m = 0;
  for (int A = 7; A <= kLdsMaxLog; ++A) m = std::max(m, lds_cols(1, A));
  for (int A = 5; A <= kLdsMaxLog - 2; ++A) m = std::max(m, lds_cols(3, A));
  for (int A = 4; A <= kLdsMaxLog - 3; ++A) m = std::max(m, lds_cols(5, A));
  return m;
}
constexpr int lds_rows_most() {
  int m = 0;
  for (int B = 6; B <= kLdsMaxLog; ++B) m = std::max(m, lds_rows(B));
  return m;
}

}  // namespace

// Length of a pair: M = R 2^m, M1 = R 2^A, M2 = 2^(m - A).  Double-float plans leave R = 5 out up
// to N = 2^14: their five-point butterflies cost more there than the longer M (N = 2499, one,
// 32 and 128 instances of six components: 128, 185 and 385 us with R = 5, 121, 134 and 370 with
// R = 3; N = 9999: one 140 against 116, eight 130 against 138, 32 372 against 335; but N = 39999,
// four 197 against 237, and N = 299999, two 744 against 838).
void blu_length(PairDesc& d, birk_precision prec) {
  const int64_t need = 4 * d.N;
  int64_t best = 0;
  for (int R : {1, 3, 5}) {
    if (R == 5 && prec == BIRK_DF32 && d.N <= (1 << 14)) continue;
    int m = 0;
    while (((int64_t)R << m) < need) ++m;
    if (best == 0 || ((int64_t)R << m) < best) {
      best = (int64_t)R << m;
      d.R = R;
      d.logM = m;
    }
  }
  d.M = best;
}

// Nominal log2 of M1 = 2^A, 3 2^A = 3/4 2^(A + 2), 5 2^A = 5/8 2^(A + 3).
static int nominal(int R) { return R == 1 ? 0 : R == 3 ? 2 : 3; }

bool blu_split_ok(const PairDesc& d, int x) {
  const int A = x - nominal(d.R), B = d.logM - A;
  return x >= 7 && x <= kLdsMaxLog && B >= 6 && B <= kLdsMaxLog;
}

void blu_set_split(PairDesc& d, int x) {
  d.logM1 = x - nominal(d.R);
  d.logM2 = d.logM - d.logM1;
}

int blu_split(const PairDesc& d) { return d.logM1 + nominal(d.R); }

// 2^8 columns and rows of up to 2^11 points while they last (measured in double, M = 2^19,
// six and sixty components: 90.0 and 393 us at x = 8, 92.8 and 409 at 9, 91.5 and 423 at 7;
// M = 2^22: 411 at x = 10, 422 at 11).
int blu_default_split(const PairDesc& d) {
  const int t = d.logM + nominal(d.R);
  const int x = std::max(t - kLdsMaxLog, std::min(10, std::max(8, t - 11)));
  return std::max(7, std::min(x, t - 6));
}

// Tile lists and launch sizes of a set, and its descriptors.
hipError_t blu_lists(birk_plan* p, PairSet& ps) {
  std::vector<int2> tc, tr;
  ps.thr_c = ps.thr_r = 64;
  ps.lds_c = ps.lds_r = 0;
  for (int q = 0; q < (int)ps.host.size(); ++q) {
    const PairDesc& d = ps.host[q];
    const int ls = log_sub(d.R, d.logM1), W = 1 << (ls - d.logM1), h = 1 << (d.logM2 - 1);
    for (int b = 0; b <= (h + W - 1) / W; ++b) tc.push_back(make_int2(q, b));
    const int lp = std::max(d.logM2, kLogRows), Wr = 1 << (lp - d.logM2);
    const int nrows = (int)(d.M >> d.logM2) / 2 + 1;
    for (int b = 0; b < (nrows + Wr - 1) / Wr; ++b) tr.push_back(make_int2(q, b));
    ps.thr_c = std::max(ps.thr_c, (d.R << ls) / kPPT);
    ps.thr_r = std::max(ps.thr_r, (1 << lp) / kPPT);
    ps.lds_c = std::max(ps.lds_c, lds_cols(d.R, d.logM1));
    ps.lds_r = std::max(ps.lds_r, lds_rows(d.logM2));
  }
  ps.n_c4 = (int)tc.size();
  ps.n_r4 = (int)tr.size();
  void* x = nullptr;
  hipError_t e = upload_raw(p, ps.host.data(), ps.host.size() * sizeof(PairDesc), &x);
  ps.dev = (PairDesc*)x;
  if (e == hipSuccess) e = upload_raw(p, tc.data(), tc.size() * sizeof(int2), &x);
  ps.tiles_c4 = (int2*)x;
  if (e == hipSuccess) e = upload_raw(p, tr.data(), tr.size() * sizeof(int2), &x);
  ps.tiles_r4 = (int2*)x;
  return e;
}

void blu_free_lists(birk_plan* p, PairSet& ps) {
  for (void* x : {(void*)ps.dev, (void*)ps.tiles_c4, (void*)ps.tiles_r4}) {
    const auto it = std::find(p->allocs.begin(), p->allocs.end(), x);
    if (x && it != p->allocs.end()) {
      p->allocs.erase(it);
      (void)hipFree(x);
    }
  }
  ps.dev = nullptr;
  ps.tiles_c4 = ps.tiles_r4 = nullptr;
}

// Filter spectra of the set's pairs (one per distinct length N; each pair's work slots are
// used) in its split's row order, double first, then the plan's other precision.  Blocks.
hipError_t blu_filters(birk_plan* p, const PairSet& ps, hipStream_t s) {
  if (ps.host.empty()) return hipSuccess;
  cplx<double>* G = (cplx<double>*)p->work[0];
  cplx<double>* Y = (cplx<double>*)p->work[1];
  const cplx<double>* tw = (const cplx<double>*)p->lds_tw[0];
  lds_limit(k_blu_cols<double>, lds_cols_most() * (int)sizeof(double));
  lds_limit(k_blu_rows<double, true>, lds_rows_most() * (int)sizeof(double));
  hipLaunchKernelGGL(k_blu_cols<double>, dim3(ps.n_c4), dim3(ps.thr_c), ps.lds_c * sizeof(double), s, nullptr, Y, G,
                     ps.dev, ps.tiles_c4, tw, (int)kSrcFilter);
  hipLaunchKernelGGL((k_blu_rows<double, true>), dim3(ps.n_r4), dim3(ps.thr_r), ps.lds_r * sizeof(double), s, G,
                     ps.dev, ps.tiles_r4, tw);
  for (const PairDesc& d : ps.host) {
    const int64_t n = ((d.M >> d.logM2) / 2 + 1) << d.logM2;
    const dim3 grid((unsigned)((n + 255) / 256));
    const cplx<double>* src = (const cplx<double>*)d.filt[0];
    if (d.filt[1]) hipLaunchKernelGGL(k_convert<float>, grid, dim3(256), 0, s, src, (cplx<float>*)d.filt[1], n);
    if (d.filt[2]) hipLaunchKernelGGL(k_convert<df32>, grid, dim3(256), 0, s, src, (cplx<df32>*)d.filt[2], n);
  }
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? hipStreamSynchronize(s) : e;
}

template <typename T>
hipError_t product_blu(birk_plan* p, const PairSet& ps, const T* v, T* out, int transpose, hipStream_t s) {
  if (ps.host.empty()) return hipSuccess;
  cplx<T>* G = (cplx<T>*)p->work[0];
  cplx<T>* Y = (cplx<T>*)p->work[1];
  const cplx<T>* tw = (const cplx<T>*)p->lds_tw[prec_index<T>()];
  const size_t lc = ps.lds_c * sizeof(T), lr = ps.lds_r * sizeof(T);
  constexpr int mc = lds_cols_most() * (int)sizeof(T), mr = lds_rows_most() * (int)sizeof(T);
  lds_limit(k_blu_cols<T>, mc);
  lds_limit(k_blu_rows<T, false>, mr);
  lds_limit(k_blu_icols<T, false>, mc);
  lds_limit(k_blu_icols<T, true>, mc);
  const dim3 gc(ps.n_c4), gr(ps.n_r4), bc(ps.thr_c), br(ps.thr_r);
  hipLaunchKernelGGL(k_blu_cols<T>, gc, bc, lc, s, v, Y, G, ps.dev, ps.tiles_c4, tw,
                     (int)(transpose ? kSrcVT : kSrcV));
  hipLaunchKernelGGL((k_blu_rows<T, false>), gr, br, lr, s, G, ps.dev, ps.tiles_r4, tw);
  hipLaunchKernelGGL((k_blu_icols<T, false>), gc, bc, lc, s, G, Y, out, ps.dev, ps.tiles_c4, tw, transpose);
  hipLaunchKernelGGL(k_blu_cols<T>, gc, bc, lc, s, v, Y, G, ps.dev, ps.tiles_c4, tw,
                     (int)(transpose ? kSrcTr : kSrcFwd));
  hipLaunchKernelGGL((k_blu_rows<T, false>), gr, br, lr, s, G, ps.dev, ps.tiles_r4, tw);
  hipLaunchKernelGGL((k_blu_icols<T, true>), gc, bc, lc, s, G, Y, out, ps.dev, ps.tiles_c4, tw, transpose);
  return hipGetLastError();
}

template hipError_t product_blu<double>(birk_plan*, const PairSet&, const double*, double*, int, hipStream_t);
template hipError_t product_blu<float>(birk_plan*, const PairSet&, const float*, float*, int, hipStream_t);
template hipError_t product_blu<df32>(birk_plan*, const PairSet&, const df32*, df32*, int, hipStream_t);

}  // namespace birk
