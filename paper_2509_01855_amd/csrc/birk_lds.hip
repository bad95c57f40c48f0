// Products whose transforms fit one workgroup (gfx950): N <= 2048 a power of two, or any N
// with 3N <= 4096.  One launch takes a component or a pair of them from v to out: DCT-I, the
// coefficient stencil with c^_0, DCT-I, all in LDS, so that a product reads v and writes
// out once and a small product is one launch instead of five (Bluestein) to seven (pack,
// transform, stencil, c^_0, transform, unpack).
//
// k_lds_product: a pair of components as one complex vector, N < 512 and the chirp lengths.
// k_lds_even: one component, N = 512, 1024, 2048.  There, as in the three passes of longer
// powers of two, no component may meet another's rounding or infinities (states are often
// in units 10^3 apart), so a pair must not share a complex vector.
//
// A DCT-I is half the DFT of the even extension, of length L = 2N (see birk_dct.hip): L a
// power of two is transformed as it is, any other L by Bluestein's convolution in a
// power-of-two length M >= 3N.  A thread holds eight elements n = tid + i blockDim of its
// pairs' M-long buffers from the first load to the last store; the chirp (even, so its
// N + 1 first values serve every n) and the filter spectrum are read once for both DCTs.
//
// What bounds it: at few pairs the chain of LDS stages behind barriers (four transforms of
// four stages at M = 1024); with many pairs LDS bandwidth.  A pair of components per
// workgroup (M / 8 threads) keeps the chain short and uses as many CUs as there are pairs;
// plans whose largest M is below 512 put 512 / M pairs in one wave.  Measured per product,
// six components in double, before (five to seven launches) and after: N = 255 (M = 1024)
// 36.6 -> 16.5 us, 256 28.4 -> 11.2, 999 (M = 4096) 36.1 -> 29.7; 192 components: N = 256
// 46.2 -> 11.5 us.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "birk_fft.h"
#include "birk_internal.h"
#include "birk_mid.h"

namespace birk {
namespace {

constexpr int kPPT = fast::kPPT;

template <typename T, int LOGM>
__device__ __forceinline__ void put(T* sm, int t, int n, cplx<T> v) {
  constexpr int LD = fast::padded_ld(1 << LOGM);
  sm[2 * t * LD + fast::pad(n)] = v.x;
  sm[(2 * t + 1) * LD + fast::pad(n)] = v.y;
}

template <typename T, int LOGM>
__device__ __forceinline__ cplx<T> get(const T* sm, int t, int n) {
  constexpr int LD = fast::padded_ld(1 << LOGM);
  return fast::mk<T>(sm[2 * t * LD + fast::pad(n)], sm[(2 * t + 1) * LD + fast::pad(n)]);
}

// The pairs [tile.x, tile.x + tile.y) of one length M = 2^LOGM: one pair from M = 512 on, up
// to 512 / M below; CHIRP: Bluestein.  NT threads work, any others only keep the barriers.
// HOLD: chirp and filter stay in registers between their uses, else they are read again.
// sm: 8 NT complex values in split padded rows; red: the c^_0 partial sums.
template <typename T, int LOGM, bool CHIRP, bool HOLD>
__device__ __forceinline__ void lds_product(const T* __restrict__ x, T* __restrict__ out,
                                            const PairDesc* __restrict__ pd, int2 tile,
                                            const cplx<T>* __restrict__ tw, int trans, T* sm, double* red) {
  constexpr int pi = prec_index<T>();
  constexpr int M = 1 << LOGM;
  constexpr int NT = M / kPPT > 64 ? M / kPPT : 64;
  constexpr int COUNT = kPPT * NT / M;
  constexpr int G = M < 64 ? M : 64;   // lanes of a wave that share a pair
  const int tid = (int)threadIdx.x;
  const bool on = tid < NT;
  // element i of the thread: entry n of pair t (a missing pair t repeats the tile's last
  // one; it is not stored)
  auto where = [&](int i, int& t, int& n) {
    const int e = tid + i * NT;
    t = COUNT > 1 ? e >> LOGM : 0;
    n = e & (M - 1);
  };
  auto desc = [&](int t) -> const PairDesc& { return pd[tile.x + (COUNT > 1 ? min(t, tile.y - 1) : 0)]; };
  cplx<T> v[kPPT], fv[CHIRP ? kPPT : 1], cv[CHIRP ? kPPT : 1];
  auto load_chirp = [&] {
    if constexpr (CHIRP) {
#pragma unroll
      for (int i = 0; i < kPPT; ++i) {
        int t, n;
        where(i, t, n);
        const PairDesc& d = desc(t);
        const int N = (int)d.N, L = 2 * N;
        cv[i] = ((const cplx<T>*)d.chirp[pi])[n <= N ? n : n < L ? L - n : 0];
      }
    }
  };
  auto load_filter = [&] {
    if constexpr (CHIRP) {
#pragma unroll
      for (int i = 0; i < kPPT; ++i) {
        int t, n;
        where(i, t, n);
        fv[i] = ((const cplx<T>*)desc(t).filt[pi])[n];
      }
    }
  };
  if (on) {
    // every load of the thread from a valid address, none behind a branch
    T va[kPPT], vb[kPPT];
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      int t, n;
      where(i, t, n);
      const PairDesc& d = desc(t);
      const int N = (int)d.N, L = 2 * N;
      const int k = n <= N ? n : n < L ? L - n : 0;
      const T* xa = x + d.src;
      va[i] = xa[k];
      vb[i] = xa[(d.has2 ? d.Nn : 0) + k];
    }
    load_chirp();
    if (HOLD) load_filter();
#pragma unroll
    for (int i = 0; i < kPPT; ++i) {
      int t, n;
      where(i, t, n);
      const PairDesc& d = desc(t);
      const int N = (int)d.N, L = 2 * N;
      const T e = (trans && (n == 0 || n == N)) ? T(2) : T(1);   // E^{-1}: ends doubled
      v[i] = fast::mk<T>(n < L ? e * va[i] : T(0), n < L && d.has2 ? e * vb[i] : T(0));
    }
  }
#pragma unroll 1
  for (int dct = 0; dct < 2; ++dct) {
    if (on) {
      if (!HOLD && dct == 1) load_chirp();
#pragma unroll
      for (int i = 0; i < kPPT; ++i) {
        int t, n;
        where(i, t, n);
        if constexpr (CHIRP) v[i] = fast::cmul<T>(v[i], cv[i]);
        put<T, LOGM>(sm, t, n, v[i]);
      }
    }
    __syncthreads();
    fast::fft_ct<T, LOGM, COUNT, true>(sm, tw);
    if constexpr (CHIRP) {
      // x filter, inverse transform as conj FFT conj, x chirp: Y_n, n <= N
      if (on) {
        if (!HOLD) load_filter();
#pragma unroll
        for (int i = 0; i < kPPT; ++i) {
          int t, n;
          where(i, t, n);
          put<T, LOGM>(sm, t, n, fast::conjg<T>(fast::cmul<T>(get<T, LOGM>(sm, t, n), fv[i])));
        }
      }
      __syncthreads();
      fast::fft_ct<T, LOGM, COUNT, true>(sm, tw);
      if (on) {
        if (!HOLD) load_chirp();
#pragma unroll
        for (int i = 0; i < kPPT; ++i) {
          int t, n;
          where(i, t, n);
          put<T, LOGM>(sm, t, n, fast::cmul<T>(fast::conjg<T>(get<T, LOGM>(sm, t, n)), cv[i]));
        }
      }
      __syncthreads();
    }
    if (dct == 1) break;
    // stencil: the thread's inputs of the second DCT, and the c^_0 sums (each Y_k, k <= N,
    // once) of G consecutive entries
    if (on) {
#pragma unroll
      for (int i = 0; i < kPPT; ++i) {
        int t, n;
        where(i, t, n);
        const int N = (int)desc(t).N, L = 2 * N;
        const int k = n <= N ? n : n < L ? L - n : 0;
        const cplx<T> Ym = get<T, LOGM>(sm, t, max(k - 1, 0));
        const cplx<T> Yp = get<T, LOGM>(sm, t, min(k + 1, N));
        cplx<T> r;
        if (trans) {
          r = mid_tr<T>(k, N, get<T, LOGM>(sm, t, 0), Ym, Yp, T(1) / T(2 * N + 2));
        } else {
          r = mid_fwd<T>(max(k, 1), N, Ym, Yp, T(1) / T(N), T(1) / T(4 * N + 4));
          const cplx<T> Y = get<T, LOGM>(sm, t, k);
          const double w = n <= N ? c0_weight(n, N) : 0.0;
          double s0 = w * (double)Y.x, s1 = w * (double)Y.y;
          if constexpr (G == 64) {
            s0 = wave_sum_last(s0);
            s1 = wave_sum_last(s1);
          } else {
#pragma unroll
            for (int off = G / 2; off > 0; off >>= 1) {
              s0 += __shfl_xor(s0, off, 64);
              s1 += __shfl_xor(s1, off, 64);
            }
          }
          if ((tid & (G - 1)) == G - 1) {
            double* p = red + 2 * ((tid + i * NT) / G);
            p[0] = s0;
            p[1] = s1;
          }
        }
        v[i] = (n < L && (trans || k > 0)) ? r : fast::mk<T>(T(0), T(0));
      }
    }
    __syncthreads();
  }
  if (!on) return;
  // out = Y / 2 + c^_0, or e_j Y_j / N
  constexpr int per = M / G;   // partial sums per pair, consecutive
  T ca = T(0), cb = T(0);
  int tc = -1;
#pragma unroll
  for (int i = 0; i < kPPT; ++i) {
    int t, n;
    where(i, t, n);
    if (COUNT > 1 && t >= tile.y) continue;
    const PairDesc& d = desc(t);
    const int N = (int)d.N;
    if (n > N) continue;
    cplx<T> Y = get<T, LOGM>(sm, t, n);
    if (trans) {
      const T sc = ((n == 0 || n == N) ? T(0.5) : T(1)) / T(N);
      Y.x = Y.x * sc;
      Y.y = Y.y * sc;
    } else {
      if (t != tc) {
        // four chains, so that the reads do not wait for the adds
        constexpr int U = per < 4 ? per : 4;
        double s0[U], s1[U];
#pragma unroll
        for (int u = 0; u < U; ++u) s0[u] = s1[u] = 0.0;
        for (int q = 0; q < per; q += U) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            s0[u] += red[2 * (t * per + q + u)];
            s1[u] += red[2 * (t * per + q + u) + 1];
          }
        }
#pragma unroll
        for (int u = 1; u < U; ++u) {
          s0[0] += s0[u];
          s1[0] += s1[u];
        }
        ca = (T)(s0[0] / (double)N);
        cb = (T)(s1[0] / (double)N);
        tc = t;
      }
      Y.x = T(0.5) * Y.x + ca;
      Y.y = T(0.5) * Y.y + cb;
    }
    T* o = out + d.src;
    o[n] = Y.x;
    if (d.has2) o[d.Nn + n] = Y.y;
  }
}

template <typename T, bool CHIRP>
__global__ __launch_bounds__(kLdsMax / kPPT) void k_lds_product(const T* __restrict__ x, T* __restrict__ out,
                                                               const PairDesc* __restrict__ pd,
                                                               const int2* __restrict__ tiles,
                                                               const cplx<T>* __restrict__ tw, int trans) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[2 * kLdsMax / 64];   // 64 lanes a sum from M = 64 on; 512 points below
  T* sm = reinterpret_cast<T*>(smem_raw);
  const int2 tile = tiles[blockIdx.x];
  switch (pd[tile.x].logM) {
#define BIRK_LDS_CASE(LG) \
  case LG: lds_product<T, LG, CHIRP, true>(x, out, pd, tile, tw, trans, sm, red); break;
    BIRK_LDS_CASE(3)
    BIRK_LDS_CASE(4)
    BIRK_LDS_CASE(5)
    BIRK_LDS_CASE(6)
    BIRK_LDS_CASE(7)
    BIRK_LDS_CASE(8)
    BIRK_LDS_CASE(9)
    BIRK_LDS_CASE(10)
    BIRK_LDS_CASE(11)
    BIRK_LDS_CASE(12)
#undef BIRK_LDS_CASE
    default: break;
  }
}

// The longest chirp products in float, where there are more of them than CUs: chirp and filter are
// read again at each use (from the L2), since the registers they would take in between leave room
// for one workgroup a CU instead of two.  N = 1000, 1536 pairs: 151 -> 113 us; 96 pairs 26.0, as
// with the tables held.
template <typename T>
__global__ __launch_bounds__(kLdsMax / kPPT, 4) void k_lds_long(const T* __restrict__ x, T* __restrict__ out,
                                                                const PairDesc* __restrict__ pd,
                                                                const int2* __restrict__ tiles,
                                                                const cplx<T>* __restrict__ tw, int trans) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[2 * kLdsMax / 64];
  lds_product<T, kLdsMaxLog, true, false>(x, out, pd, tiles[blockIdx.x], tw, trans, reinterpret_cast<T*>(smem_raw), red);
}

// One component of N = 2^LOGN per workgroup, N / 8 threads.  The even extension y_m,
// m < 2N, goes through a complex transform of half its length, z_n = y_2n + i y_(2n+1).  Both
// halves are symmetric (y_2n in n -> N - n, y_(2n+1) in n -> N - 1 - n), so that with
// c - i s = W_2N^k, a = (Im Z_k + Im Z_(N-k)) / 2 and b = (Re Z_(N-k) - Re Z_k) / 2
//     E = (Re Z_k + Re Z_(N-k)) / 2,  R = c a + s b,  Y_k = E + R,  Y_(N-k) = E - R
// are the DFT values, all of them real.  Thread t holds k = t + i N/8, i < 4, and N - k;
// Y_(N/2) is Re Z_(N/2) as it stands.  Bound: as above, the chain of LDS stages, then LDS
// bandwidth.  Six components in double at N = 512, 1024, 2048: 6.9, 8.7, 10.4 us; pairs of
// components in transforms of 2N points took 10.5, 12.5, 18.6 (16386 components at N = 2048:
// 353 against 668), a lone component with a zero partner the same and twice as much per
// component once the chip is full.
template <typename T, int LOGN>
__device__ __forceinline__ void lds_even(const T* __restrict__ x, T* __restrict__ out, const PairDesc& d,
                                         const cplx<T>* __restrict__ tw, int trans, T* sm, double* red) {
  constexpr int N = 1 << LOGN, NT = N / kPPT, H = kPPT / 2, LD = fast::padded_ld(N);
  const int t = (int)threadIdx.x;
  const bool on = t < NT;
  T* re = sm;        // N + 1 places: also row Y_0 .. Y_N between the transforms
  T* im = sm + LD;
  T ve[H], vo[H], last = T(0);
  // element 2n (and its mirror) or 2n + 1 of the extension
  auto put_even = [&](int n, T v) {
    re[fast::pad(n)] = v;
    if (n > 0 && n < N / 2) re[fast::pad(N - n)] = v;
  };
  auto put_odd = [&](int n, T v) {
    im[fast::pad(n)] = v;
    im[fast::pad(N - 1 - n)] = v;
  };
  // Y_k and Y_(N-k) of the thread's i-th k
  auto values = [&](int i, T& lo, T& hi) {
    const int k = t + i * NT, m = (N - k) & (N - 1);
    const T zr = re[fast::pad(k)], zi = im[fast::pad(k)], wr = re[fast::pad(m)], wi = im[fast::pad(m)];
    const cplx<T> w = tw[k << (kLdsMaxLog - 1 - LOGN)];   // c - i s
    const T E = T(0.5) * (zr + wr);
    const T R = T(0.5) * (w.x * (zi + wi) - w.y * (wr - zr));
    lo = E + R;
    hi = E - R;
  };
  if (on) {
    const T* xa = x + d.src;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int n = t + i * NT;
      ve[i] = xa[2 * n];
      vo[i] = xa[2 * n + 1];
    }
    if (t == 0) last = xa[N];
    const T e = trans ? T(2) : T(1);   // E^{-1} of the transpose: ends doubled
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int n = t + i * NT;
      put_even(n, n == 0 ? e * ve[i] : ve[i]);
      put_odd(n, vo[i]);
    }
    if (t == 0) put_even(N / 2, e * last);
  }
  __syncthreads();
  fast::fft_ct<T, LOGN, 1, true>(sm, tw);
  // Y in place of the real row (a k and its mirror are read and written by one thread), and
  // the c^_0 sums
  if (on) {
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int k = t + i * NT;
      T lo, hi;
      values(i, lo, hi);
      re[fast::pad(k)] = lo;
      re[fast::pad(N - k)] = hi;
      if (!trans) s += c0_weight(k, N) * (double)lo + c0_weight(N - k, N) * (double)hi;
    }
    if (!trans) {
      if (t == 0) s += c0_weight(N / 2, N) * (double)re[fast::pad(N / 2)];   // W_2N^(N/2) = -i: Y = E = Re Z
      s = wave_sum_last(s);
      if ((t & 63) == 63) red[t >> 6] = s;
    }
  }
  __syncthreads();
  // stencil: the inputs of the second DCT from Y, all read before any is written
  if (on) {
    const T invN = T(1) / T(N), inv4N1 = T(1) / T(4 * N + 4), inv2N1 = T(1) / T(2 * N + 2);
    const T Y0 = re[0];
    auto stencil = [&](int k) {
      const T Ym = re[fast::pad(max(k - 1, 0))], Yp = re[fast::pad(min(k + 1, N))];
      if (trans) return TrStencil<T>(k, N, inv2N1)(Y0, Ym, Yp);
      return FwdStencil<T>(max(k, 1), N, invN, inv4N1)(Ym, Yp);
    };
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int n = t + i * NT;
      const T v = stencil(2 * n);
      ve[i] = (trans || n > 0) ? v : T(0);   // d_0 is c^_0, added at the end
      vo[i] = stencil(2 * n + 1);
    }
    if (t == 0) last = stencil(N);
  }
  __syncthreads();
  if (on) {
#pragma unroll
    for (int i = 0; i < H; ++i) {
      put_even(t + i * NT, ve[i]);
      put_odd(t + i * NT, vo[i]);
    }
    if (t == 0) put_even(N / 2, last);
  }
  __syncthreads();
  fast::fft_ct<T, LOGN, 1, true>(sm, tw);
  if (!on) return;
  // out = Y / 2 + c^_0, or e_j Y_j / N
  T sc = T(0.5), c0 = T(0);
  if (trans) {
    sc = T(1) / T(N);
  } else {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < (NT + 63) / 64; ++w) s += red[w];
    c0 = (T)(s / (double)N);
  }
  T* o = out + d.src;
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const int k = t + i * NT;
    T lo, hi;
    values(i, lo, hi);
    const T f = (trans && k == 0) ? T(0.5) * sc : sc;
    o[k] = f * lo + c0;
    o[N - k] = f * hi + c0;
  }
  if (t == 0) o[N / 2] = sc * re[fast::pad(N / 2)] + c0;
}

template <typename T>
__global__ __launch_bounds__(kLdsMax / 2 / kPPT) void k_lds_even(const T* __restrict__ x, T* __restrict__ out,
                                                                const PairDesc* __restrict__ pd,
                                                                const cplx<T>* __restrict__ tw, int trans) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[kLdsMax / 2 / kPPT / 64];
  T* sm = reinterpret_cast<T*>(smem_raw);
  const PairDesc& d = pd[blockIdx.x];
  switch (d.logM) {
    case 9: lds_even<T, 9>(x, out, d, tw, trans, sm, red); break;
    case 10: lds_even<T, 10>(x, out, d, tw, trans, sm, red); break;
    case 11: lds_even<T, 11>(x, out, d, tw, trans, sm, red); break;
    default: break;
  }
}

// Pairs of length 2^logM in a workgroup, and the LDS (reals) they take.
int lds_pairs(int logM) { return logM >= 9 ? 1 : 512 >> logM; }
int lds_reals(int logM) { return 2 * lds_pairs(logM) * fast::padded_ld(1 << logM); }

template <typename T, bool CHIRP>
hipError_t launch(birk_plan* p, const LdsSet& ls, const T* v, T* out, int transpose, hipStream_t s) {
  const cplx<T>* tw = (const cplx<T>*)p->lds_tw[prec_index<T>()];
  const int bytes = ls.lds_reals * (int)sizeof(T);
  int n = ls.ntiles;
  if constexpr (CHIRP && std::is_same<T, float>::value) {
    if (ls.nlong > kCus) {   // the last tiles of the list
      n -= ls.nlong;
      lds_limit(k_lds_long<T>, bytes);
      hipLaunchKernelGGL(k_lds_long<T>, dim3(ls.nlong), dim3(ls.threads), bytes, s, v, out, ls.dev, ls.tiles + n, tw,
                         transpose);
    }
  }
  if (n > 0) {
    const auto f = k_lds_product<T, CHIRP>;
    lds_limit(f, lds_reals(kLdsMaxLog) * (int)sizeof(T));
    hipLaunchKernelGGL(f, dim3(n), dim3(ls.threads), bytes, s, v, out, ls.dev, ls.tiles, tw, transpose);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t finalize_lds(birk_plan* p, LdsSet& ls) {
  if (ls.host.empty()) return hipSuccess;
  std::stable_sort(ls.host.begin(), ls.host.end(), [](const PairDesc& a, const PairDesc& b) { return a.logM < b.logM; });
  ls.threads = std::max(64, (1 << ls.host.back().logM) / kPPT);
  ls.lds_reals = 0;
  std::vector<int2> tiles;
  const int np = (int)ls.host.size();
  for (int q = 0; q < np;) {
    const int logM = ls.host[q].logM;
    const int per = lds_pairs(logM);
    int cnt = 1;
    while (q + cnt < np && cnt < per && ls.host[q + cnt].logM == logM) ++cnt;
    tiles.push_back(make_int2(q, cnt));
    if (logM == kLdsMaxLog) ++ls.nlong;
    ls.lds_reals = std::max(ls.lds_reals, lds_reals(logM));
    q += cnt;
  }
  ls.ntiles = (int)tiles.size();
  void* d = nullptr;
  hipError_t e = upload_raw(p, ls.host.data(), ls.host.size() * sizeof(PairDesc), &d);
  ls.dev = (PairDesc*)d;
  if (e == hipSuccess) e = upload_raw(p, tiles.data(), tiles.size() * sizeof(int2), &d);
  ls.tiles = (int2*)d;
  return e;
}

// Components by length, and their descriptors.
hipError_t finalize_lds_even(birk_plan* p, LdsSet& ls) {
  if (ls.host.empty()) return hipSuccess;
  std::stable_sort(ls.host.begin(), ls.host.end(), [](const PairDesc& a, const PairDesc& b) { return a.logM < b.logM; });
  const int longest = ls.host.back().logM;
  ls.threads = (1 << longest) / kPPT;
  ls.lds_reals = 2 * fast::padded_ld(1 << longest);
  ls.ntiles = (int)ls.host.size();
  void* d = nullptr;
  const hipError_t e = upload_raw(p, ls.host.data(), ls.host.size() * sizeof(PairDesc), &d);
  ls.dev = (PairDesc*)d;
  return e;
}

template <typename T>
hipError_t product_lds(birk_plan* p, const T* v, T* out, int transpose, hipStream_t s) {
  const LdsSet& le = p->lds_even;
  if (le.ntiles > 0) {
    const int bytes = le.lds_reals * (int)sizeof(T);
    lds_limit(k_lds_even<T>, 2 * fast::padded_ld(kLdsMax / 2) * (int)sizeof(T));
    hipLaunchKernelGGL(k_lds_even<T>, dim3(le.ntiles), dim3(le.threads), bytes, s, v, out, le.dev,
                       (const cplx<T>*)p->lds_tw[prec_index<T>()], transpose);
  }
  const hipError_t e = launch<T, false>(p, p->lds[0], v, out, transpose, s);
  return e == hipSuccess ? launch<T, true>(p, p->lds[1], v, out, transpose, s) : e;
}

template hipError_t product_lds<double>(birk_plan*, const double*, double*, int, hipStream_t);
template hipError_t product_lds<float>(birk_plan*, const float*, float*, int, hipStream_t);
template hipError_t product_lds<df32>(birk_plan*, const df32*, df32*, int, hipStream_t);

}  // namespace birk
