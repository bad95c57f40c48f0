// Vector passes and scalars of the Krylov solvers (gfx950): at most kMaxDots basis vectors per
// call, reductions in double.
//
// Bound: memory (an element of every vector read or written once per pass; 50 MB a vector at
// N = 2^20, n_x = 6).  The passes of a one-step GMRES solve there took 340 us and take 190: chi
// and J chi are written in one launch where they were cleared and added to in four (102 us, now
// 39), the residual's norm is taken where the residual is formed (45, now 39), a basis vector is
// scaled when a step needs it and not after the last one (17), and the tile sums are read
// along their slot (8.2 us a reduction, now 4.5).  At 65537 nodes combining one vector took 13
// us (32 predicated terms an element, one element at a time) and takes 5.7.

#include <hip/hip_runtime.h>

#include <cmath>

#include "birk_internal.h"
#include "birk_mid.h"

namespace birk {

constexpr int kMaxDots = kKryMaxDots;
constexpr int kItems = kSegChunk / 256;   // elements of a tile per thread

static inline unsigned nblocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// z = a - b  (FastAX step 3)
template <typename T>
__global__ void k_sub(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ z, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  z[e] = a[e] - b[e];
}

// ---- segmented forms: one launch over every instance of the batch ----
// A tile is kSegChunk consecutive elements of one instance, thread t's at t + 256 k.  Partial
// sums go to part[slot][tile] (slot: basis vector, kMaxDots the norm; the tiles of an instance
// side by side, so that their sum reads whole lines) and are summed per instance over its tile
// range in a fixed order.  Products are fused into the sums explicitly: left to the compiler,
// which one of a sum's first two products is rounded differs from kernel to kernel.

struct Tile {
  int inst;
  int64_t base, n;   // first element, elements
};
__device__ __forceinline__ Tile tile_of(const SegSet& sg, int b) {
  const int2 t = sg.tiles[b];
  const int64_t o = (int64_t)t.y * kSegChunk;
  return {t.x, sg.ioff[t.x] + o, min((int64_t)kSegChunk, sg.ilen[t.x] - o)};
}

// Sums over the workgroup (256 threads) of n <= N values each: that of value k in thread k.
template <int N>
__device__ __forceinline__ double group_sums(double (&v)[N], int n, double* sh) {
  const int wv = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63);
#pragma unroll
  for (int k = 0; k < N; ++k)
    if (k < n) {
      const double s = wave_sum_last(v[k]);
      if (l == 63) sh[wv * N + k] = s;
    }
  __syncthreads();
  const int k = (int)threadIdx.x;
  return k < n ? ((sh[k] + sh[N + k]) + sh[2 * N + k]) + sh[3 * N + k] : 0.0;
}

// Elements in flight per thread: U of its kItems at a time, all loads before their use.
// NQ basis vectors exactly up to 2, at most NQ above.
template <int NQ>
constexpr int kUnroll = NQ <= 1 ? 8 : NQ <= 2 ? 4 : NQ <= 8 ? 2 : 1;

// part <- tile sums of Q_k . u and ||u||^2.  SUB: u = a - b (in T, as k_sub does), stored.
template <typename T, int NQ, int SUB>
__global__ __launch_bounds__(256) void k_sdots(const T* __restrict__ Q, int64_t ld, int nq, const T* __restrict__ u_in,
                                               const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ u_out,
                                               SegSet sg, double* __restrict__ part) {
  constexpr int U = kUnroll<NQ>;
  __shared__ double sh[4 * (NQ + 1)];
  const Tile t = tile_of(sg, blockIdx.x);
  double acc[NQ + 1];
#pragma unroll
  for (int i = 0; i <= NQ; ++i) acc[i] = 0.0;
#pragma unroll 1
  for (int k0 = 0; k0 < kItems; k0 += U) {
    if (k0 * 256 >= t.n) break;
    double u[U];
    bool in[U];
    int64_t e[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int r = (int)threadIdx.x + 256 * (k0 + k);
      in[k] = r < t.n;
      e[k] = t.base + (in[k] ? r : 0);
      if (SUB) {
        const T d = a[e[k]] - b[e[k]];
        if (in[k]) u_out[e[k]] = d;
        u[k] = in[k] ? (double)d : 0.0;
      } else {
        const double v = (double)u_in[e[k]];
        u[k] = in[k] ? v : 0.0;
      }
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (NQ <= 2 || i < nq) {
        double q[U];
#pragma unroll
        for (int k = 0; k < U; ++k) q[k] = (double)Q[(int64_t)i * ld + e[k]];
#pragma unroll
        for (int k = 0; k < U; ++k) acc[i] = fma(q[k], u[k], acc[i]);
      }
#pragma unroll
    for (int k = 0; k < U; ++k) acc[NQ] = fma(u[k], u[k], acc[NQ]);
  }
  // the norm in the last slot of the nq + 1 that are summed
  if (NQ > 2) {
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (i == nq) acc[i] = acc[NQ];
  }
  const double s = group_sums<NQ + 1>(acc, nq + 1, sh);
  const int k = (int)threadIdx.x;
  if (k <= nq) part[(int64_t)(k < nq ? k : kMaxDots) * sg.ntiles + blockIdx.x] = s;
}

// CALL with NQ a bound of the nq basis vectors (exact up to 2)
#define BIRK_NQ_SWITCH(nq, CALL)                           \
  if ((nq) == 0) { constexpr int NQ = 0; CALL; }           \
  else if ((nq) == 1) { constexpr int NQ = 1; CALL; }      \
  else if ((nq) == 2) { constexpr int NQ = 2; CALL; }      \
  else if ((nq) <= 8) { constexpr int NQ = 8; CALL; }      \
  else { constexpr int NQ = kMaxDots; CALL; }

// Sum of instance i's tiles of one slot, in thread 0 (256 threads).
__device__ __forceinline__ double tiles_sum(const double* __restrict__ part, const SegSet& sg, int i, int slot,
                                            double* sh) {
  const int2 r = sg.ranges[i];
  const double* p = part + (int64_t)slot * sg.ntiles;
  double s[1] = {0.0};
#pragma unroll 4
  for (int b = r.x + (int)threadIdx.x; b < r.y; b += 256) s[0] += p[b];
  return group_sums<1>(s, 1, sh);
}

// grid = (nq + 1, instances): block (x, i) sums output x (x == nq: the norm slot) of
// instance i over its tiles into out[i * ostride + slot].
__global__ __launch_bounds__(256) void k_sreduce(const double* __restrict__ part, SegSet sg, int nq,
                                                 double* __restrict__ out, int64_t ostride) {
  __shared__ double sh[4];
  const int i = blockIdx.y;
  const int slot = (blockIdx.x < (unsigned)nq) ? (int)blockIdx.x : kMaxDots;
  const double tot = tiles_sum(part, sg, i, slot, sh);
  if (threadIdx.x == 0) out[(int64_t)i * ostride + slot] = tot;
}

// u -= sum_k h[i][k] Q_k on instance i's tiles; part <- tile sums of ||u||^2, and with DOTS
// also of Q_k . u (the updated u), the first half of the next Gram-Schmidt pass.
template <typename T, bool DOTS, int NQ>
__global__ __launch_bounds__(256) void k_saxpys(const T* __restrict__ Q, int64_t ld, int nq,
                                                const double* __restrict__ h, int64_t hstride, T* __restrict__ u,
                                                SegSet sg, double* __restrict__ part) {
  constexpr int U = kUnroll<NQ>, ND = DOTS ? NQ : 0;
  __shared__ double sh[4 * (ND + 1)];
  const Tile t = tile_of(sg, blockIdx.x);
  const double* hi = h + (int64_t)t.inst * hstride;
  double acc[ND + 1];
#pragma unroll
  for (int i = 0; i <= ND; ++i) acc[i] = 0.0;
#pragma unroll 1
  for (int k0 = 0; k0 < kItems; k0 += U) {
    if (k0 * 256 >= t.n) break;
    double ue[U], q[NQ + 1][U];
    bool in[U];
    int64_t e[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int r = (int)threadIdx.x + 256 * (k0 + k);
      in[k] = r < t.n;
      e[k] = t.base + (in[k] ? r : 0);
      ue[k] = (double)u[e[k]];
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (NQ <= 2 || i < nq) {
#pragma unroll
        for (int k = 0; k < U; ++k) q[i][k] = (double)Q[(int64_t)i * ld + e[k]];
        const double c = hi[i];
#pragma unroll
        for (int k = 0; k < U; ++k) ue[k] = fma(-c, q[i][k], ue[k]);
      }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const T us = (T)ue[k];
      if (in[k]) u[e[k]] = us;
      const double un = in[k] ? (double)us : 0.0;
      acc[ND] = fma(un, un, acc[ND]);
      if constexpr (DOTS) {
#pragma unroll
        for (int i = 0; i < NQ; ++i)
          if (NQ <= 2 || i < nq) acc[i] = fma(q[i][k], un, acc[i]);
      }
    }
  }
  if (DOTS && NQ > 2) {
#pragma unroll
    for (int i = 0; i < ND; ++i)
      if (i == nq) acc[i] = acc[ND];
  }
  const int ns = DOTS ? nq : 0;
  const double s = group_sums<ND + 1>(acc, ns + 1, sh);
  const int k = (int)threadIdx.x;
  if (k <= ns) part[(int64_t)(k < ns ? k : kMaxDots) * sg.ntiles + blockIdx.x] = s;
}

// One pass over a tile, four elements a thread in flight: f(element).
template <typename F>
__device__ __forceinline__ void each4(const Tile& t, F&& f) {
#pragma unroll 4
  for (int k = 0; k < kItems; ++k) {
    const int r = (int)threadIdx.x + 256 * k;
    if (r < t.n) f(t.base + r);
  }
}

// r = beta - (x - t) = beta - x + t; part <- tile sums of ||r||^2
__global__ __launch_bounds__(256) void k_sresidual(const double* __restrict__ beta, const double* __restrict__ x,
                                                   const double* __restrict__ tv, double* __restrict__ r, SegSet sg,
                                                   double* __restrict__ part) {
  __shared__ double sh[4];
  const Tile t = tile_of(sg, blockIdx.x);
  double acc[1] = {0.0};
  each4(t, [&](int64_t e) {
    const double v = beta[e] - x[e] + tv[e];
    r[e] = v;
    acc[0] = fma(v, v, acc[0]);
  });
  const double s = group_sums<1>(acc, 1, sh);
  if (threadIdx.x == 0) part[(int64_t)kMaxDots * sg.ntiles + blockIdx.x] = s;
}

// G = X - xa - G, component by component; part <- tile sums of ||G||^2 (norm slot) and ||X||^2
// (slot 0), in the pass that has both at hand.
__global__ __launch_bounds__(256) void k_sivp(const InstDesc* __restrict__ idesc, const double* __restrict__ xa,
                                              const double* __restrict__ X, double* __restrict__ G, SegSet sg,
                                              double* __restrict__ part) {
  __shared__ double sh[8];
  const Tile t = tile_of(sg, blockIdx.x);
  const int64_t Nn = idesc[t.inst].Nn, rel = t.base - sg.ioff[t.inst] + threadIdx.x;
  const double* xc = xa + sg.icol[t.inst];
  int64_t c = rel / Nn, r = rel - c * Nn;   // component and node of the thread's element
  double acc[2] = {0.0, 0.0};
#pragma unroll 4
  for (int k = 0; k < kItems; ++k) {
    const int64_t i = (int64_t)threadIdx.x + 256 * k;
    if (i < t.n) {
      const double x = X[t.base + i], g = x - xc[c] - G[t.base + i];
      G[t.base + i] = g;
      acc[0] = fma(x, x, acc[0]);
      acc[1] = fma(g, g, acc[1]);
    }
    r += 256;
    while (r >= Nn) {
      r -= Nn;
      ++c;
    }
  }
  const double s = group_sums<2>(acc, 2, sh);
  if (threadIdx.x < 2) part[(int64_t)(threadIdx.x ? kMaxDots : 0) * sg.ntiles + blockIdx.x] = s;
}

// q = u / sqrt(nrm2[i]) on instance i's tiles; a zero or non-finite norm writes zeros
// (the instance has stopped; its later basis vectors are never combined).
__device__ __forceinline__ double inv_norm(double n2) { return (n2 > 0.0 && isfinite(n2)) ? 1.0 / sqrt(n2) : 0.0; }

template <typename T>
__global__ __launch_bounds__(256) void k_snormalize(const T* __restrict__ u, const double* __restrict__ nrm2,
                                                    int64_t stride, T* __restrict__ q, SegSet sg) {
  const Tile t = tile_of(sg, blockIdx.x);
  const double inv = inv_norm(nrm2[(int64_t)t.inst * stride]);
  each4(t, [&](int64_t e) { q[e] = (T)(inv == 0.0 ? 0.0 : (double)u[e] * inv); });
}

// y = alpha[i] x on instance i's tiles
__global__ __launch_bounds__(256) void k_sscale(const double* __restrict__ x, double* __restrict__ y,
                                                const double* __restrict__ alpha, SegSet sg) {
  const Tile t = tile_of(sg, blockIdx.x);
  const double a = alpha[t.inst];
  each4(t, [&](int64_t e) { y[e] = a == 0.0 ? 0.0 : a * x[e]; });
}

// x = x0 (or zero where null) + sum_{k < cnt[i]} c[i][k] Q_k on instance i's tiles (x double, sum
// in double; x may be x0); blockIdx.y chooses between the two sets (GMRES: chi and J chi).
template <typename T>
struct Combine {
  const T* Q;
  const double* x0;
  double* x;
};
template <typename T>
__global__ __launch_bounds__(256) void k_scombine(Combine<T> s0, Combine<T> s1, int64_t ld, const double* __restrict__ c,
                                                  int64_t cstride, const int* __restrict__ cnt, SegSet sg) {
  const Combine<T> s = blockIdx.y ? s1 : s0;
  const Tile t = tile_of(sg, blockIdx.x);
  const int nq = cnt[t.inst];
  const double* ci = c + (int64_t)t.inst * cstride;
  double acc[kItems];
  int64_t e[kItems];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int r = (int)threadIdx.x + 256 * k;
    e[k] = t.base + (r < t.n ? r : 0);
    acc[k] = 0.0;
  }
#pragma unroll 2
  for (int i = 0; i < nq; ++i) {
    const double w = ci[i];
    const T* q = s.Q + (int64_t)i * ld;
#pragma unroll
    for (int k = 0; k < kItems; ++k) acc[k] = fma(w, (double)q[e[k]], acc[k]);
  }
  double x0[kItems];
#pragma unroll
  for (int k = 0; k < kItems; ++k) x0[k] = s.x0 ? s.x0[e[k]] : 0.0;
#pragma unroll
  for (int k = 0; k < kItems; ++k)
    if ((int)threadIdx.x + 256 * k < t.n) s.x[e[k]] = x0[k] + acc[k];
}

// ---- GMRES scalars on the device: per instance the rotated Hessenberg columns R, the
// right-hand side g of the small least-squares problem, the Givens rotations, and
// (running, columns kept, iterations, status, tolerance, ||r||); one thread per instance.
__device__ __forceinline__ void gm_init(int i, const double* __restrict__ prm, double* __restrict__ st) {
  double* s = st + (int64_t)i * kGmStride;
  for (int k = 0; k < kGmLd; ++k) s[kGmG + k] = 0.0;
  s[kGmG] = 1.0;
  s[kGmMisc + GM_RUN] = prm[3 * i];
  s[kGmMisc + GM_ACTIVE] = prm[3 * i];
  s[kGmMisc + GM_JEND] = 0.0;
  s[kGmMisc + GM_INNER] = 0.0;
  s[kGmMisc + GM_STATUS] = 0.0;
  s[kGmMisc + GM_TOL] = prm[3 * i + 1];
  s[kGmMisc + GM_RNORM] = prm[3 * i + 2];
}

// Start of a cycle: q_0 = r / ||r|| on every instance's tiles (zero where it is not active), and
// the instances' states, from the (active, tolerance, ||r||) that the host sends.
// One launch and one copy where there were two each: 200 -> 193 us for the solve at 257 nodes.
template <typename T>
__global__ __launch_bounds__(256) void k_gm_start(const double* __restrict__ r, T* __restrict__ q,
                                                  const double* __restrict__ prm, double* __restrict__ st, SegSet sg) {
  const Tile t = tile_of(sg, blockIdx.x);
  const double rn = prm[3 * t.inst + 2];
  const double a = prm[3 * t.inst] != 0.0 && rn > 0.0 ? 1.0 / rn : 0.0;
  each4(t, [&](int64_t e) { q[e] = (T)(a == 0.0 ? 0.0 : a * r[e]); });
  if (threadIdx.x == 0 && (int)blockIdx.x == sg.ranges[t.inst].x) gm_init(t.inst, prm, st);
}

// Arnoldi column j of a running instance i from the CGS2 dot products (d1 + d2 = the
// coefficients, the norm slot of d2 = ||u||^2): earlier rotations, a new rotation that
// annihilates h_{j+1,j}, the update of g; the instance stops when |g_{j+1}| <= tol, on a
// lucky breakdown, on breakdown (no column kept) or on a non-finite value.
__device__ __forceinline__ void gm_column(int i, int j, const double* dots, int64_t dstride, double* __restrict__ st) {
  double* s = st + (int64_t)i * kGmStride;
  double* misc = s + kGmMisc;
  if (misc[GM_RUN] == 0.0) return;
  misc[GM_INNER] += 1.0;
  const double* d1 = dots + (int64_t)i * dstride;
  const double* d2 = d1 + kGmLd;
  double* col = s + kGmR + (int64_t)j * kGmLd;
  double* cs = s + kGmCs;
  double* sn = s + kGmSn;
  double* g = s + kGmG;
  const double hn2 = d2[kMaxDots];
  const double hn = isfinite(hn2) ? sqrt(hn2 > 0.0 ? hn2 : 0.0) : NAN;
  bool finite = isfinite(hn);
  for (int k = 0; k <= j; ++k) {
    col[k] = d1[k] + d2[k];
    finite = finite && isfinite(col[k]);
  }
  if (!finite) {
    misc[GM_STATUS] = (double)BIRK_ERR_NONFINITE;
    misc[GM_RUN] = 0.0;
    misc[GM_JEND] = (double)j;
    return;
  }
  double below = hn;
  for (int k = 0; k < j; ++k) {
    // (fused in one way, so that both callers round alike)
    const double a = fma(cs[k], col[k], sn[k] * col[k + 1]);
    col[k + 1] = fma(cs[k], col[k + 1], -(sn[k] * col[k]));
    col[k] = a;
  }
  const double den = hypot(col[j], below);
  if (den == 0.0) {
    misc[GM_STATUS] = (double)BIRK_ERR_BREAKDOWN;
    misc[GM_RUN] = 0.0;
    misc[GM_JEND] = (double)j;
    return;
  }
  cs[j] = col[j] / den;
  sn[j] = below / den;
  col[j] = den;
  g[j + 1] = -sn[j] * g[j];
  g[j] = cs[j] * g[j];
  misc[GM_JEND] = (double)(j + 1);
  const bool lucky = hn <= 1e-14 * den;
  if (fabs(g[j + 1]) <= misc[GM_TOL] || lucky) misc[GM_RUN] = 0.0;
}

// End of a step: ||u||^2 from its tile sums, the column, and whether the instance is still
// running into flags[i] for the host.  One workgroup per instance.
__global__ __launch_bounds__(256) void k_gm_column(int j, double* __restrict__ dots, int64_t dstride,
                                                   const double* __restrict__ part, SegSet sg, double* __restrict__ st,
                                                   double* __restrict__ flags) {
  __shared__ double sh[4];
  const int i = blockIdx.x;
  const double n2 = tiles_sum(part, sg, i, kMaxDots, sh);
  if (threadIdx.x) return;
  dots[(int64_t)i * dstride + kGmLd + kMaxDots] = n2;
  gm_column(i, j, dots, dstride, st);
  flags[i] = st[(int64_t)i * kGmStride + kGmMisc + GM_RUN];
}

// The whole orthogonalisation of step j for plans whose instances are one tile each:
// u = a - b, the two Gram-Schmidt passes against q_0 .. q_j, the column and q_{j+1}, u in
// registers.  Element to thread and the order of every sum are those of the kernels above,
// whose results this gives bit for bit.  Bound: launches and latency; a step of the solve at
// 257 nodes took eight of them and 27 us, and takes this one and 7.
template <typename T>
__global__ __launch_bounds__(256) void k_gs_tile(T* __restrict__ Q, int64_t ld, int j, const T* __restrict__ a,
                                                 const T* __restrict__ b, double* __restrict__ dots, int64_t dstride,
                                                 SegSet sg, double* __restrict__ st, double* __restrict__ flags) {
  __shared__ double sh[4 * (kMaxDots + 1)], hs[kMaxDots + 1];
  const int i = blockIdx.x, tid = (int)threadIdx.x, wv = tid >> 6, nq = j + 1;
  const int n = (int)sg.ilen[i];
  const int64_t base = sg.ioff[i];
  T u[kItems];
  bool in[kItems];
  int64_t e[kItems];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int r = tid + 256 * k;
    in[k] = r < n;
    e[k] = base + (in[k] ? r : 0);
    const T v = a[e[k]] - b[e[k]];
    u[k] = in[k] ? v : T(0);
  }
  // pass 0: Q . u; pass 1: u -= h . Q, Q . u; pass 2: u -= h . Q, ||u||^2
  double* d = dots + (int64_t)i * dstride;
#pragma unroll 1
  for (int pass = 0; pass < 3; ++pass) {
    if (pass) {
      double ue[kItems];
#pragma unroll
      for (int k = 0; k < kItems; ++k) ue[k] = (double)u[k];
#pragma unroll 2
      for (int q = 0; q < nq; ++q) {
        const double c = hs[q];
#pragma unroll
        for (int k = 0; k < kItems; ++k) ue[k] = fma(-c, (double)Q[(int64_t)q * ld + e[k]], ue[k]);
      }
#pragma unroll
      for (int k = 0; k < kItems; ++k) u[k] = in[k] ? (T)ue[k] : T(0);
    }
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) s = fma((double)u[k], (double)u[k], s);
    s = wave_sum_last(s);
    if ((tid & 63) == 63) sh[wv * (kMaxDots + 1) + kMaxDots] = s;
    if (pass < 2) {
#pragma unroll 2
      for (int q = 0; q < nq; ++q) {
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) v = fma((double)Q[(int64_t)q * ld + e[k]], (double)u[k], v);
        v = wave_sum_last(v);
        if ((tid & 63) == 63) sh[wv * (kMaxDots + 1) + q] = v;
      }
    }
    __syncthreads();
    if (tid <= kMaxDots && (tid == kMaxDots || (pass < 2 && tid < nq))) {
      const double v = ((sh[tid] + sh[kMaxDots + 1 + tid]) + sh[2 * (kMaxDots + 1) + tid]) + sh[3 * (kMaxDots + 1) + tid];
      hs[tid] = v;
      d[(pass ? kGmLd : 0) + tid] = v;
    }
    __syncthreads();
  }
  const double inv = inv_norm(hs[kMaxDots]);
#pragma unroll
  for (int k = 0; k < kItems; ++k)
    if (in[k]) Q[(int64_t)nq * ld + e[k]] = (T)(inv == 0.0 ? 0.0 : (double)u[k] * inv);
  if (tid == 0) {
    __threadfence_block();
    gm_column(i, j, dots, dstride, st);
    flags[i] = st[(int64_t)i * kGmStride + kGmMisc + GM_RUN];
  }
}

// End of a cycle: y = R^{-1} g on the kept columns, coefficients ||r|| y and their count
// for the combination chi += sum_k c_k z_k; (running, iterations, status) per instance
// into flags[3 i ...] for the host.
__global__ void k_gm_solve(double* __restrict__ st, double* __restrict__ coef, int64_t cstride, int* __restrict__ cnt,
                           double* __restrict__ flags, int ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
  double* s = st + (int64_t)i * kGmStride;
  const double* misc = s + kGmMisc;
  double* c = coef + (int64_t)i * cstride;
  const int k = misc[GM_ACTIVE] != 0.0 ? (int)misc[GM_JEND] : 0;
  const double* R = s + kGmR;
  const double* g = s + kGmG;
  double y[kMaxDots];
  for (int a = k - 1; a >= 0; --a) {
    double acc = g[a];
    for (int b = a + 1; b < k; ++b) acc -= R[(int64_t)b * kGmLd + a] * y[b];
    y[a] = acc / R[(int64_t)a * kGmLd + a];
  }
  for (int a = 0; a < k; ++a) c[a] = y[a] * misc[GM_RNORM];
  cnt[i] = k;
  flags[3 * i] = misc[GM_RUN];
  flags[3 * i + 1] = misc[GM_INNER];
  flags[3 * i + 2] = misc[GM_STATUS];
}


// Host-side launch helpers used by the GMRES driver.
namespace kry {

bool one_tile(const birk_plan* p) { return p->seg.ntiles == (int)p->inst.size(); }

template <typename T>
void sub(const T* a, const T* b, T* z, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_sub<T>, dim3(nblocks(n, 256)), dim3(256), 0, s, a, b, z, n);
}

static void sreduce(const birk_plan* p, int nq, double* out, int64_t ostride, hipStream_t s) {
  hipLaunchKernelGGL(k_sreduce, dim3(nq + 1, (unsigned)p->inst.size()), dim3(256), 0, s, p->krylov_part, p->seg, nq,
                     out, ostride);
}

void snorms(const birk_plan* p, const double* v, double* out, int64_t ostride, hipStream_t s) {
  hipLaunchKernelGGL((k_sdots<double, 0, 0>), dim3(p->seg.ntiles), dim3(256), 0, s, (const double*)nullptr,
                     p->total_len, 0, v, (const double*)nullptr, (const double*)nullptr, (double*)nullptr, p->seg,
                     p->krylov_part);
  sreduce(p, 0, out, ostride, s);
}

void residual(const birk_plan* p, const double* beta, const double* x, const double* t, double* r, double* out,
              int64_t ostride, hipStream_t s) {
  hipLaunchKernelGGL(k_sresidual, dim3(p->seg.ntiles), dim3(256), 0, s, beta, x, t, r, p->seg, p->krylov_part);
  sreduce(p, 0, out, ostride, s);
}

void ivp_residual(const birk_plan* p, const double* xa, const double* X, double* G, double* out, int64_t ostride,
                  hipStream_t s) {
  hipLaunchKernelGGL(k_sivp, dim3(p->seg.ntiles), dim3(256), 0, s, p->idesc, xa, X, G, p->seg, p->krylov_part);
  sreduce(p, 1, out, ostride, s);
}

template <typename T>
void gram_schmidt(const birk_plan* p, T* Q, int j, const T* a, const T* b, T* u, double* dots, int64_t dstride,
                  double* st, double* flags, hipStream_t s) {
  const SegSet& sg = p->seg;
  const int nq = j + 1, B = (int)p->inst.size();
  const int64_t ld = p->total_len;
  if (one_tile(p)) {
    hipLaunchKernelGGL(k_gs_tile<T>, dim3(B), dim3(256), 0, s, Q, ld, j, a, b, dots, dstride, sg, st, flags);
    return;
  }
  double* d2 = dots + kGmLd;
  BIRK_NQ_SWITCH(nq, hipLaunchKernelGGL((k_sdots<T, NQ, 1>), dim3(sg.ntiles), dim3(256), 0, s, (const T*)Q, ld, nq,
                                        (const T*)nullptr, a, b, u, sg, p->krylov_part))
  sreduce(p, nq, dots, dstride, s);
  BIRK_NQ_SWITCH(nq, hipLaunchKernelGGL((k_saxpys<T, true, NQ>), dim3(sg.ntiles), dim3(256), 0, s, (const T*)Q, ld, nq,
                                        (const double*)dots, dstride, u, sg, p->krylov_part))
  sreduce(p, nq, d2, dstride, s);
  BIRK_NQ_SWITCH(nq, hipLaunchKernelGGL((k_saxpys<T, false, NQ>), dim3(sg.ntiles), dim3(256), 0, s, (const T*)Q, ld,
                                        nq, (const double*)d2, dstride, u, sg, p->krylov_part))
  hipLaunchKernelGGL(k_gm_column, dim3(B), dim3(256), 0, s, j, dots, dstride, (const double*)p->krylov_part, sg, st,
                     flags);
}

template <typename T>
void next_vector(const birk_plan* p, const T* u, const double* dots, int64_t dstride, T* q, hipStream_t s) {
  if (one_tile(p)) return;   // k_gs_tile has written it
  hipLaunchKernelGGL(k_snormalize<T>, dim3(p->seg.ntiles), dim3(256), 0, s, u, dots + kGmLd + kMaxDots, dstride, q,
                     p->seg);
}

void sscale(const birk_plan* p, const double* x, double* y, const double* alpha, hipStream_t s) {
  hipLaunchKernelGGL(k_sscale, dim3(p->seg.ntiles), dim3(256), 0, s, x, y, alpha, p->seg);
}

template <typename T>
void scombine(const birk_plan* p, const double* c, int64_t cstride, const int* cnt, const T* Q0, const double* x0,
              double* x, const T* Q1, const double* y0, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_scombine<T>, dim3(p->seg.ntiles, Q1 ? 2 : 1), dim3(256), 0, s, Combine<T>{Q0, x0, x},
                     Combine<T>{Q1, y0, y}, p->total_len, c, cstride, cnt, p->seg);
}

template <typename T>
void gm_start(const birk_plan* p, const double* r, T* q, const double* prm, double* st, hipStream_t s) {
  hipLaunchKernelGGL(k_gm_start<T>, dim3(p->seg.ntiles), dim3(256), 0, s, r, q, prm, st, p->seg);
}
void gm_solve(const birk_plan* p, double* st, double* coef, int64_t cstride, int* cnt, double* flags, hipStream_t s) {
  const int B = (int)p->inst.size();
  hipLaunchKernelGGL(k_gm_solve, dim3(nblocks(B, 64)), dim3(64), 0, s, st, coef, cstride, cnt, flags, B);
}

#define INST(T)                                                                                                        \
  template void sub<T>(const T*, const T*, T*, int64_t, hipStream_t);                                                  \
  template void gram_schmidt<T>(const birk_plan*, T*, int, const T*, const T*, T*, double*, int64_t, double*, double*, \
                                hipStream_t);                                                                          \
  template void next_vector<T>(const birk_plan*, const T*, const double*, int64_t, T*, hipStream_t);                   \
  template void gm_start<T>(const birk_plan*, const double*, T*, const double*, double*, hipStream_t);                \
  template void scombine<T>(const birk_plan*, const double*, int64_t, const int*, const T*, const double*, double*,    \
                            const T*, const double*, double*, hipStream_t);
INST(double)
INST(float)
#undef INST
#undef BIRK_NQ_SWITCH

}  // namespace kry
}  // namespace birk
