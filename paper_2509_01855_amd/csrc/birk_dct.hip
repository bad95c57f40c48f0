// Fast Birkhoff products B^a v and B^aT g on the CGL grid (gfx950): the general path,
// for any N, batched over every pair of components of every instance of a plan.
//
// FastBV (arXiv 2509.01855, FastBV box) applies Fastv2a, the integration recurrence
// with the T_{N+1} alias (eq:c_k=bydef, eq:chatk=) and Fasta2v.  Writing C for the
// DCT-I of eq:vm=DCT-1, R for index reversal, E = diag(1/2, 1, ..., 1, 1/2) and
// S = diag((-1)^k), Fastv2a is E (2/N) C R and Fasta2v is R C E^{-1}.  Because
// C R = S C and R C = C S, the reversals become sign flips in coefficient space:
//
//     B^a  = (2/N) C [E^{-1} S M S E] C          (M: a -> c^, the recurrence)
//     B^aT = (2/N) E C [S M^T S] C E^{-1}        (C^T = E C E^{-1})
//
// so both products are DCT-I, a three-point coefficient stencil, DCT-I.
//
// The DCT-I of a length-(N+1) vector x is half the DFT of its even extension of
// length L = 2N.  Two real vectors are packed into one complex sequence (the DFT of a
// real even sequence is real, so real and imaginary parts separate).  Which path takes it:
//   * transforms that fit one workgroup (N <= 2048 a power of two, any N with 3N <= 4096):
//     one launch (birk_lds.hip);
//   * N a larger power of two: the three passes of birk_fast.hip, or with BIRK_FAST=0 the
//     plain four-step FFTs of this file;
//   * any other N: chirp convolutions on even sequences (birk_blu.hip).
// This file lays the pairs of every path out, builds the tables and tunes the last one.
//
// Batching: the pairs of all instances of one kind form a set.  Each phase of the product
// is ONE launch over the whole set, whatever the mix of sizes: the grid is a list of
// (pair, block) tiles built at plan creation, and every block reads its pair's sizes,
// offsets and tables from a descriptor.  A product of a batch of uneven instances is
// therefore a fixed number of launches.

#include <hip/hip_runtime.h>

#include <type_traits>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <vector>

#include "birk_fft.h"
#include "birk_internal.h"
#include "birk_mid.h"

namespace birk {

template <typename T>
__device__ __forceinline__ cplx<T> cmul(cplx<T> a, cplx<T> b) {
  cplx<T> r;
  r.x = a.x * b.x - a.y * b.y;
  r.y = a.x * b.y + a.y * b.x;
  return r;
}

template <typename T>
__device__ __forceinline__ cplx<T> cadd(cplx<T> a, cplx<T> b) {
  cplx<T> r;
  r.x = a.x + b.x;
  r.y = a.y + b.y;
  return r;
}

template <typename T>
__device__ __forceinline__ cplx<T> csub(cplx<T> a, cplx<T> b) {
  cplx<T> r;
  r.x = a.x - b.x;
  r.y = a.y - b.y;
  return r;
}

template <typename T>
__host__ __device__ __forceinline__ cplx<T> mk(T x, T y) {
  cplx<T> r;
  r.x = x;
  r.y = y;
  return r;
}

// One radix-R (R = 2 or 4) Stockham autosort stage over `count` contiguous transforms
// of length 2^logL held in LDS.  Ns = 2^logNs is the length of the sub-transforms
// already formed.  All reads of the stage complete before any write (in place).
template <typename T, int R, int NB>
__device__ __forceinline__ void stockham_stage(cplx<T>* buf, int logL, int count, int logNs,
                                               const cplx<T>* __restrict__ tw) {
  constexpr int logR = (R == 4) ? 2 : 1;
  const int logNb = logL - logR;
  const int nb = 1 << logNb;  // butterflies per transform
  const int total = count << logNb;
  const int Ns = 1 << logNs;
  const int tshift = kLdsMaxLog - (logNs + logR);
  cplx<T> v[NB][R];
  int dst[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = threadIdx.x + i * blockDim.x;
    dst[i] = -1;
    if (b < total) {
      const int t = b >> logNb;
      const int j = b & (nb - 1);
      const cplx<T>* base = buf + (t << logL);
#pragma unroll
      for (int r = 0; r < R; ++r) v[i][r] = base[j + r * nb];
      const int jm = j & (Ns - 1);
#pragma unroll
      for (int r = 1; r < R; ++r) {
        v[i][r] = cmul<T>(v[i][r], tw[(jm * r) << tshift]);
      }
      if (R == 2) {
        cplx<T> a = v[i][0], c = v[i][1];
        v[i][0] = cadd<T>(a, c);
        v[i][1] = csub<T>(a, c);
      } else {
        cplx<T> t0 = cadd<T>(v[i][0], v[i][2]);
        cplx<T> t1 = csub<T>(v[i][0], v[i][2]);
        cplx<T> t2 = cadd<T>(v[i][1], v[i][3]);
        cplx<T> d = csub<T>(v[i][1], v[i][3]);
        cplx<T> t3 = mk<T>(d.y, -d.x);   // x -i
        v[i][0] = cadd<T>(t0, t2);
        v[i][2] = csub<T>(t0, t2);
        v[i][1] = cadd<T>(t1, t3);
        v[i][3] = csub<T>(t1, t3);
      }
      dst[i] = (t << logL) + ((j >> logNs) << (logNs + logR)) + jm;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    if (dst[i] >= 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) buf[dst[i] + r * Ns] = v[i][r];
    }
  }
  __syncthreads();
}

// `count` in-place FFTs of length 2^logL in LDS (count << logL <= 4 * NB * blockDim.x).
template <typename T, int NB>
__device__ void lds_fft(cplx<T>* buf, int logL, int count, const cplx<T>* __restrict__ tw) {
  int logNs = 0;
  if (logL & 1) {
    stockham_stage<T, 2, 2 * NB>(buf, logL, count, 0, tw);
    logNs = 1;
  }
  for (; logNs < logL; logNs += 2) stockham_stage<T, 4, NB>(buf, logL, count, logNs, tw);
}


// Whole transforms of length M = 2^logM <= kLdsMax: tile = (first pair, count); the
// pairs of a tile have the same M and adjacent work slots.
template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_fft_lds(cplx<T>* __restrict__ data, const PairDesc* __restrict__ pd,
                                                        const int2* __restrict__ tiles,
                                                        const cplx<T>* __restrict__ tw) {
  __shared__ cplx<T> buf[kLdsMax];
  const int2 tile = tiles[blockIdx.x];
  const PairDesc& d = pd[tile.x];
  const int logM = d.logM;
  const int n = tile.y << logM;
  cplx<T>* g = data + d.work;
  for (int e = threadIdx.x; e < n; e += blockDim.x) buf[e] = g[e];
  __syncthreads();
  lds_fft<T, 4>(buf, logM, tile.y, tw);
  for (int e = threadIdx.x; e < n; e += blockDim.x) g[e] = buf[e];
}

template <typename T>
__device__ __forceinline__ cplx<T> tw4(const cplx<T>* __restrict__ hi, const cplx<T>* __restrict__ lo,
                                       int shift, int64_t t) {
  return cmul<T>(hi[t >> shift], lo[t & ((1 << shift) - 1)]);
}

// Four-step, pass 1: columns n2 of x[M2 n1 + n2], FFT over n1 (length M1), twiddle
// W_M^(n2 k1), store tmp[k1 M2 + n2].  tile = (pair, column block of W).
template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_fft4_cols(const cplx<T>* __restrict__ x, cplx<T>* __restrict__ tmp,
                                                          const PairDesc* __restrict__ pd,
                                                          const int2* __restrict__ tiles,
                                                          const cplx<T>* __restrict__ tw) {
  __shared__ cplx<T> buf[kLdsMax];
  constexpr int pi = prec_index<T>();
  const int2 tile = tiles[blockIdx.x];
  const PairDesc& d = pd[tile.x];
  const int logM1 = d.logM1, logM2 = d.logM2;
  const int M1 = 1 << logM1;
  const int logW = min(kLdsMaxLog - logM1, logM2);
  const int W = 1 << logW;
  const int c0 = tile.y << logW;
  const cplx<T>* xs = x + d.work;
  cplx<T>* ts = tmp + d.work;
  const cplx<T>* thi = (const cplx<T>*)d.thi[pi];
  const cplx<T>* tlo = (const cplx<T>*)d.tlo[pi];
  const int n = M1 << logW;
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const int w = e & (W - 1), n1 = e >> logW;
    buf[(w << logM1) + n1] = xs[((int64_t)n1 << logM2) + c0 + w];
  }
  __syncthreads();
  lds_fft<T, 4>(buf, logM1, W, tw);
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const int w = e & (W - 1), k1 = e >> logW;
    const int64_t t = (int64_t)(c0 + w) * k1;
    ts[((int64_t)k1 << logM2) + c0 + w] = cmul<T>(buf[(w << logM1) + k1], tw4<T>(thi, tlo, d.tw_shift, t));
  }
}

// Four-step, pass 2: rows k1 of tmp, FFT over n2 (length M2), store X[k1 + M1 k2].
// tile = (pair, row block of W).
template <typename T>
__global__ __launch_bounds__(kFftThreads) void k_fft4_rows(const cplx<T>* __restrict__ tmp, cplx<T>* __restrict__ x,
                                                          const PairDesc* __restrict__ pd,
                                                          const int2* __restrict__ tiles,
                                                          const cplx<T>* __restrict__ tw) {
  __shared__ cplx<T> buf[kLdsMax];
  const int2 tile = tiles[blockIdx.x];
  const PairDesc& d = pd[tile.x];
  const int logM1 = d.logM1, logM2 = d.logM2;
  const int M2 = 1 << logM2;
  const int logW = min(kLdsMaxLog - logM2, logM1);
  const int W = 1 << logW;
  const int r0 = tile.y << logW;
  const cplx<T>* ts = tmp + d.work + ((int64_t)r0 << logM2);
  cplx<T>* xs = x + d.work;
  const int n = M2 << logW;
  for (int e = threadIdx.x; e < n; e += blockDim.x) buf[e] = ts[e];
  __syncthreads();
  lds_fft<T, 4>(buf, logM2, W, tw);
  for (int e = threadIdx.x; e < n; e += blockDim.x) {
    const int w = e & (W - 1), k2 = e >> logW;
    xs[r0 + w + ((int64_t)k2 << logM1)] = buf[(w << logM2) + k2];
  }
}

// FFTs of length M over every pair of the set, in place in `data` (tmp: four-step
// intermediate).
template <typename T>
static hipError_t fft_set(const birk_plan* p, const PairSet& ps, cplx<T>* data, cplx<T>* tmp, hipStream_t s) {
  const cplx<T>* tw = (const cplx<T>*)p->lds_tw[prec_index<T>()];
  if (ps.n_lds > 0)
    hipLaunchKernelGGL(k_fft_lds<T>, dim3(ps.n_lds), dim3(kFftThreads), 0, s, data, ps.dev, ps.tiles_lds, tw);
  if (ps.n_c4 > 0) {
    hipLaunchKernelGGL(k_fft4_cols<T>, dim3(ps.n_c4), dim3(kFftThreads), 0, s, data, tmp, ps.dev, ps.tiles_c4, tw);
    hipLaunchKernelGGL(k_fft4_rows<T>, dim3(ps.n_r4), dim3(kFftThreads), 0, s, tmp, data, ps.dev, ps.tiles_r4, tw);
  }
  return hipGetLastError();
}

// ----------------------------------------------------------------- DCT-I plumbing

// Pack components (2p, 2p+1) into the even extension of length L = M, optionally
// doubling the end points (the E^{-1} pre-factor of the transpose).  tile = (pair, block
// over M).
template <typename T>
__global__ __launch_bounds__(256) void k_pack(const T* __restrict__ x, cplx<T>* __restrict__ z,
                                              const PairDesc* __restrict__ pd, const int2* __restrict__ tiles,
                                              int ends2) {
  const int2 tile = tiles[blockIdx.x];
  const PairDesc& d = pd[tile.x];
  const int64_t n = (int64_t)tile.y * blockDim.x + threadIdx.x;
  if (n >= d.M) return;
  const int64_t N = d.N;
  const int64_t k = n <= N ? n : d.L - n;
  const T* xa = x + d.src;
  T a = xa[k];
  T b = d.has2 ? xa[d.Nn + k] : T(0);
  if (ends2 && (k == 0 || k == N)) {
    a = a + a;
    b = b + b;
  }
  z[d.work + n] = mk<T>(a, b);
}

// Forward mid stage.  From Y = DFT(even ext of v) (so C v = Y/2), form the Chebyshev
// coefficients a_k = (-1)^k e_k Y_k / N (Fastv2a), the integrated coefficients c^_k
// (eq:c_k=bydef with the alias of eq:chatk=), and d_k = (-1)^k c^_k / e_k, the input of
// Fasta2v's DCT.  Writes d into the packed even extension for the second transform,
// except d_0, which needs c^_0, a reduction over all k; partial sums of
//     c^_0 = (1/N) [ e_0 Y_0 + Y_1 / 4 - sum_{k>=2} e_k Y_k / (k^2 - 1) ]
// go to the pair's partials (double, two per block).  tile = (pair, block over N_n).
template <typename T>
__global__ __launch_bounds__(256) void k_mid_fwd(const cplx<T>* __restrict__ z, cplx<T>* __restrict__ z2,
                                                 const PairDesc* __restrict__ pd, const int2* __restrict__ tiles,
                                                 double* __restrict__ part) {
  const int2 tile = tiles[blockIdx.x];
  const PairDesc& d = pd[tile.x];
  const int N = (int)d.N, L = (int)d.L;
  const cplx<T>* zz = z + d.work;
  cplx<T>* z2p = z2 + d.work;
  const int k = tile.y * (int)blockDim.x + (int)threadIdx.x;
  double s0 = 0.0, s1 = 0.0;
  if (k <= N) {
    const cplx<T> Yk = zz[k];
    const double c = c0_weight(k, N);
    s0 = c * (double)Yk.x;
    s1 = c * (double)Yk.y;
    if (k >= 1) {
      const cplx<T> dv = mid_fwd<T>(k, N, zz[k - 1], zz[min(k + 1, N)], T(1) / T(N), T(1) / T(4 * (int64_t)N + 4));
      z2p[k] = dv;
      if (k < N) z2p[L - k] = dv;
    }
  }
  // block reduction of the c^_0 partials, fixed order
  __shared__ double r0[256], r1[256];
  r0[threadIdx.x] = s0;
  r1[threadIdx.x] = s1;
  __syncthreads();
  for (int st = blockDim.x / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
      r0[threadIdx.x] += r0[threadIdx.x + st];
      r1[threadIdx.x] += r1[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[d.part + 2 * tile.y + 0] = r0[0];
    part[d.part + 2 * tile.y + 1] = r1[0];
  }
}

// d_0 = 2 c^_0 from the partials: one block per pair, fixed-order tree reduction.
template <typename T>
__global__ __launch_bounds__(256) void k_c0(const double* __restrict__ part, cplx<T>* __restrict__ z2,
                                            const PairDesc* __restrict__ pd) {
  const PairDesc& d = pd[blockIdx.x];
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < d.nblk; i += blockDim.x) {
    a += part[d.part + 2 * i + 0];
    b += part[d.part + 2 * i + 1];
  }
  __shared__ double ra[256], rb[256];
  ra[threadIdx.x] = a;
  rb[threadIdx.x] = b;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) {
      ra[threadIdx.x] += ra[threadIdx.x + st];
      rb[threadIdx.x] += rb[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double s = 2.0 / (double)d.N;
    z2[d.work] = mk<T>((T)(ra[0] * s), (T)(rb[0] * s));
  }
}

// Transpose mid stage.  p = C E^{-1} g = Y / 2; q = S M^T S p, i.e.
//   q_0 = p_0 - p_1,   q_1 = (p_0 - p_2) / 4,
//   q_j = -p_0/(j^2-1) + p_{j-1} (1/(2(j-1)) - [j = N]/(2(N+1))) - [j < N] p_{j+1}/(2(j+1)).
template <typename T>
__global__ __launch_bounds__(256) void k_mid_tr(const cplx<T>* __restrict__ z, cplx<T>* __restrict__ z2,
                                                const PairDesc* __restrict__ pd, const int2* __restrict__ tiles) {
  const int2 tile = tiles[blockIdx.x];
  const PairDesc& d = pd[tile.x];
  const int N = (int)d.N, L = (int)d.L;
  const cplx<T>* zz = z + d.work;
  cplx<T>* z2p = z2 + d.work;
  const int j = tile.y * (int)blockDim.x + (int)threadIdx.x;
  if (j > N) return;
  const cplx<T> q =
      mid_tr<T>(j, N, zz[0], zz[max(j - 1, 0)], zz[min(j + 1, N)], T(1) / T(2 * (int64_t)N + 2));
  z2p[j] = q;
  if (j >= 1 && j < N) z2p[L - j] = q;
}

// Final stage: out_j = scale_j * Y_j for j in [0, N], unpacking the pair.
// forward: scale = 1/2; transpose: scale = e_j / N.  tile = (pair, block over N_n).
template <typename T>
__global__ __launch_bounds__(256) void k_final(const cplx<T>* __restrict__ z, T* __restrict__ out,
                                               const PairDesc* __restrict__ pd, const int2* __restrict__ tiles,
                                               int transpose) {
  const int2 tile = tiles[blockIdx.x];
  const PairDesc& d = pd[tile.x];
  const int64_t N = d.N;
  const int64_t j = (int64_t)tile.y * blockDim.x + threadIdx.x;
  if (j > N) return;
  const cplx<T> Y = z[d.work + j];
  T sc;
  if (transpose) sc = ((j == 0 || j == N) ? T(0.5) : T(1)) / T(N);
  else sc = T(0.5);
  T* o = out + d.src;
  o[j] = Y.x * sc;
  if (d.has2) o[d.Nn + j] = Y.y * sc;
}

// Product over a set with L = 2N a power of two: pack, FFT (= DCT-I, unnormalised), stencil
// and c^_0, FFT, unpack.
template <typename T>
static hipError_t product_set(birk_plan* p, const PairSet& ps, const T* v, T* out, int transpose, hipStream_t s) {
  if (ps.host.empty()) return hipSuccess;
  cplx<T>* z = (cplx<T>*)p->work[0];
  cplx<T>* z2 = (cplx<T>*)p->work[1];
  cplx<T>* tmp = (cplx<T>*)p->work[2];
  hipLaunchKernelGGL(k_pack<T>, dim3(ps.n_m), dim3(256), 0, s, v, z, ps.dev, ps.tiles_m, transpose);
  hipError_t e = fft_set<T>(p, ps, z, tmp, s);
  if (e != hipSuccess) return e;
  if (!transpose) {
    hipLaunchKernelGGL(k_mid_fwd<T>, dim3(ps.n_n), dim3(256), 0, s, z, z2, ps.dev, ps.tiles_n, p->partials);
    hipLaunchKernelGGL(k_c0<T>, dim3((unsigned)ps.host.size()), dim3(256), 0, s, p->partials, z2, ps.dev);
  } else {
    hipLaunchKernelGGL(k_mid_tr<T>, dim3(ps.n_n), dim3(256), 0, s, z, z2, ps.dev, ps.tiles_n);
  }
  e = fft_set<T>(p, ps, z2, tmp, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_final<T>, dim3(ps.n_n), dim3(256), 0, s, z2, out, ps.dev, ps.tiles_n, transpose);
  return hipGetLastError();
}

template <typename T>
hipError_t apply_product(birk_plan* p, const T* v, T* out, int transpose, hipStream_t s) {
  for (const FastGroup& g : p->fgroups) {
    hipError_t e = fast_product<T>(p, g, v, out, transpose, s);
    if (e != hipSuccess) return e;
  }
  hipError_t e = product_lds<T>(p, v, out, transpose, s);
  if (e == hipSuccess) e = product_set<T>(p, p->gen[0], v, out, transpose, s);
  if (e == hipSuccess) e = product_blu<T>(p, p->gen[1], v, out, transpose, s);
  return e;
}

template hipError_t apply_product<double>(birk_plan*, const double*, double*, int, hipStream_t);
template hipError_t apply_product<float>(birk_plan*, const float*, float*, int, hipStream_t);
template hipError_t apply_product<df32>(birk_plan*, const df32*, df32*, int, hipStream_t);

// ----------------------------------------------------------------- tables

// exp(-i pi num / den) in double.  The angle is reduced exactly in integers and folded
// into [0, pi/4] before the library sin/cos, so each entry is correctly rounded to
// within about one ulp.
static void expi_pi(int64_t num, int64_t den, double* c, double* s) {
  // theta = pi * m / den with m in [0, 2 den); work with numerators over 4 den so that
  // the octant boundaries are integers.
  int64_t m = num % (2 * den);
  if (m < 0) m += 2 * den;
  int64_t q = 4 * m;            // theta = pi * q / (4 den), q in [0, 8 den)
  const int64_t D = 4 * den;    // pi  <-> D
  double sgn_c = 1.0, sgn_s = 1.0;
  if (q >= D) { q -= D; sgn_c = -sgn_c; sgn_s = -sgn_s; }          // theta - pi
  bool swap = false;
  if (2 * q > D) { q = D - q; sgn_c = -sgn_c; }                     // pi - theta
  if (4 * q > D) { q = D / 2 - q; swap = true; }                    // pi/2 - theta (D even)
  const double th = M_PI * (double)q / (double)D;
  double cs = std::cos(th), sn = std::sin(th);
  if (q == 0) { cs = 1.0; sn = 0.0; }
  if (swap) { const double t = cs; cs = sn; sn = t; }
  *c = sgn_c * cs;
  *s = -(sgn_s * sn);
}

hipError_t upload_raw(birk_plan* p, const void* h, size_t bytes, void** d) {
  *d = nullptr;
  hipError_t e = hipMalloc(d, std::max<size_t>(bytes, 16));
  if (e != hipSuccess) return e;
  p->allocs.push_back(*d);
  return hipMemcpy(*d, h, bytes, hipMemcpyHostToDevice);
}

template <typename T>
static hipError_t upload_cplx(birk_plan* p, const std::vector<double>& re, const std::vector<double>& im,
                              const void** dptr) {
  const size_t n = re.size();
  std::vector<cplx<T>> h(n);
  for (size_t i = 0; i < n; ++i) h[i] = mk<T>((T)re[i], (T)im[i]);
  void* d = nullptr;
  hipError_t e = upload_raw(p, h.data(), n * sizeof(cplx<T>), &d);
  *dptr = d;
  return e;
}

// One table in double and in the plan's own precision.
static hipError_t upload_all(birk_plan* p, const std::vector<double>& re, const std::vector<double>& im,
                             const void** dst) {
  hipError_t e = upload_cplx<double>(p, re, im, &dst[0]);
  if (e == hipSuccess && (p->prec == BIRK_F32 || p->prec == BIRK_F32_REFINE_F64))
    e = upload_cplx<float>(p, re, im, &dst[1]);
  if (e == hipSuccess && p->prec == BIRK_DF32) e = upload_cplx<df32>(p, re, im, &dst[2]);
  return e;
}

// Filter of the one-workgroup convolutions (length M >= 3N, see birk_lds.hip): conj(chirp)
// at lags 0..N at m = lag, lags -1..-(L - 1) at m = M + lag, zero between; the chirp has
// period L and is even, so its first N + 1 values give every lag.
template <typename T>
__global__ void k_build_filter(cplx<T>* __restrict__ b, const cplx<T>* __restrict__ chirp, int64_t L,
                               int64_t M) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= M) return;
  cplx<T> v = mk<T>(T(0), T(0));
  const int64_t lag = m <= L / 2 ? m : M - m;
  if (lag < L) {
    v = chirp[lag <= L / 2 ? lag : L - lag];
    v.y = -v.y;
  }
  b[m] = v;
}

// dst = s src
template <typename T>
__global__ void k_scale_to(const cplx<double>* __restrict__ src, cplx<T>* __restrict__ dst, int64_t M, double s) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m < M) dst[m] = mk<T>((T)(src[m].x * s), (T)(src[m].y * s));
}

static int ilog2_ceil(int64_t x) {
  int l = 0;
  while ((int64_t(1) << l) < x) ++l;
  return l;
}

// Twiddle tables of length M (1, 3 or 5 times a power of two): W^t = hi[t >> shift] lo[...].
static int tw_shift_of(int64_t M) { return std::min((ilog2_ceil(M) + 1) / 2, __builtin_ctzll(M)); }

static PairDesc make_pair(const birk_plan* p, int64_t src, int64_t Nn, int has2) {
  PairDesc d;
  d.src = src;
  d.Nn = Nn;
  d.N = Nn - 1;
  d.L = 2 * d.N;
  const bool pow2 = (d.L & (d.L - 1)) == 0 && d.L >= 8;   // the shortest compiled transform
  d.M = pow2 ? d.L : (int64_t(1) << ilog2_ceil(d.N + d.L));
  d.logM = ilog2_ceil(d.M);
  d.slot = d.L == 4 ? 4 : d.M;
  d.cls = d.logM;
  if (d.logM > kLdsMaxLog) {
    if (pow2) {
      d.logM1 = (d.logM + 1) / 2;
      d.logM2 = d.logM - d.logM1;
    } else {
      blu_length(d, p->prec);
      blu_set_split(d, p->blu_split && blu_split_ok(d, p->blu_split) ? p->blu_split : blu_default_split(d));
    }
    d.tw_shift = tw_shift_of(d.M);
  }
  d.has2 = has2;
  d.nblk = (int)((Nn + 255) / 256);
  return d;
}

// Sort the pairs by M, then give each its work slot and partials.
static void layout_set(PairSet& ps, int64_t& woff, int64_t& poff) {
  std::stable_sort(ps.host.begin(), ps.host.end(),
                   [](const PairDesc& a, const PairDesc& b) { return a.M < b.M; });
  ps.work = 0;
  ps.parts = 0;
  for (PairDesc& d : ps.host) {
    d.work = woff;
    woff += d.slot;
    ps.work += d.slot;
    d.part = poff;
    poff += 2 * (int64_t)d.nblk;
    ps.parts += 2 * (int64_t)d.nblk;
  }
}

// Longest power-of-two N whose products run in one workgroup's LDS, a component each
// (birk_lds.hip).  Up to there one launch that reads v and writes out once beats the three
// passes and their two intermediate arrays at every batch size (N = 512 / 1024 / 2048, three
// passes against one launch: 25 / 26 / 30 us against 6.9 / 8.7 / 10.4 at six components in
// double, 379 / 528 / 854 against 140 / 167 / 353 at 16386; double-float at 2048 62 against 36
// and 1520 against 1197).
constexpr int64_t kLdsMaxN = kLdsMax / 2;

void plan_products(birk_plan* p) {
  p->fgroups.clear();
  for (int k = 0; k < 2; ++k) {
    p->gen[k] = PairSet();
    p->lds[k] = LdsSet();
  }
  p->lds_even = LdsSet();
  p->noalloc_nbuf = 2;
  int64_t woff = 0, poff = 0;
  const int B = (int)p->inst.size();
  for (int i = 0; i < B;) {
    const Instance& in = p->inst[i];
    if (p->use_fast && fast_eligible(in.N)) {
      FastGroup g;
      g.Nn = in.Nn;
      g.N = in.N;
      g.off = in.off;
      g.kn = p->fast_kn;
      int j = i;
      while (j < B && p->inst[j].N == in.N) g.nc += p->inst[j++].nx;
      int64_t fw = 0, fp = 0;
      fast_sizes(p, g.N, g.nc, &fw, &fp);
      if (g.N <= kLdsMaxN) {
        // no workspace used; the plan's size (what birk_apply_noalloc accepts) counts it
        // as for the three-pass groups
        PairDesc d;
        d.Nn = g.Nn;
        d.N = g.N;
        d.logM = ilog2_ceil(g.N);
        for (int c = 0; c < g.nc; ++c) {
          d.src = g.off + (int64_t)c * g.Nn;
          p->lds_even.host.push_back(d);
        }
        i = j;
        woff += fw;
        poff += fp;
        continue;
      }
      g.work_off = woff;
      g.part_off = poff;
      woff += fw;
      poff += fp;
      p->fgroups.push_back(g);
      i = j;
      continue;
    }
    const int np = (in.nx + 1) / 2;
    for (int q = 0; q < np; ++q) {
      PairDesc d = make_pair(p, in.off + 2 * (int64_t)q * in.Nn, in.Nn, 2 * q + 1 < in.nx);
      const int chirp = d.L == d.slot && d.L > 4 ? 0 : 1;
      p->noalloc_nbuf = 3;
      if (d.cls > kLdsMaxLog) {
        p->gen[chirp].host.push_back(d);
        continue;
      }
      // whole product in LDS: a work slot only for the filter's set-up at plan creation
      // (and in the plan's size)
      d.work = woff;
      woff += d.slot;
      poff += 2 * (int64_t)d.nblk;
      p->lds[chirp].host.push_back(d);
    }
    ++i;
  }
  layout_set(p->gen[0], woff, poff);
  layout_set(p->gen[1], woff, poff);
  p->total_work = woff;
  p->total_part = poff;
}

// Tile lists of a set (see PairSet), uploaded with the descriptors.
static hipError_t finalize_set(birk_plan* p, PairSet& ps) {
  std::vector<int2> tm, tn, tl, tc, tr;
  const int np = (int)ps.host.size();
  for (int q = 0; q < np; ++q) {
    const PairDesc& d = ps.host[q];
    for (int64_t b = 0; b < (d.M + 255) / 256; ++b) tm.push_back(make_int2(q, (int)b));
    for (int b = 0; b < d.nblk; ++b) tn.push_back(make_int2(q, b));
    if (d.logM > kLdsMaxLog) {
      const int logW1 = std::min(kLdsMaxLog - d.logM1, d.logM2);
      const int logW2 = std::min(kLdsMaxLog - d.logM2, d.logM1);
      for (int b = 0; b < (1 << (d.logM2 - logW1)); ++b) tc.push_back(make_int2(q, b));
      for (int b = 0; b < (1 << (d.logM1 - logW2)); ++b) tr.push_back(make_int2(q, b));
    }
  }
  for (int q = 0; q < np;) {
    const PairDesc& d = ps.host[q];
    if (d.logM > kLdsMaxLog) {
      ++q;
      continue;
    }
    const int per = kLdsMax >> d.logM;
    int cnt = 1;
    while (q + cnt < np && cnt < per && ps.host[q + cnt].M == d.M && ps.host[q + cnt].work == d.work + cnt * d.M)
      ++cnt;
    tl.push_back(make_int2(q, cnt));
    q += cnt;
  }
  ps.n_m = (int)tm.size();
  ps.n_n = (int)tn.size();
  ps.n_lds = (int)tl.size();
  ps.n_c4 = (int)tc.size();
  ps.n_r4 = (int)tr.size();
  void* d = nullptr;
  hipError_t e = upload_raw(p, ps.host.data(), ps.host.size() * sizeof(PairDesc), &d);
  ps.dev = (PairDesc*)d;
  auto up = [&](const std::vector<int2>& v, int2** dst) {
    void* x = nullptr;
    if (e == hipSuccess) e = upload_raw(p, v.data(), v.size() * sizeof(int2), &x);
    *dst = (int2*)x;
  };
  up(tm, &ps.tiles_m);
  up(tn, &ps.tiles_n);
  up(tl, &ps.tiles_lds);
  up(tc, &ps.tiles_c4);
  up(tr, &ps.tiles_r4);
  return e;
}

// ----------------------------------------------------------------- general-path tuner
// The chirp convolutions of birk_blu.hip run their two-step FFTs with M = M1 M2.  Pairs
// whose 3N lies under the same power of two 2^m form a class (their M are 3/4, 1, 5/4 or
// 3/2 times it) and share a nominal M1 = 2^x (a pair's own M1 is 2^x, 3/4 2^x or
// 5/8 2^x).  For each class the tuner times the plan's product with every x the compiled
// kernels support for all of its pairs, one class at a time with the others fixed, and
// keeps the fastest (the current choice stays unless another is more than 2 % faster; it may
// differ between the pairs of a class, whose lengths do not all allow every x).  A change of
// split rebuilds the class's filter spectra in the new rows-pass order and the
// tile lists; the products change only in rounding order.
static hipError_t set_blu_split(birk_plan* p, int cls, const std::vector<int>& xs, hipStream_t s) {
  PairSet& ps = p->gen[1];
  hipError_t e = hipStreamSynchronize(s);   // the lists in use are freed below
  if (e != hipSuccess) return e;
  // the new lists are built next to the old ones, which stay if an allocation fails
  PairSet next = ps, fs;
  next.dev = nullptr;
  next.tiles_c4 = next.tiles_r4 = nullptr;
  std::vector<int64_t> seen;
  for (size_t q = 0; q < next.host.size(); ++q) {
    PairDesc& d = next.host[q];
    if (d.cls != cls) continue;
    blu_set_split(d, xs[q]);
    if (std::find(seen.begin(), seen.end(), d.N) != seen.end()) continue;
    seen.push_back(d.N);
    fs.host.push_back(d);
  }
  e = blu_lists(p, next);
  if (e == hipSuccess) e = blu_lists(p, fs);
  if (e == hipSuccess) e = blu_filters(p, fs, s);
  blu_free_lists(p, fs);
  if (e != hipSuccess) {
    blu_free_lists(p, next);
    return e;
  }
  blu_free_lists(p, ps);
  ps = next;
  return hipSuccess;
}

template <typename T>
static hipError_t tune_general_t(birk_plan* p, hipStream_t s, std::string* report) {
  std::vector<int> sizes;
  for (const PairDesc& d : p->gen[1].host)
    if (std::find(sizes.begin(), sizes.end(), d.cls) == sizes.end()) sizes.push_back(d.cls);
  if (sizes.empty()) {
    *report += "general path: no Bluestein sizes above the LDS limit\n";
    return hipSuccess;
  }
  T* in[2] = {(T*)p->tmp_vec[0], (T*)p->tmp_vec[2]};
  T* out[2] = {(T*)p->tmp_vec[1], (T*)p->tmp_vec[3]};
  hipError_t e = hipSuccess;
  for (int b = 0; b < 2 && e == hipSuccess; ++b) e = hipMemsetAsync(in[b], 0, (size_t)p->total_len * sizeof(T), s);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (e == hipSuccess) e = hipEventCreate(&e0);
  if (e == hipSuccess) e = hipEventCreate(&e1);
  auto time_product = [&](float* ms) -> hipError_t {
    hipError_t r = apply_product<T>(p, in[0], out[0], 0, s);
    float best = 0.0f;
    for (int round = 0; round < 2 && r == hipSuccess; ++round) {
      r = hipEventRecord(e0, s);
      for (int k = 0; k < 3 && r == hipSuccess; ++k) r = apply_product<T>(p, in[k & 1], out[k & 1], 0, s);
      if (r == hipSuccess) r = hipEventRecord(e1, s);
      if (r == hipSuccess) r = hipEventSynchronize(e1);
      float t = 0.0f;
      if (r == hipSuccess) r = hipEventElapsedTime(&t, e0, e1);
      if (round == 0 || t < best) best = t;
    }
    *ms = best / 3.0f;
    return r;
  };
  std::sort(sizes.begin(), sizes.end());
  char line[160];
  for (int cls : sizes) {
    if (e != hipSuccess) break;
    const size_t np = p->gen[1].host.size();
    std::vector<int> keep(np);   // every pair's split (those of the class are used)
    int cur = 0;                 // the class's last
    for (size_t q = 0; q < np; ++q) {
      keep[q] = blu_split(p->gen[1].host[q]);
      if (p->gen[1].host[q].cls == cls) cur = keep[q];
    }
    std::vector<int> chosen = keep;
    float best_ms = 0.0f;
    if ((e = time_product(&best_ms)) != hipSuccess) break;
    snprintf(line, sizeof line, "general path M=2^%d: [M1 2^%d] %.1f us;", cls, cur, 1000.0 * best_ms);
    *report += line;
    int best = cur;
    for (int x = 7; x <= kLdsMaxLog && e == hipSuccess; ++x) {
      bool ok = true, same = true;
      for (const PairDesc& d : p->gen[1].host) {
        if (d.cls != cls) continue;
        ok = ok && blu_split_ok(d, x);
        same = same && keep[&d - p->gen[1].host.data()] == x;
      }
      if (!ok || same) continue;
      const std::vector<int> all(np, x);
      if ((e = set_blu_split(p, cls, all, s)) != hipSuccess) break;
      float ms = 0.0f;
      if ((e = time_product(&ms)) != hipSuccess) break;
      snprintf(line, sizeof line, " [M1 2^%d] %.1f us;", x, 1000.0 * ms);
      *report += line;
      if (ms < best_ms * (1.0f - 0.02f)) {
        best_ms = ms;
        best = x;
        chosen = all;
      }
    }
    if (e == hipSuccess) e = set_blu_split(p, cls, chosen, s);
    snprintf(line, sizeof line, " chosen [M1 2^%d]\n", best);
    *report += line;
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  return e;
}

hipError_t tune_general(birk_plan* p, hipStream_t s, std::string* report) {
  if (p->prec == BIRK_F64) return tune_general_t<double>(p, s, report);
  if (p->prec == BIRK_DF32) return tune_general_t<df32>(p, s, report);
  return tune_general_t<float>(p, s, report);
}

hipError_t build_tables(birk_plan* p) {
  hipError_t e;
  {
    std::vector<double> re(kLdsMax), im(kLdsMax);
    for (int t = 0; t < kLdsMax; ++t) expi_pi(2 * (int64_t)t, kLdsMax, &re[t], &im[t]);
    if ((e = upload_all(p, re, im, p->lds_tw)) != hipSuccess) return e;
  }
  // four-step twiddles, one set per transform length
  std::map<int64_t, TwiddleSet> twsets;
  auto twiddles = [&](int64_t M, TwiddleSet* out) -> hipError_t {
    auto it = twsets.find(M);
    if (it != twsets.end()) {
      *out = it->second;
      return hipSuccess;
    }
    TwiddleSet ts;
    ts.shift = tw_shift_of(M);
    const int64_t nlo = (int64_t)1 << ts.shift, nhi = M >> ts.shift;
    std::vector<double> re(nlo), im(nlo);
    for (int64_t t = 0; t < nlo; ++t) expi_pi(2 * t, M, &re[t], &im[t]);
    hipError_t err = upload_all(p, re, im, ts.lo);
    re.assign(nhi, 0.0);
    im.assign(nhi, 0.0);
    for (int64_t t = 0; t < nhi; ++t) expi_pi(2 * (t << ts.shift), M, &re[t], &im[t]);
    if (err == hipSuccess) err = upload_all(p, re, im, ts.hi);
    twsets[M] = ts;
    *out = ts;
    return err;
  };
  for (FastGroup& g : p->fgroups)
    if ((e = twiddles(2 * g.N, &g.tw)) != hipSuccess) return e;
  for (int k = 0; k < 2; ++k)
    for (PairDesc& d : p->gen[k].host)
      if (d.cls > kLdsMaxLog) {
        TwiddleSet ts;
        if ((e = twiddles(d.M, &ts)) != hipSuccess) return e;
        for (int pi = 0; pi < kNumPrec; ++pi) {
          d.thi[pi] = ts.hi[pi];
          d.tlo[pi] = ts.lo[pi];
        }
      }
  // chirp (N + 1 values) and filter spectrum, one per distinct N: the spectrum of the plain
  // convolution for one-workgroup pairs, of the even one for the others
  struct Blue {
    const void* chirp[kNumPrec] = {nullptr, nullptr, nullptr};
    void* filt[kNumPrec] = {nullptr, nullptr, nullptr};
  };
  std::map<int64_t, Blue> blue;
  std::vector<PairDesc*> chirped;
  for (PairDesc& d : p->gen[1].host) chirped.push_back(&d);
  for (PairDesc& d : p->lds[1].host) chirped.push_back(&d);
  PairSet small, large;  // one pair per distinct N
  for (PairDesc* dp : chirped) {
    PairDesc& d = *dp;
    const bool is_large = d.cls > kLdsMaxLog;
    auto it = blue.find(d.N);
    if (it == blue.end()) {
      Blue b;
      std::vector<double> re(d.Nn), im(d.Nn);
      for (int64_t n = 0; n <= d.N; ++n) expi_pi((int64_t)(((__int128)n * n) % (2 * d.L)), d.L, &re[n], &im[n]);
      if ((e = upload_all(p, re, im, b.chirp)) != hipSuccess) return e;
      // M/2 + M2 values at the longest row of any split
      const int64_t len = is_large ? d.M / 2 + kLdsMax : d.M;
      for (int pi = 0; pi < kNumPrec; ++pi) {
        if (!b.chirp[pi]) continue;
        const size_t bytes[kNumPrec] = {sizeof(cplx<double>), sizeof(cplx<float>), sizeof(cplx<df32>)};
        if ((e = hipMalloc(&b.filt[pi], len * bytes[pi])) != hipSuccess) return e;
        p->allocs.push_back(b.filt[pi]);
      }
      it = blue.emplace(d.N, b).first;
      (is_large ? large : small).host.push_back(d);
    }
    for (int pi = 0; pi < kNumPrec; ++pi) {
      d.chirp[pi] = it->second.chirp[pi];
      d.filt[pi] = it->second.filt[pi];
    }
  }
  for (PairSet* fs : {&small, &large})
    for (PairDesc& f : fs->host)
      for (int pi = 0; pi < kNumPrec; ++pi) {
        f.chirp[pi] = blue[f.N].chirp[pi];
        f.filt[pi] = blue[f.N].filt[pi];
      }
  if (!small.host.empty()) {
    int64_t woff = 0, poff = 0;
    for (PairDesc& f : small.host) f.slot = f.M;
    layout_set(small, woff, poff);  // filter slots from the start of work[0]
    for (const PairDesc& f : small.host)
      hipLaunchKernelGGL(k_build_filter<double>, dim3((unsigned)((f.M + 255) / 256)), dim3(256), 0, p->stream,
                         (cplx<double>*)p->work[0] + f.work, (const cplx<double>*)f.chirp[0], f.L, f.M);
    if ((e = finalize_set(p, small)) != hipSuccess) return e;
    e = fft_set<double>(p, small, (cplx<double>*)p->work[0], (cplx<double>*)p->work[2], p->stream);
    if (e != hipSuccess) return e;
    for (const PairDesc& f : small.host) {
      const cplx<double>* bw = (const cplx<double>*)p->work[0] + f.work;
      const double s = 1.0 / (double)f.M;
      const dim3 grid((unsigned)((f.M + 255) / 256)), blk(256);
      hipLaunchKernelGGL(k_scale_to<double>, grid, blk, 0, p->stream, bw, (cplx<double>*)f.filt[0], f.M, s);
      if (f.filt[1])
        hipLaunchKernelGGL(k_scale_to<float>, grid, blk, 0, p->stream, bw, (cplx<float>*)f.filt[1], f.M, s);
      if (f.filt[2])
        hipLaunchKernelGGL(k_scale_to<df32>, grid, blk, 0, p->stream, bw, (cplx<df32>*)f.filt[2], f.M, s);
    }
    if ((e = hipStreamSynchronize(p->stream)) != hipSuccess) return e;
  }
  if (!large.host.empty()) {
    e = blu_lists(p, large);
    if (e == hipSuccess) e = blu_filters(p, large, p->stream);
    blu_free_lists(p, large);
    if (e == hipSuccess) e = blu_lists(p, p->gen[1]);
    if (e != hipSuccess) return e;
  }
  if (!p->gen[0].host.empty() && (e = finalize_set(p, p->gen[0])) != hipSuccess) return e;
  for (int k = 0; k < 2; ++k)
    if ((e = finalize_lds(p, p->lds[k])) != hipSuccess) return e;
  if ((e = finalize_lds_even(p, p->lds_even)) != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace birk
