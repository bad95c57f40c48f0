// Jacobian products, the Birkhoff preconditioner and the Krylov BLAS-1 kernels (gfx950).
//
// Preconditioner (arXiv 2509.01855, "Development of a Special Birkhoff-Centric
// Preconditioner"): P = I - B~^a J with B~^a lower triangular, w_j below the diagonal
// and w_j / 2 on it (w = CC weights).
//
//   P y:      y - B~^a (J y); B~^a u is an exclusive prefix sum of w u plus w u / 2
//             (FastBccV).  Three kernels: block sums, a scan of the block sums, and
//             the block-local scan.  Sums are carried in double.
//   P^{-1} y: exact block forward substitution (FastPinvY box, with its running-sum
//             update read as forward substitution):
//                 xi_k = K_k^{-1} (y_k + S_k),  K_k = I - w_k J_k / 2,
//                 S_{k+1} = S_k + w_k J_k xi_k.
//             As an affine map of the carried sum, S_{k+1} = G_k S_k + h_k with
//             G_k = I + w_k J_k K_k^{-1} and h_k = w_k J_k K_k^{-1} y_k.  The chain is
//             evaluated as a scan of affine maps S_out = A S_in + b: birk_scan.hip to
//             n_x = 8, birk_wide.hip to 12.

#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "birk_internal.h"

namespace birk {

// ------------------------------------------------------------------ P y (forward)
constexpr int kScanItems = 4;
constexpr int kScanBlock = 256 * kScanItems;

template <typename T>
__device__ __forceinline__ double wju(const double* __restrict__ J, int per_node, const T* __restrict__ y,
                                      const double* __restrict__ w, int r, int nx, int64_t Nn, int64_t k) {
  double acc = 0.0;
  for (int c = 0; c < nx; ++c) {
    const double j = per_node ? J[((int64_t)(r * nx + c)) * Nn + k] : J[r * nx + c];
    acc += j * (double)y[(int64_t)c * Nn + k];
  }
  return w[k] * acc;
}

__device__ __forceinline__ double block_sum256(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// P y = y - B~^a (J y) per component r: an exclusive prefix sum of u_k = w_k (J_k y_k)_r
// plus half the node's own term (B~^a: w_j below the diagonal, w_k / 2 on it).  Three
// launches: block sums over tiles of kScanBlock nodes, an exclusive scan of the block sums
// (one workgroup per component), and the final pass, which scans inside the tile.  Global
// accesses are coalesced (node k = tile base + i * 256 + thread); the final pass moves u
// through LDS to scan it in node order.  Double plans with n_x <= 16 form u once for all
// components (k_pfwd_sums_all, u kept in out); otherwise each component's passes rebuild
// their u_r from J and y.

// One workgroup per tile of kScanBlock nodes of one component of one instance, over the
// whole batch: tile = (instance, component * ntiles + tile index); the tile sums of
// (instance i, component r) sit at scan[scan_off(i) + r * ntiles(i) + tile].
__device__ __forceinline__ int pfwd_ntiles(int64_t Nn) { return (int)((Nn + kScanBlock - 1) / kScanBlock); }

template <typename T>
__global__ __launch_bounds__(256) void k_pfwd_sums(const int2* __restrict__ tiles, const InstDesc* __restrict__ idesc,
                                                   const double* __restrict__ J, int per_node,
                                                   const T* __restrict__ y, double* __restrict__ scan) {
  __shared__ double sh[256];
  const int2 t = tiles[blockIdx.x];
  const InstDesc d = idesc[t.x];
  const int nt = pfwd_ntiles(d.Nn);
  const int r = t.y / nt, b = t.y - r * nt;
  const double* Ji = J + (per_node ? d.joff : d.jcoff);
  const T* yi = y + d.off;
  const int64_t base = (int64_t)b * kScanBlock;
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + i * 256 + threadIdx.x;
    if (k < d.Nn) acc += wju<T>(Ji, per_node, yi, d.w, r, (int)d.nx, d.Nn, k);
  }
  const double s = block_sum256(acc, sh);
  if (threadIdx.x == 0) scan[d.scan_off + t.y] = s;
}

// Inclusive scan of v over the 256 threads of the workgroup (Hillis-Steele in LDS).
__device__ __forceinline__ double block_scan256(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int st = 1; st < 256; st <<= 1) {
    const double a = threadIdx.x >= st ? sh[threadIdx.x - st] : 0.0;
    __syncthreads();
    sh[threadIdx.x] += a;
    __syncthreads();
  }
  const double r = sh[threadIdx.x];
  __syncthreads();
  return r;
}

// Exclusive scan of the tile sums of one (instance, component) per workgroup, in chunks
// of 256.
__global__ __launch_bounds__(256) void k_pfwd_scanparts(const int2* __restrict__ pairs,
                                                        const InstDesc* __restrict__ idesc,
                                                        double* __restrict__ scan) {
  __shared__ double sh[256];
  __shared__ double total;
  const int2 q = pairs[blockIdx.x];
  const InstDesc d = idesc[q.x];
  const int nblk = pfwd_ntiles(d.Nn);
  double* pr = scan + d.scan_off + (int64_t)q.y * nblk;
  double carry = 0.0;
  for (int b0 = 0; b0 < nblk; b0 += 256) {
    const int b = b0 + (int)threadIdx.x;
    const double v = b < nblk ? pr[b] : 0.0;
    const double incl = block_scan256(v, sh);
    if (b < nblk) pr[b] = carry + incl - v;
    if (threadIdx.x == 255) total = incl;
    __syncthreads();
    carry += total;
    __syncthreads();
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_pfwd_final(const int2* __restrict__ tiles, const InstDesc* __restrict__ idesc,
                                                    const double* __restrict__ J, int per_node,
                                                    const T* __restrict__ y, const double* __restrict__ scan,
                                                    T* __restrict__ out) {
  __shared__ double su[kScanBlock];
  __shared__ double sh[256];
  const int2 t = tiles[blockIdx.x];
  const InstDesc d = idesc[t.x];
  const int nt = pfwd_ntiles(d.Nn);
  const int r = t.y / nt, b = t.y - r * nt;
  const double* Ji = J + (per_node ? d.joff : d.jcoff);
  const T* yi = y + d.off;
  const int64_t base = (int64_t)b * kScanBlock;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + i * 256 + threadIdx.x;
    su[i * 256 + threadIdx.x] = (k < d.Nn) ? wju<T>(Ji, per_node, yi, d.w, r, (int)d.nx, d.Nn, k) : 0.0;
  }
  __syncthreads();
  // thread t scans nodes base + kScanItems t + j, j < kScanItems, in order
  double u[kScanItems];
  double tsum = 0.0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    u[j] = su[threadIdx.x * kScanItems + j];
    tsum += u[j];
  }
  double run = scan[d.scan_off + t.y] + block_scan256(tsum, sh) - tsum;
  // each thread rewrites only the entries it read itself
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    su[threadIdx.x * kScanItems + j] = run + 0.5 * u[j];
    run += u[j];
  }
  __syncthreads();
  T* oi = out + d.off + (int64_t)r * d.Nn;
  const T* yr = yi + (int64_t)r * d.Nn;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + i * 256 + threadIdx.x;
    if (k < d.Nn) oi[k] = (T)((double)yr[k] - su[i * 256 + threadIdx.x]);
  }
}

// Double plans with n_x <= 16: one workgroup per tile forms u_k = w_k J_k y_k for all
// components (J and y read once), stores u in out (which does not overlap y) and sums it
// per component; the final pass of component r then reads u_r back instead of J and all
// of y.  Tile = (instance, tile); the sums go where k_pfwd_sums puts them.  NXC > 0: every
// instance has n_x = NXC, so the loops unroll completely and a node's J and y loads issue
// together.
template <int MAXNX, int NXC = 0>
__global__ __launch_bounds__(256) void k_pfwd_sums_all(const int2* __restrict__ tiles,
                                                       const InstDesc* __restrict__ idesc,
                                                       const double* __restrict__ J, int per_node,
                                                       const double* __restrict__ y, double* __restrict__ u,
                                                       double* __restrict__ scan) {
  __shared__ double sh[4][MAXNX];
  const int2 t = tiles[blockIdx.x];
  const InstDesc d = idesc[t.x];
  const int nt = pfwd_ntiles(d.Nn), b = t.y, nx = NXC > 0 ? NXC : (int)d.nx;
  const int64_t Nn = d.Nn;
  const double* Ji = J + (per_node ? d.joff : d.jcoff);
  const double* yi = y + d.off;
  double* ui = u + d.off;
  const int64_t base = (int64_t)b * kScanBlock;
  double acc[MAXNX];
#pragma unroll
  for (int r = 0; r < MAXNX; ++r) acc[r] = 0.0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + i * 256 + threadIdx.x;
    if (k >= Nn) break;
    double yv[MAXNX];
#pragma unroll
    for (int c = 0; c < MAXNX; ++c) yv[c] = c < nx ? yi[(int64_t)c * Nn + k] : 0.0;
    const double wk = d.w[k];
#pragma unroll
    for (int r = 0; r < MAXNX; ++r) {
      if (r >= nx) break;
      double a = 0.0;
#pragma unroll
      for (int c = 0; c < MAXNX; ++c) {
        if (c >= nx) break;
        a += (per_node ? Ji[(int64_t)(r * nx + c) * Nn + k] : Ji[r * nx + c]) * yv[c];
      }
      a *= wk;
      ui[(int64_t)r * Nn + k] = a;
      acc[r] += a;
    }
  }
  const int w = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63);
#pragma unroll
  for (int r = 0; r < MAXNX; ++r) {
    if (r >= nx) break;
    double v = acc[r];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (l == 0) sh[w][r] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < nx) {
    const int r = (int)threadIdx.x;
    scan[d.scan_off + (int64_t)r * nt + b] = ((sh[0][r] + sh[1][r]) + sh[2][r]) + sh[3][r];
  }
}

// Final pass of component r from u_r held in out (in place: a workgroup reads its tile of
// u_r before it writes the same elements of out).
__global__ __launch_bounds__(256) void k_pfwd_final_u(const int2* __restrict__ tiles, const InstDesc* __restrict__ idesc,
                                                      const double* __restrict__ y, const double* __restrict__ scan,
                                                      double* __restrict__ out) {
  __shared__ double su[kScanBlock];
  __shared__ double sh[256];
  const int2 t = tiles[blockIdx.x];
  const InstDesc d = idesc[t.x];
  const int nt = pfwd_ntiles(d.Nn);
  const int r = t.y / nt, b = t.y - r * nt;
  const int64_t base = (int64_t)b * kScanBlock;
  double* oi = out + d.off + (int64_t)r * d.Nn;
  const double* yr = y + d.off + (int64_t)r * d.Nn;
  double yv[kScanItems];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + i * 256 + threadIdx.x;
    su[i * 256 + threadIdx.x] = (k < d.Nn) ? oi[k] : 0.0;
    yv[i] = (k < d.Nn) ? yr[k] : 0.0;
  }
  __syncthreads();
  // thread t scans nodes base + kScanItems t + j, j < kScanItems, in order
  double uu[kScanItems];
  double tsum = 0.0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    uu[j] = su[threadIdx.x * kScanItems + j];
    tsum += uu[j];
  }
  double run = scan[d.scan_off + t.y] + block_scan256(tsum, sh) - tsum;
  // each thread rewrites only the entries it read itself
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    su[threadIdx.x * kScanItems + j] = run + 0.5 * uu[j];
    run += uu[j];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + i * 256 + threadIdx.x;
    if (k < d.Nn) oi[k] = yv[i] - su[i * 256 + threadIdx.x];
  }
}

template <typename T>
hipError_t precond_forward(birk_plan* p, int jac_kind, const double* J, const T* y, T* out,
                           hipStream_t s) {
  const int pn = jac_kind == BIRK_J_PER_NODE ? 1 : 0;
  if constexpr (std::is_same<T, double>::value) {
    if (p->pfwd_maxnx <= 16) {
      static constexpr decltype(&k_pfwd_sums_all<8>) kUniform[9] = {
          nullptr,
          k_pfwd_sums_all<1, 1>,
          k_pfwd_sums_all<2, 2>,
          k_pfwd_sums_all<3, 3>,
          k_pfwd_sums_all<4, 4>,
          k_pfwd_sums_all<5, 5>,
          k_pfwd_sums_all<6, 6>,
          k_pfwd_sums_all<7, 7>,
          k_pfwd_sums_all<8, 8>};
      auto f = (p->pfwd_unx >= 1 && p->pfwd_unx <= 8) ? kUniform[p->pfwd_unx]
               : p->pfwd_maxnx <= 4                   ? k_pfwd_sums_all<4>
               : p->pfwd_maxnx <= 8                   ? k_pfwd_sums_all<8>
                                                      : k_pfwd_sums_all<16>;
      hipLaunchKernelGGL(f, dim3(p->pfwd_nbtiles), dim3(256), 0, s, p->pfwd_btiles, p->idesc, J, pn, y, out, p->scan);
      hipLaunchKernelGGL(k_pfwd_scanparts, dim3(p->pfwd_npairs), dim3(256), 0, s, p->pfwd_pairs, p->idesc, p->scan);
      hipLaunchKernelGGL(k_pfwd_final_u, dim3(p->pfwd_ntiles), dim3(256), 0, s, p->pfwd_tiles, p->idesc, y,
                         (const double*)p->scan, out);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL(k_pfwd_sums<T>, dim3(p->pfwd_ntiles), dim3(256), 0, s, p->pfwd_tiles, p->idesc, J, pn, y,
                     p->scan);
  hipLaunchKernelGGL(k_pfwd_scanparts, dim3(p->pfwd_npairs), dim3(256), 0, s, p->pfwd_pairs, p->idesc, p->scan);
  hipLaunchKernelGGL(k_pfwd_final<T>, dim3(p->pfwd_ntiles), dim3(256), 0, s, p->pfwd_tiles, p->idesc, J, pn, y,
                     (const double*)p->scan, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ J x per node

// y_k = J_k x_k per node for every instance of a class.  tile = (k, block of 256 nodes).
template <int NX, typename T>
__global__ __launch_bounds__(256) void k_jac_class(const double* __restrict__ J, int per_node,
                                                   const T* __restrict__ x, T* __restrict__ y,
                                                   const ScanDesc* __restrict__ sd, const int2* __restrict__ tiles) {
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int64_t k = (int64_t)t.y * blockDim.x + threadIdx.x;
  const int64_t Nn = d.Nn;
  if (k >= Nn) return;
  const T* xi = x + d.off;
  T* yi = y + d.off;
  double xv[NX];
#pragma unroll
  for (int c = 0; c < NX; ++c) xv[c] = (double)xi[(int64_t)c * Nn + k];
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < NX; ++c) {
      const double j = per_node ? J[d.joff + ((int64_t)(r * NX + c)) * Nn + k] : J[d.jcoff + r * NX + c];
      acc += j * xv[c];
    }
    yi[(int64_t)r * Nn + k] = (T)acc;
  }
}

static inline unsigned nblocks(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

static hipError_t upload_tiles(birk_plan* p, const std::vector<int2>& v, int2** dst) {
  void* d = nullptr;
  hipError_t e = hipMalloc(&d, std::max<size_t>(v.size(), 1) * sizeof(int2));
  if (e != hipSuccess) return e;
  p->allocs.push_back(d);
  *dst = (int2*)d;
  if (v.empty()) return hipSuccess;
  return hipMemcpy(d, v.data(), v.size() * sizeof(int2), hipMemcpyHostToDevice);
}

hipError_t plan_solve(birk_plan* p) {
  hipError_t e = hipSuccess;
  {
    // P y work lists: every tile of every component of every instance, and every
    // (instance, component) scan
    std::vector<int2> tl, pr;
    for (int i = 0; i < (int)p->inst.size(); ++i) {
      const Instance& in = p->inst[i];
      const int nt = (int)((in.Nn + kScanBlock - 1) / kScanBlock);
      for (int r = 0; r < in.nx; ++r) {
        pr.push_back(make_int2(i, r));
        for (int b = 0; b < nt; ++b) tl.push_back(make_int2(i, r * nt + b));
      }
    }
    if ((e = upload_tiles(p, tl, &p->pfwd_tiles)) != hipSuccess) return e;
    p->pfwd_ntiles = (int)tl.size();
    if ((e = upload_tiles(p, pr, &p->pfwd_pairs)) != hipSuccess) return e;
    p->pfwd_npairs = (int)pr.size();
    std::vector<int2> bt;
    p->pfwd_maxnx = 0;
    p->pfwd_unx = p->inst.empty() ? 0 : (int)p->inst[0].nx;
    for (int i = 0; i < (int)p->inst.size(); ++i) {
      const Instance& in = p->inst[i];
      const int nt = (int)((in.Nn + kScanBlock - 1) / kScanBlock);
      for (int b = 0; b < nt; ++b) bt.push_back(make_int2(i, b));
      p->pfwd_maxnx = std::max(p->pfwd_maxnx, (int)in.nx);
      if ((int)in.nx != p->pfwd_unx) p->pfwd_unx = 0;
    }
    if ((e = upload_tiles(p, bt, &p->pfwd_btiles)) != hipSuccess) return e;
    p->pfwd_nbtiles = (int)bt.size();
  }
  // Krylov segmentation
  {
    const int B = (int)p->inst.size();
    std::vector<int2> tiles, ranges(B);
    std::vector<int64_t> ioff(B), ilen(B);
    for (int i = 0; i < B; ++i) {
      const Instance& in = p->inst[i];
      ioff[i] = in.off;
      ilen[i] = in.Nn * in.nx;
      ranges[i].x = (int)tiles.size();
      for (int64_t c = 0; c * kSegChunk < ilen[i]; ++c) tiles.push_back(make_int2(i, (int)c));
      ranges[i].y = (int)tiles.size();
    }
    SegSet& sg = p->seg;
    sg.ntiles = (int)tiles.size();
    if ((e = upload_tiles(p, tiles, &sg.tiles)) != hipSuccess) return e;
    if ((e = upload_tiles(p, ranges, &sg.ranges)) != hipSuccess) return e;
    void* d1 = nullptr;
    void* d2 = nullptr;
    if ((e = hipMalloc(&d1, B * sizeof(int64_t))) != hipSuccess) return e;
    p->allocs.push_back(d1);
    if ((e = hipMalloc(&d2, B * sizeof(int64_t))) != hipSuccess) return e;
    p->allocs.push_back(d2);
    sg.ioff = (int64_t*)d1;
    sg.ilen = (int64_t*)d2;
    if ((e = hipMemcpy(d1, ioff.data(), B * sizeof(int64_t), hipMemcpyHostToDevice)) != hipSuccess) return e;
    if ((e = hipMemcpy(d2, ilen.data(), B * sizeof(int64_t), hipMemcpyHostToDevice)) != hipSuccess) return e;
  }
  return hipSuccess;
}

#define BIRK_NX_SWITCH(nx, CALL)                                       \
  switch (nx) {                                                        \
    case 1: { constexpr int NXC = 1; CALL; } break;                    \
    case 2: { constexpr int NXC = 2; CALL; } break;                    \
    case 3: { constexpr int NXC = 3; CALL; } break;                    \
    case 4: { constexpr int NXC = 4; CALL; } break;                    \
    case 5: { constexpr int NXC = 5; CALL; } break;                    \
    case 6: { constexpr int NXC = 6; CALL; } break;                    \
    case 7: { constexpr int NXC = 7; CALL; } break;                    \
    case 8: { constexpr int NXC = 8; CALL; } break;                    \
    case 9: { constexpr int NXC = 9; CALL; } break;                    \
    case 10: { constexpr int NXC = 10; CALL; } break;                  \
    case 11: { constexpr int NXC = 11; CALL; } break;                  \
    case 12: { constexpr int NXC = 12; CALL; } break;                  \
    default: return hipErrorInvalidValue;                              \
  }

template <int NX, typename T>
static void jac_class(const ScanClass& sc, const double* J, int pn, const T* x, T* y, hipStream_t s) {
  hipLaunchKernelGGL((k_jac_class<NX, T>), dim3(sc.n_nodes), dim3(256), 0, s, J, pn, x, y, sc.dev, sc.nodes);
}

template <typename T>
hipError_t jac_times(birk_plan* p, int jac_kind, const double* J, const T* x, T* y, hipStream_t s) {
  const int pn = jac_kind == BIRK_J_PER_NODE ? 1 : 0;
  for (const ScanClass& sc : p->sclass) {
    BIRK_NX_SWITCH(sc.nx, (jac_class<NXC, T>(sc, J, pn, x, y, s)))
  }
  return hipGetLastError();
}

#undef BIRK_NX_SWITCH

template hipError_t jac_times<double>(birk_plan*, int, const double*, const double*, double*, hipStream_t);
template hipError_t jac_times<float>(birk_plan*, int, const double*, const float*, float*, hipStream_t);
template hipError_t precond_forward<double>(birk_plan*, int, const double*, const double*, double*, hipStream_t);
template hipError_t precond_forward<float>(birk_plan*, int, const double*, const float*, float*, hipStream_t);

// ------------------------------------------------------------------ Krylov BLAS-1
// Krylov BLAS-1: at most kMaxDots basis vectors per call, reductions in double.
constexpr int kMaxDots = 32;

// z = a - b  (FastAX step 3)
template <typename T>
__global__ void k_sub(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ z, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  z[e] = a[e] - b[e];
}

// r = beta - (x - t) = beta - x + t, in double
__global__ void k_residual(const double* __restrict__ beta, const double* __restrict__ x,
                           const double* __restrict__ t, double* __restrict__ r, int64_t n) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  r[e] = beta[e] - x[e] + t[e];
}


// ---- segmented forms: one launch over every instance of the batch ----
// A tile is kSegChunk consecutive elements of one instance; partial results go to
// part[tile][kMaxDots + 1] and are summed per instance over its tile range in a fixed
// order.

// MAXQ >= nq bounds the per-thread accumulators (registers) at compile time.  SUB = 1
// first forms u = a - b (in T, as k_sub does) and stores it, in the same pass.
template <typename T, int MAXQ, int SUB>
__global__ __launch_bounds__(256) void k_sdots(const T* __restrict__ Q, int64_t ld, int nq, const T* u_in,
                                               const T* __restrict__ a, const T* __restrict__ b, T* u_out,
                                               SegSet sg, double* __restrict__ part) {
  const int2 t = sg.tiles[blockIdx.x];
  const int64_t base = sg.ioff[t.x] + (int64_t)t.y * kSegChunk;
  const int64_t end = sg.ioff[t.x] + min((int64_t)(t.y + 1) * kSegChunk, sg.ilen[t.x]);
  double acc[MAXQ], nrm = 0.0;
#pragma unroll
  for (int i = 0; i < MAXQ; ++i) acc[i] = 0.0;
  for (int64_t e = base + threadIdx.x; e < end; e += blockDim.x) {
    double ue;
    if (SUB) {
      const T d = a[e] - b[e];
      u_out[e] = d;
      ue = (double)d;
    } else {
      ue = (double)u_in[e];
    }
#pragma unroll
    for (int i = 0; i < MAXQ; ++i)
      if (i < nq) acc[i] += (double)Q[(int64_t)i * ld + e] * ue;
    nrm += ue * ue;
  }
  __shared__ double sh[256];
#pragma unroll
  for (int i = 0; i < MAXQ; ++i) {
    if (i < nq) {
      const double v = block_sum256(acc[i], sh);
      if (threadIdx.x == 0) part[(int64_t)blockIdx.x * (kMaxDots + 1) + i] = v;
    }
  }
  const double v = block_sum256(nrm, sh);
  if (threadIdx.x == 0) part[(int64_t)blockIdx.x * (kMaxDots + 1) + kMaxDots] = v;
}

// Smallest accumulator bound of the Krylov kernels that covers nq basis vectors.
#define BIRK_MAXQ_SWITCH(nq, CALL)                         \
  if ((nq) <= 2) { constexpr int MQ = 2; CALL; }           \
  else if ((nq) <= 8) { constexpr int MQ = 8; CALL; }      \
  else { constexpr int MQ = kMaxDots; CALL; }

// grid = (nq + 1, instances): block (x, i) sums output x (x == nq: the norm slot) of
// instance i over its tiles into out[i * ostride + slot].
__global__ __launch_bounds__(256) void k_sreduce(const double* __restrict__ part, SegSet sg, int nq,
                                                 double* __restrict__ out, int64_t ostride) {
  __shared__ double sh[256];
  const int i = blockIdx.y;
  const int slot = (blockIdx.x < (unsigned)nq) ? (int)blockIdx.x : kMaxDots;
  const int2 r = sg.ranges[i];
  double s = 0.0;
  for (int b = r.x + threadIdx.x; b < r.y; b += blockDim.x) s += part[(int64_t)b * (kMaxDots + 1) + slot];
  const double tot = block_sum256(s, sh);
  if (threadIdx.x == 0) out[(int64_t)i * ostride + slot] = tot;
}

// u -= sum_k h[i][k] Q_k on instance i's tiles; part <- tile sums of ||u||^2 when asked,
// and with DOTS also of Q_k . u (the updated u), the first half of the next Gram-Schmidt
// pass fused into this one.
template <typename T, bool DOTS, int MAXQ>
__global__ __launch_bounds__(256) void k_saxpys(const T* __restrict__ Q, int64_t ld, int nq,
                                                const double* __restrict__ h, int64_t hstride, T* __restrict__ u,
                                                SegSet sg, double* __restrict__ part) {
  const int2 t = sg.tiles[blockIdx.x];
  __shared__ double hs[kMaxDots];
  if (threadIdx.x < kMaxDots) hs[threadIdx.x] = (int)threadIdx.x < nq ? h[(int64_t)t.x * hstride + threadIdx.x] : 0.0;
  __syncthreads();
  const int64_t base = sg.ioff[t.x] + (int64_t)t.y * kSegChunk;
  const int64_t end = sg.ioff[t.x] + min((int64_t)(t.y + 1) * kSegChunk, sg.ilen[t.x]);
  constexpr int ND = DOTS ? MAXQ : 1;
  double acc[ND];
#pragma unroll
  for (int i = 0; i < ND; ++i) acc[i] = 0.0;
  double nrm = 0.0;
  for (int64_t e = base + threadIdx.x; e < end; e += blockDim.x) {
    double ue = (double)u[e];
    double qv[ND];
#pragma unroll
    for (int i = 0; i < MAXQ; ++i)
      if (i < nq) {
        const double q = (double)Q[(int64_t)i * ld + e];
        if constexpr (DOTS) qv[i] = q;
        ue -= hs[i] * q;
      }
    const T us = (T)ue;
    u[e] = us;
    const double un = (double)us;
    nrm += un * un;
    if constexpr (DOTS) {
#pragma unroll
      for (int i = 0; i < MAXQ; ++i)
        if (i < nq) acc[i] += qv[i] * un;
    }
  }
  if (part) {
    __shared__ double sh[256];
    if constexpr (DOTS) {
#pragma unroll
      for (int i = 0; i < MAXQ; ++i) {
        if (i < nq) {
          const double v = block_sum256(acc[i], sh);
          if (threadIdx.x == 0) part[(int64_t)blockIdx.x * (kMaxDots + 1) + i] = v;
        }
      }
    }
    const double v = block_sum256(nrm, sh);
    if (threadIdx.x == 0) part[(int64_t)blockIdx.x * (kMaxDots + 1) + kMaxDots] = v;
  }
}

// q = u / sqrt(nrm2[i]) on instance i's tiles; a zero or non-finite norm writes zeros
// (the instance has stopped; its later basis vectors are never combined).
template <typename T>
__global__ __launch_bounds__(256) void k_snormalize(const T* __restrict__ u, const double* __restrict__ nrm2,
                                                    int64_t stride, T* __restrict__ q, SegSet sg) {
  const int2 t = sg.tiles[blockIdx.x];
  const double n2 = nrm2[(int64_t)t.x * stride];
  const double inv = (n2 > 0.0 && isfinite(n2)) ? 1.0 / sqrt(n2) : 0.0;
  const int64_t base = sg.ioff[t.x] + (int64_t)t.y * kSegChunk;
  const int64_t end = sg.ioff[t.x] + min((int64_t)(t.y + 1) * kSegChunk, sg.ilen[t.x]);
  for (int64_t e = base + threadIdx.x; e < end; e += blockDim.x) q[e] = (T)(inv == 0.0 ? 0.0 : (double)u[e] * inv);
}

// y = alpha[i] x on instance i's tiles
template <typename TI, typename TO>
__global__ __launch_bounds__(256) void k_sscale_conv(const TI* __restrict__ x, TO* __restrict__ y,
                                                     const double* __restrict__ alpha, SegSet sg) {
  const int2 t = sg.tiles[blockIdx.x];
  const double a = alpha[t.x];
  const int64_t base = sg.ioff[t.x] + (int64_t)t.y * kSegChunk;
  const int64_t end = sg.ioff[t.x] + min((int64_t)(t.y + 1) * kSegChunk, sg.ilen[t.x]);
  for (int64_t e = base + threadIdx.x; e < end; e += blockDim.x) y[e] = (TO)(a == 0.0 ? 0.0 : a * (double)x[e]);
}

// x += sum_{k < cnt[i]} c[i][k] Q_k on instance i's tiles (x double, sum in double)
template <typename T>
__global__ __launch_bounds__(256) void k_scombine(const T* __restrict__ Q, int64_t ld, const double* __restrict__ c,
                                                  int64_t cstride, const int* __restrict__ cnt,
                                                  double* __restrict__ x, SegSet sg) {
  const int2 t = sg.tiles[blockIdx.x];
  const int nq = cnt[t.x];
  __shared__ double cs[kMaxDots];
  if (threadIdx.x < kMaxDots) cs[threadIdx.x] = (int)threadIdx.x < nq ? c[(int64_t)t.x * cstride + threadIdx.x] : 0.0;
  __syncthreads();
  const int64_t base = sg.ioff[t.x] + (int64_t)t.y * kSegChunk;
  const int64_t end = sg.ioff[t.x] + min((int64_t)(t.y + 1) * kSegChunk, sg.ilen[t.x]);
  for (int64_t e = base + threadIdx.x; e < end; e += blockDim.x) {
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < kMaxDots; ++i)
      if (i < nq) acc += cs[i] * (double)Q[(int64_t)i * ld + e];
    x[e] += acc;
  }
}

// ---- GMRES scalars on the device: per instance the rotated Hessenberg columns R, the
// right-hand side g of the small least-squares problem, the Givens rotations, and
// (running, columns kept, iterations, status, tolerance, ||r||); one thread per instance.
__global__ void k_gm_init(const double* __restrict__ prm, double* __restrict__ st, int ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
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

// Arnoldi column j of every running instance from the CGS2 dot products (d1 + d2 = the
// coefficients, the norm slot of d2 = ||u||^2): earlier rotations, a new rotation that
// annihilates h_{j+1,j}, the update of g; the instance stops when |g_{j+1}| <= tol, on a
// lucky breakdown, on breakdown (no column kept) or on a non-finite value.
__global__ void k_gm_column(int j, const double* __restrict__ dots, int64_t dstride, double* __restrict__ st,
                            int ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
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
    const double a = cs[k] * col[k] + sn[k] * col[k + 1];
    col[k + 1] = -sn[k] * col[k] + cs[k] * col[k + 1];
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

// running flag per instance into flags[i] (read by the host between chunks)
__global__ void k_gm_running(const double* __restrict__ st, double* __restrict__ flags, int ninst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ninst) return;
  flags[i] = st[(int64_t)i * kGmStride + kGmMisc + GM_RUN];
}

// Host-side launch helpers used by the GMRES driver.
namespace kry {

template <typename T>
void sub(const T* a, const T* b, T* z, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_sub<T>, dim3(nblocks(n, 256)), dim3(256), 0, s, a, b, z, n);
}

void residual(const double* beta, const double* x, const double* t, double* r, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_residual, dim3(nblocks(n, 256)), dim3(256), 0, s, beta, x, t, r, n);
}


template <typename T>
void sdots(const birk_plan* p, const T* Q, int nq, const T* u, double* out, int64_t ostride, hipStream_t s) {
  const SegSet& sg = p->seg;
  BIRK_MAXQ_SWITCH(nq, hipLaunchKernelGGL((k_sdots<T, MQ, 0>), dim3(sg.ntiles), dim3(256), 0, s, Q, p->total_len, nq,
                                           u, (const T*)nullptr, (const T*)nullptr, (T*)nullptr, sg, p->krylov_part))
  hipLaunchKernelGGL(k_sreduce, dim3(nq + 1, (unsigned)p->inst.size()), dim3(256), 0, s, p->krylov_part, sg, nq, out,
                     ostride);
}

template <typename T>
void sub_sdots(const birk_plan* p, const T* Q, int nq, const T* a, const T* b, T* u, double* out, int64_t ostride,
               hipStream_t s) {
  const SegSet& sg = p->seg;
  BIRK_MAXQ_SWITCH(nq, hipLaunchKernelGGL((k_sdots<T, MQ, 1>), dim3(sg.ntiles), dim3(256), 0, s, Q, p->total_len, nq,
                                           (const T*)nullptr, a, b, u, sg, p->krylov_part))
  hipLaunchKernelGGL(k_sreduce, dim3(nq + 1, (unsigned)p->inst.size()), dim3(256), 0, s, p->krylov_part, sg, nq, out,
                     ostride);
}

template <typename T>
void saxpys(const birk_plan* p, const T* Q, int nq, const double* h, int64_t hstride, T* u, double* nrm_out,
            hipStream_t s) {
  const SegSet& sg = p->seg;
  BIRK_MAXQ_SWITCH(nq, hipLaunchKernelGGL((k_saxpys<T, false, MQ>), dim3(sg.ntiles), dim3(256), 0, s, Q,
                                           p->total_len, nq, h, hstride, u, sg, nrm_out ? p->krylov_part : nullptr))
  if (nrm_out)
    hipLaunchKernelGGL(k_sreduce, dim3(1, (unsigned)p->inst.size()), dim3(256), 0, s, p->krylov_part, sg, 0, nrm_out,
                       hstride);
}

template <typename T>
void saxpys_dots(const birk_plan* p, const T* Q, int nq, const double* h, int64_t hstride, T* u, double* out,
                 int64_t ostride, hipStream_t s) {
  const SegSet& sg = p->seg;
  BIRK_MAXQ_SWITCH(nq, hipLaunchKernelGGL((k_saxpys<T, true, MQ>), dim3(sg.ntiles), dim3(256), 0, s, Q,
                                           p->total_len, nq, h, hstride, u, sg, p->krylov_part))
  hipLaunchKernelGGL(k_sreduce, dim3(nq + 1, (unsigned)p->inst.size()), dim3(256), 0, s, p->krylov_part, sg, nq, out,
                     ostride);
}

template <typename T>
void snormalize(const birk_plan* p, const T* u, const double* nrm2, int64_t stride, T* q, hipStream_t s) {
  hipLaunchKernelGGL(k_snormalize<T>, dim3(p->seg.ntiles), dim3(256), 0, s, u, nrm2, stride, q, p->seg);
}

template <typename TI, typename TO>
void sscale_conv(const birk_plan* p, const TI* x, TO* y, const double* alpha, hipStream_t s) {
  hipLaunchKernelGGL((k_sscale_conv<TI, TO>), dim3(p->seg.ntiles), dim3(256), 0, s, x, y, alpha, p->seg);
}

template <typename T>
void scombine(const birk_plan* p, const T* Q, const double* c, int64_t cstride, const int* cnt, double* x,
              hipStream_t s) {
  hipLaunchKernelGGL(k_scombine<T>, dim3(p->seg.ntiles), dim3(256), 0, s, Q, p->total_len, c, cstride, cnt, x,
                     p->seg);
}

void gm_init(const birk_plan* p, const double* prm, double* st, hipStream_t s) {
  const int B = (int)p->inst.size();
  hipLaunchKernelGGL(k_gm_init, dim3(nblocks(B, 64)), dim3(64), 0, s, prm, st, B);
}
void gm_column(const birk_plan* p, int j, const double* dots, int64_t dstride, double* st, hipStream_t s) {
  const int B = (int)p->inst.size();
  hipLaunchKernelGGL(k_gm_column, dim3(nblocks(B, 64)), dim3(64), 0, s, j, dots, dstride, st, B);
}
void gm_solve(const birk_plan* p, double* st, double* coef, int64_t cstride, int* cnt, double* flags, hipStream_t s) {
  const int B = (int)p->inst.size();
  hipLaunchKernelGGL(k_gm_solve, dim3(nblocks(B, 64)), dim3(64), 0, s, st, coef, cstride, cnt, flags, B);
}
void gm_running(const birk_plan* p, const double* st, double* flags, hipStream_t s) {
  const int B = (int)p->inst.size();
  hipLaunchKernelGGL(k_gm_running, dim3(nblocks(B, 64)), dim3(64), 0, s, st, flags, B);
}

template void sdots<double>(const birk_plan*, const double*, int, const double*, double*, int64_t, hipStream_t);
template void sdots<float>(const birk_plan*, const float*, int, const float*, double*, int64_t, hipStream_t);
template void sub_sdots<double>(const birk_plan*, const double*, int, const double*, const double*, double*, double*,
                                int64_t, hipStream_t);
template void sub_sdots<float>(const birk_plan*, const float*, int, const float*, const float*, float*, double*,
                               int64_t, hipStream_t);
template void saxpys_dots<double>(const birk_plan*, const double*, int, const double*, int64_t, double*, double*,
                                  int64_t, hipStream_t);
template void saxpys_dots<float>(const birk_plan*, const float*, int, const double*, int64_t, float*, double*,
                                 int64_t, hipStream_t);
template void saxpys<double>(const birk_plan*, const double*, int, const double*, int64_t, double*, double*,
                             hipStream_t);
template void saxpys<float>(const birk_plan*, const float*, int, const double*, int64_t, float*, double*,
                            hipStream_t);
template void snormalize<double>(const birk_plan*, const double*, const double*, int64_t, double*, hipStream_t);
template void snormalize<float>(const birk_plan*, const float*, const double*, int64_t, float*, hipStream_t);
template void sscale_conv<double, double>(const birk_plan*, const double*, double*, const double*, hipStream_t);
template void sscale_conv<double, float>(const birk_plan*, const double*, float*, const double*, hipStream_t);
template void scombine<double>(const birk_plan*, const double*, const double*, int64_t, const int*, double*,
                               hipStream_t);
template void scombine<float>(const birk_plan*, const float*, const double*, int64_t, const int*, double*,
                              hipStream_t);

template void sub<double>(const double*, const double*, double*, int64_t, hipStream_t);
template void sub<float>(const float*, const float*, float*, int64_t, hipStream_t);
}  // namespace kry
}  // namespace birk
