// Jacobian products and the Birkhoff preconditioner's P y (gfx950).
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

// The same, or y_k = J_k^T x_k, for the instances with more states than there are classes for
// (n_x > kWideNx; the others' tiles return at once).  tile = (instance, component * tiles + tile),
// as in the P y passes.  Bound: J per node from memory; x and one J per instance from the caches.
template <typename T, bool TRANS>
__global__ __launch_bounds__(256) void k_jac_many(const int2* __restrict__ tiles, const InstDesc* __restrict__ idesc,
                                                  const double* __restrict__ J, int per_node,
                                                  const T* __restrict__ x, T* __restrict__ y) {
  const int2 t = tiles[blockIdx.x];
  const InstDesc d = idesc[t.x];
  if (d.nx <= kWideNx) return;
  const int nt = pfwd_ntiles(d.Nn), r = t.y / nt, nx = (int)d.nx;
  const int64_t Nn = d.Nn, base = (int64_t)(t.y - r * nt) * kScanBlock;
  const double* Ji = J + (per_node ? d.joff : d.jcoff);
  const T* xi = x + d.off;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t k = base + i * 256 + threadIdx.x;
    if (k >= Nn) break;
    double acc = 0.0;
    for (int c = 0; c < nx; ++c) {
      const int64_t e = TRANS ? (int64_t)c * nx + r : (int64_t)r * nx + c;
      acc += (per_node ? Ji[e * Nn + k] : Ji[e]) * (double)xi[(int64_t)c * Nn + k];
    }
    y[d.off + (int64_t)r * Nn + k] = (T)acc;
  }
}

template <typename T, bool TRANS>
hipError_t jac_many(birk_plan* p, int jac_kind, const double* J, const T* x, T* y, hipStream_t s) {
  if (p->pfwd_maxnx <= kWideNx) return hipSuccess;
  hipLaunchKernelGGL((k_jac_many<T, TRANS>), dim3(p->pfwd_ntiles), dim3(256), 0, s, p->pfwd_tiles, p->idesc, J,
                     jac_kind == BIRK_J_PER_NODE ? 1 : 0, x, y);
  return hipGetLastError();
}
template hipError_t jac_many<double, true>(birk_plan*, int, const double*, const double*, double*, hipStream_t);


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
    std::vector<int64_t> ioff(B), ilen(B), icol(B);
    int64_t ncol = 0;
    for (int i = 0; i < B; ++i) {
      const Instance& in = p->inst[i];
      ioff[i] = in.off;
      ilen[i] = in.Nn * in.nx;
      icol[i] = ncol;
      ncol += in.nx;
      ranges[i].x = (int)tiles.size();
      for (int64_t c = 0; c * kSegChunk < ilen[i]; ++c) tiles.push_back(make_int2(i, (int)c));
      ranges[i].y = (int)tiles.size();
    }
    SegSet& sg = p->seg;
    sg.ntiles = (int)tiles.size();
    if ((e = upload_tiles(p, tiles, &sg.tiles)) != hipSuccess) return e;
    if ((e = upload_tiles(p, ranges, &sg.ranges)) != hipSuccess) return e;
    for (auto [src, dst] : {std::pair{&ioff, &sg.ioff}, std::pair{&ilen, &sg.ilen}, std::pair{&icol, &sg.icol}}) {
      void* d = nullptr;
      if ((e = upload_raw(p, src->data(), B * sizeof(int64_t), &d)) != hipSuccess) return e;
      *dst = (int64_t*)d;
    }
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
  return jac_many<T, false>(p, jac_kind, J, x, y, s);
}

#undef BIRK_NX_SWITCH

template hipError_t jac_times<double>(birk_plan*, int, const double*, const double*, double*, hipStream_t);
template hipError_t jac_times<float>(birk_plan*, int, const double*, const float*, float*, hipStream_t);
template hipError_t precond_forward<double>(birk_plan*, int, const double*, const double*, double*, hipStream_t);
template hipError_t precond_forward<float>(birk_plan*, int, const double*, const float*, float*, hipStream_t);

}  // namespace birk
