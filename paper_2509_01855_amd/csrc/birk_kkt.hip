// The symmetric saddle-point (KKT) form of the collocated system and its MINRES solve.
//
// The paper counts matrix-free KKT solves per SQP step (Table 1, orbit-transfer results)
// without writing the system down.  Here: the equality-constrained quadratic model
//     min 1/2 (chi - chi_r)^T H (chi - chi_r)  s.t.  A chi = g,   A = I - (I (x) B^a) J
// (eq:Newton-ivp), H = diag(h) > 0, whose optimality conditions are
//     K [chi; lambda] = [f; g],   K = [[H, A^T], [A, 0]],   f = H chi_r,
// symmetric and indefinite.  MINRES (Paige-Saunders) with the symmetric positive definite
// block preconditioner M = blockdiag(H, P H^{-1} P^T), P = I - B~^a J the Birkhoff
// preconditioner (B~^a section) standing in for A in the Schur complement A H^{-1} A^T:
//     M^{-1} [r1; r2] = [r1 / h; P^{-T} (h * P^{-1} r2)].
//
// P^{-T}: P^T is block upper triangular in node order; row j of P^T x = y reads
//     (I - w_j J_j^T / 2) x_j - w_j J_j^T T_j = y_j,   T_j = sum_{k>j} x_k,
// i.e. with G_j = H_j^T, H_j = w_j (I - w_j J_j / 2)^{-1} J_j (the matrix of the forward
// substitution),
//     x_j = y_j + G_j (y_j / 2 + T_j),   T_{j-1} = T_j + x_j
//         = (I + G_j) T_j + (I + G_j / 2) y_j,
// an affine recurrence run from the last node down, evaluated as a scan of affine maps
// (birk_scan.hip, birk_wide.hip).  All arithmetic in double.
//
// MINRES keeps its scalar recurrences (the Lanczos coefficients, the Givens rotations and
// the step lengths) per instance in device memory, updated by one-thread-per-instance
// kernels between the vector passes, so an iteration enqueues no host work; the host
// reads the per-instance states once per chunk of iterations to test convergence.

#include <hip/hip_runtime.h>

#include <cmath>

#include "birk_dense.h"
#include "birk_internal.h"

namespace birk {
namespace kkt {

// ------------------------------------------------------------------ J^T x per node
template <int NX>
__global__ __launch_bounds__(256) void k_jac_t(const double* __restrict__ J, int per_node,
                                               const double* __restrict__ x, double* __restrict__ yv,
                                               const ScanDesc* __restrict__ dd, const int2* __restrict__ tiles) {
  const int2 tile = tiles[blockIdx.x];
  const ScanDesc& d = dd[tile.x];
  const int64_t k = (int64_t)tile.y * 256 + threadIdx.x;
  if (k >= d.Nn) return;
  double xv[NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) xv[r] = x[d.off + (int64_t)r * d.Nn + k];
#pragma unroll
  for (int c = 0; c < NX; ++c) {
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const double j = per_node ? J[d.joff + (int64_t)(r * NX + c) * d.Nn + k] : J[d.jcoff + r * NX + c];
      acc += j * xv[r];
    }
    yv[d.off + (int64_t)c * d.Nn + k] = acc;
  }
}

// ------------------------------------------------------------------ segmented vector passes
// The KKT vectors are pairs [top (n); bottom (n)].  A launch covers both halves: block b works
// half b % 2 of the plan's segment tile b / 2, kPer elements of each half per thread, all
// loads of a pass before its stores.  Partial dot products: part[b], an instance's side by side.
//
// Bound: launches and latency up to some 1e5 nodes, memory beyond.  Each dot product is taken
// where its second factor is formed, the scalars follow in the reduction's launch, and the
// first residual of a solve from zero is the right-hand side.  Five iterations at 65537 nodes,
// n_x = 6: 1244 us with a launch for each operation (27 an iteration), 1045 with 20.
struct Seg {
  const int2* tiles;
  const int64_t* ioff;
  const int64_t* ilen;
  const int2* ranges;
  int ntiles;
  int64_t n;
};
constexpr int kPer = kSegChunk / 512;

struct Elems {
  int inst;
  int64_t e[kPer];   // clamped into the block's range
  bool in[kPer];
};
__device__ __forceinline__ Elems elems_of(const Seg& sg, int blk) {
  const int2 t = sg.tiles[blk >> 1];
  const int64_t o = (int64_t)t.y * kSegChunk, left = sg.ilen[t.x] - o;
  Elems r;
  r.inst = t.x;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = (blk & 1) * (kSegChunk / 2) + (int)threadIdx.x + 256 * k;
    r.in[k] = i < left;
    r.e[k] = sg.ioff[t.x] + o + (r.in[k] ? i : 0);
  }
  return r;
}

// Sum over the workgroup (256 threads), in thread 0.
__device__ __forceinline__ double group_sum(double v, double* sh) {
  v = wave_sum_last(v);
  if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return threadIdx.x ? 0.0 : ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// Per-instance state of MINRES (doubles, kSt per instance).
enum {
  S_BETA1, S_BETA, S_OLDB, S_ALPHA, S_DBAR, S_EPS, S_PHIBAR, S_CS, S_SN, S_ACTIVE, S_SV, S_C1, S_C2, S_AV,
  S_A1, S_A2, S_PHI, S_THR, S_ITERS, S_IT0, kSt
};

// per-block partial of a . b over both halves
__global__ __launch_bounds__(256) void k_kv_dot(const double* __restrict__ a, const double* __restrict__ b,
                                                double* __restrict__ part, Seg sg) {
  __shared__ double sh[4];
  const Elems x = elems_of(sg, blockIdx.x);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const double v = a[x.e[k]] * b[x.e[k]] + a[sg.n + x.e[k]] * b[sg.n + x.e[k]];
    acc += x.in[k] ? v : 0.0;
  }
  acc = group_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// Sum of instance i's partials, in thread 0 (256 threads).
__device__ __forceinline__ double inst_sum(const double* __restrict__ part, const Seg& sg, int i, double* sh) {
  const int2 r = sg.ranges[i];
  double s = 0.0;
#pragma unroll 4
  for (int b = 2 * r.x + (int)threadIdx.x; b < 2 * r.y; b += 256) s += part[b];
  return group_sum(s, sh);
}

// out[i] = sum of instance i's partials
__global__ __launch_bounds__(256) void k_kv_reduce(const double* __restrict__ part, Seg sg, double* __restrict__ out) {
  __shared__ double sh[4];
  const double s = inst_sum(part, sg, blockIdx.x, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// ------------------------------------------------------------------ KKT operator pieces
// K z from its parts: top = h * u + l - t (t = J^T B^aT l), bottom = u - s (s = B^a J u);
// z = [u; l], h == null: H = I.
//   RESID: out = out2 = rhs - K z (the true residual), partials of out . out
//   else:  out = K z - C1[i] r1 (r1 in rhs), partials of z . out
template <bool RESID>
__global__ __launch_bounds__(256) void k_kkt_out(const double* __restrict__ z, const double* __restrict__ t,
                                                 const double* __restrict__ s, const double* __restrict__ h,
                                                 const double* __restrict__ rhs, const double* __restrict__ st,
                                                 double* __restrict__ out, double* __restrict__ out2,
                                                 double* __restrict__ part, Seg sg) {
  __shared__ double sh[4];
  const Elems x = elems_of(sg, blockIdx.x);
  const double c1 = RESID ? 0.0 : st[(int64_t)x.inst * kSt + S_C1];
  const double *zl = z + sg.n, *rl = rhs + sg.n;
  double top[kPer], bot[kPer], acc = 0.0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int64_t e = x.e[k];
    const double u = z[e], l = zl[e];
    const double kt = (h ? h[e] * u : u) + l - t[e], kb = u - s[e];
    if (RESID) {
      top[k] = rhs[e] - kt;
      bot[k] = rl[e] - kb;
    } else {
      top[k] = kt - c1 * rhs[e];
      bot[k] = kb - c1 * rl[e];
    }
    const double d = RESID ? top[k] * top[k] + bot[k] * bot[k] : u * top[k] + l * bot[k];
    acc += x.in[k] ? d : 0.0;
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (x.in[k]) {
      out[x.e[k]] = top[k];
      out[sg.n + x.e[k]] = bot[k];
      if (RESID) {
        out2[x.e[k]] = top[k];
        out2[sg.n + x.e[k]] = bot[k];
      }
    }
  acc = group_sum(acc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = acc;
}

// y -= C2[i] r2; ztop (when given) = y's top half / h: the first half of M^{-1} y
__global__ __launch_bounds__(256) void k_kkt_orth(double* __restrict__ y, const double* __restrict__ r2,
                                                  const double* __restrict__ h, const double* __restrict__ st,
                                                  double* __restrict__ ztop, Seg sg) {
  const Elems x = elems_of(sg, blockIdx.x);
  const double c2 = st[(int64_t)x.inst * kSt + S_C2];
  double top[kPer], bot[kPer], zt[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int64_t e = x.e[k];
    top[k] = y[e] - c2 * r2[e];
    bot[k] = y[sg.n + e] - c2 * r2[sg.n + e];
    zt[k] = h ? top[k] / h[e] : top[k];
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (x.in[k]) {
      y[x.e[k]] = top[k];
      y[sg.n + x.e[k]] = bot[k];
      if (ztop) ztop[x.e[k]] = zt[k];
    }
}

// z = a / h (or a), z = h * a (or a)
__global__ __launch_bounds__(256) void k_hscale(const double* __restrict__ a, const double* __restrict__ h,
                                                double* __restrict__ z, int64_t n, int divide) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  z[e] = h ? (divide ? a[e] / h[e] : a[e] * h[e]) : a[e];
}

// ------------------------------------------------------------------ MINRES scalar recurrences
// Cycle start: beta1 = sqrt(r1 . M^{-1} r1) from dot; thr = tol[i] beta1.
__device__ __forceinline__ void mr_init(double* __restrict__ s, double b2, double tol, int run) {
  const double b = (b2 > 0.0 && isfinite(b2)) ? sqrt(b2) : 0.0;
  for (int k = 0; k < kSt; ++k) s[k] = 0.0;
  s[S_BETA1] = b;
  s[S_BETA] = b;
  s[S_PHIBAR] = b;
  s[S_CS] = -1.0;
  s[S_THR] = tol * b;
  s[S_ACTIVE] = (run && b > 0.0) ? 1.0 : 0.0;
  s[S_IT0] = 1.0;
}

// Before an iteration: v = y / beta, and the coefficient of r1 in y = K v - (beta / oldb) r1.
__device__ __forceinline__ void mr_pre(double* __restrict__ s) {
  const bool on = s[S_ACTIVE] != 0.0;
  s[S_SV] = on ? 1.0 / s[S_BETA] : 0.0;
  s[S_C1] = (on && s[S_IT0] == 0.0) ? s[S_BETA] / s[S_OLDB] : 0.0;
}

// alpha = v . y; coefficient of r2 in y -= (alpha / beta) r2.
__device__ __forceinline__ void mr_alpha(double* __restrict__ s, double dot) {
  const bool on = s[S_ACTIVE] != 0.0;
  s[S_ALPHA] = on ? dot : 0.0;
  s[S_C2] = on ? dot / s[S_BETA] : 0.0;
}

// beta_{k+1} = sqrt(r2 . M^{-1} r2), the new Givens rotation, the step phi and the
// coefficients of w_k = (v - eps_{k-1} w_{k-2} - delta w_{k-1}) / gamma; stop when
// |phibar| <= thr, on breakdown, or on a non-finite value.
__device__ __forceinline__ void mr_givens(double* __restrict__ s, double b2) {
  if (s[S_ACTIVE] == 0.0) {
    s[S_PHI] = s[S_AV] = s[S_A1] = s[S_A2] = 0.0;
    return;
  }
  const double beta = (b2 > 0.0 && isfinite(b2)) ? sqrt(b2) : (b2 == 0.0 ? 0.0 : NAN);
  const double oldeps = s[S_EPS];
  const double cs = s[S_CS], sn = s[S_SN], dbar = s[S_DBAR], alpha = s[S_ALPHA];
  const double delta = cs * dbar + sn * alpha;
  const double gbar = sn * dbar - cs * alpha;
  const double gamma = hypot(gbar, beta);
  s[S_OLDB] = s[S_BETA];
  s[S_BETA] = beta;
  s[S_EPS] = sn * beta;
  s[S_DBAR] = -cs * beta;
  s[S_IT0] = 0.0;
  s[S_ITERS] += 1.0;
  if (!(gamma > 0.0) || !isfinite(gamma)) {
    s[S_PHI] = s[S_AV] = s[S_A1] = s[S_A2] = 0.0;
    s[S_ACTIVE] = 0.0;
    if (!isfinite(gamma) || !isfinite(beta)) s[S_PHIBAR] = NAN;
    return;
  }
  const double cn = gbar / gamma, snn = beta / gamma;
  const double phi = cn * s[S_PHIBAR];
  s[S_PHIBAR] = snn * s[S_PHIBAR];
  s[S_CS] = cn;
  s[S_SN] = snn;
  s[S_PHI] = phi;
  s[S_AV] = 1.0 / gamma;
  s[S_A1] = -oldeps / gamma;
  s[S_A2] = -delta / gamma;
  if (fabs(s[S_PHIBAR]) <= s[S_THR] || beta == 0.0) s[S_ACTIVE] = 0.0;
}

// A dot product from its partials and the scalars that follow from it, one workgroup per
// instance (a launch each for the sum, the step and the next iteration's coefficients otherwise).
enum { MR_INIT, MR_ALPHA, MR_GIVENS };
template <int OP>
__global__ __launch_bounds__(256) void k_mr_scalars(double* __restrict__ st, const double* __restrict__ part,
                                                    const double* __restrict__ tol, const int* __restrict__ run,
                                                    Seg sg) {
  __shared__ double sh[4];
  const int i = blockIdx.x;
  const double dot = inst_sum(part, sg, i, sh);
  if (threadIdx.x) return;
  double* s = st + (int64_t)i * kSt;
  if (OP == MR_INIT) mr_init(s, dot, tol[i], run[i]);
  if (OP == MR_ALPHA) mr_alpha(s, dot);
  if (OP == MR_GIVENS) mr_givens(s, dot);
  if (OP != MR_ALPHA) mr_pre(s);
}

// w_new = av v + a1 w1 + a2 w2 (into w1's buffer), x += phi w_new; and the next v = SV[i] y.
// A coefficient of zero leaves its vector unread (w1 and w2 hold nothing before the third and
// second iteration).  FIRST: only v.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_mr_update(double* __restrict__ v, const double* __restrict__ y,
                                                   double* __restrict__ w1, const double* __restrict__ w2,
                                                   double* __restrict__ x, const double* __restrict__ st, Seg sg) {
  const Elems b = elems_of(sg, blockIdx.x);
  const double* s = st + (int64_t)b.inst * kSt;
  const double sv = s[S_SV];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int64_t o = half * sg.n;
    double wn[kPer], xn[kPer], vn[kPer];
    if (!FIRST) {
      const double av = s[S_AV], a1 = s[S_A1], a2 = s[S_A2], phi = s[S_PHI];
      if (phi != 0.0 || av != 0.0) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) wn[k] = av * v[o + b.e[k]];
        if (a1 != 0.0) {
#pragma unroll
          for (int k = 0; k < kPer; ++k) wn[k] += a1 * w1[o + b.e[k]];
        }
        if (a2 != 0.0) {
#pragma unroll
          for (int k = 0; k < kPer; ++k) wn[k] += a2 * w2[o + b.e[k]];
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) xn[k] = x[o + b.e[k]] + phi * wn[k];
#pragma unroll
        for (int k = 0; k < kPer; ++k)
          if (b.in[k]) {
            w1[o + b.e[k]] = wn[k];
            x[o + b.e[k]] = xn[k];
          }
      }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) vn[k] = sv * y[o + b.e[k]];
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      if (b.in[k]) v[o + b.e[k]] = vn[k];
  }
}

// ------------------------------------------------------------------ host side
template <int NX>
static void jt_class(const ScanClass& sc, const double* J, int per_node, const double* x, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_jac_t<NX>, dim3(sc.n_nodes), dim3(256), 0, s, J, per_node, x, y, sc.dev, sc.nodes);
}

#define BIRK_NX_SWITCH(nx, CALL)                                      \
  switch (nx) {                                                       \
    case 1: { constexpr int NX = 1; CALL; } break;                    \
    case 2: { constexpr int NX = 2; CALL; } break;                    \
    case 3: { constexpr int NX = 3; CALL; } break;                    \
    case 4: { constexpr int NX = 4; CALL; } break;                    \
    case 5: { constexpr int NX = 5; CALL; } break;                    \
    case 6: { constexpr int NX = 6; CALL; } break;                    \
    case 7: { constexpr int NX = 7; CALL; } break;                    \
    case 8: { constexpr int NX = 8; CALL; } break;                    \
    case 9: { constexpr int NX = 9; CALL; } break;                    \
    case 10: { constexpr int NX = 10; CALL; } break;                  \
    case 11: { constexpr int NX = 11; CALL; } break;                  \
    default: { constexpr int NX = 12; CALL; } break;                  \
  }

}  // namespace kkt

using namespace kkt;

hipError_t jac_t_times(birk_plan* p, int jac_kind, const double* J, const double* x, double* y, hipStream_t s) {
  for (const ScanClass& sc : p->sclass) {
    BIRK_NX_SWITCH(sc.nx, (jt_class<NX>(sc, J, jac_kind == BIRK_J_PER_NODE, x, y, s)))
  }
  return jac_many<double, true>(p, jac_kind, J, x, y, s);
}

#undef BIRK_NX_SWITCH

// ------------------------------------------------------------------ the MINRES driver
namespace {

static inline unsigned nb256(int64_t n) { return (unsigned)((n + 255) / 256); }

struct KktBufs {
  double *x, *v, *y, *r1, *r2, *w, *w1, *rhs;   // pair vectors (2n each)
  double *st, *part, *dot, *tol;
  int* run;
};

Seg make_seg(const birk_plan* p) {
  Seg sg;
  sg.tiles = p->seg.tiles;
  sg.ioff = p->seg.ioff;
  sg.ilen = p->seg.ilen;
  sg.ranges = p->seg.ranges;
  sg.ntiles = p->seg.ntiles;
  sg.n = p->total_len;
  return sg;
}

}  // namespace

hipError_t ensure_kkt(birk_plan* p) {
  if (p->kkt_buf) return hipSuccess;
  const size_t n = (size_t)p->total_len, B = p->inst.size();
  const size_t nt = 2 * (size_t)std::max(p->seg.ntiles, 1);
  const size_t doubles = 8 * 2 * n + B * kSt + nt + 2 * B;
  hipError_t e = hipMalloc(&p->kkt_buf, doubles * sizeof(double) + B * sizeof(int));
  return e;
}

static KktBufs kkt_bufs(birk_plan* p) {
  const int64_t n2 = 2 * p->total_len;
  const size_t B = p->inst.size();
  const size_t nt = 2 * (size_t)std::max(p->seg.ntiles, 1);
  double* q = (double*)p->kkt_buf;
  KktBufs b;
  double** vecs[] = {&b.x, &b.v, &b.y, &b.r1, &b.r2, &b.w, &b.w1, &b.rhs};
  for (double** v : vecs) {
    *v = q;
    q += n2;
  }
  b.st = q;
  q += B * kSt;
  b.part = q;
  q += nt;
  b.dot = q;
  q += B;
  b.tol = q;
  q += B;
  b.run = (int*)q;
  return b;
}

// The parts of K [u; l]: B^a J u in tmp_vec[1], J^T B^aT l in tmp_vec[3] (tmp_vec[0], [2] used).
static hipError_t kkt_parts(birk_plan* p, int jk, const double* J, const double* z, hipStream_t s) {
  const double* u = z;
  const double* l = z + p->total_len;
  double* t0 = (double*)p->tmp_vec[0];
  double* t1 = (double*)p->tmp_vec[1];
  double* t2 = (double*)p->tmp_vec[2];
  double* t3 = (double*)p->tmp_vec[3];
  hipError_t e = jac_times<double>(p, jk, J, u, t0, s);                 // J u
  if (e == hipSuccess) e = apply_product<double>(p, t0, t1, 0, s);       // B^a J u
  if (e == hipSuccess) e = apply_product<double>(p, l, t2, 1, s);        // B^aT l
  if (e == hipSuccess) e = jac_t_times(p, jk, J, t2, t3, s);             // J^T B^aT l
  return e;
}

// M^{-1} [r1; r2] = [r1 / h; P^{-T}(h * P^{-1} r2)]; top_done: z's top half is there already
static hipError_t kkt_prec(birk_plan* p, int jk, const double* J, const double* h, const double* r, double* z,
                           int use_precond, bool top_done, hipStream_t s) {
  const int64_t n = p->total_len;
  if (!use_precond) return hipMemcpyAsync(z, r, 2 * n * sizeof(double), hipMemcpyDeviceToDevice, s);
  if (!top_done) hipLaunchKernelGGL(k_hscale, dim3(nb256(n)), dim3(256), 0, s, r, h, z, n, 1);
  double* t0 = (double*)p->tmp_vec[0];
  hipError_t e = scan_inverse<double>(p, jk, J, r + n, t0, nullptr, 0, s, nullptr);
  if (e != hipSuccess) return e;
  if (h) hipLaunchKernelGGL(k_hscale, dim3(nb256(n)), dim3(256), 0, s, t0, h, t0, n, 0);
  return scan_inverse_t(p, jk, J, t0, z + n, s);
}

// MINRES on the KKT system for every instance of the batch (arguments checked by the
// caller): restarted on the true residual [f; g] - K [chi; lambda] in double until
// ||r|| <= rtol ||[f; g]|| per instance; each cycle runs MINRES on K d = r (the
// correction accumulates into the iterate) to a preconditioned-residual tolerance.
birk_status kkt_solve(birk_plan* p, int jk, const double* J, const double* h, const double* f, const double* g,
                      double* chi, double* lam, const birk_solve_opts* o, birk_solve_info* info) {
  const int B = (int)p->inst.size();
  const int64_t n = p->total_len;
  hipStream_t s = p->stream;
  hipError_t e = ensure_kkt(p);
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? BIRK_ERR_NOMEM : BIRK_ERR_DEVICE;
  KktBufs b = kkt_bufs(p);
  const Seg sg = make_seg(p);
  const unsigned nt2 = 2u * (unsigned)sg.ntiles;
  // rhs = [f; g]; x = [chi; lam] (zero unless use_x0)
  if (f) e = hipMemcpyAsync(b.rhs, f, n * sizeof(double), hipMemcpyDeviceToDevice, s);
  else e = hipMemsetAsync(b.rhs, 0, n * sizeof(double), s);
  if (e == hipSuccess) e = hipMemcpyAsync(b.rhs + n, g, n * sizeof(double), hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && o->use_x0) {
    e = hipMemcpyAsync(b.x, chi, n * sizeof(double), hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(b.x + n, lam, n * sizeof(double), hipMemcpyDeviceToDevice, s);
  } else if (e == hipSuccess) {
    e = hipMemsetAsync(b.x, 0, 2 * n * sizeof(double), s);
  }
  if (e != hipSuccess) return BIRK_ERR_DEVICE;
  const double* t1 = (const double*)p->tmp_vec[1];
  const double* t3 = (const double*)p->tmp_vec[3];
  std::vector<double> hst((size_t)B * kSt), bn(B), rn(B), tolv(B);
  std::vector<int> run(B, 1), status(B, BIRK_OK), inner(B, 0), outer(B, 0);
  std::vector<char> done(B, 0);
  auto read_norms = [&](std::vector<double>& out) -> hipError_t {   // from the squares' partials
    hipLaunchKernelGGL(k_kv_reduce, dim3(B), dim3(256), 0, s, b.part, sg, b.dot);
    hipError_t ee = hipMemcpyAsync(hst.data(), b.dot, B * sizeof(double), hipMemcpyDeviceToHost, s);
    if (ee == hipSuccess) ee = hipStreamSynchronize(s);
    for (int i = 0; i < B; ++i) out[i] = std::isfinite(hst[i]) ? std::sqrt(std::max(hst[i], 0.0)) : NAN;
    return ee;
  };
  hipLaunchKernelGGL(k_kv_dot, dim3(nt2), dim3(256), 0, s, b.rhs, b.rhs, b.part, sg);
  if (read_norms(bn) != hipSuccess) return BIRK_ERR_DEVICE;
  int budget = o->max_iter;
  // iterations between host reads of the convergence state: 2, 2, 4, then 8 per cycle
  // (the preconditioned counts are small, and an iteration past convergence costs a
  // whole operator and preconditioner application)
  constexpr int kChunkIts = 8;
  birk_status result = BIRK_OK;
  for (int cycle = 0;; ++cycle) {
    // true residual r = rhs - K x in double, into r1 and r2 (x = 0 at first without x0)
    if (cycle == 0 && !o->use_x0) {
      e = hipMemcpyAsync(b.r1, b.rhs, 2 * n * sizeof(double), hipMemcpyDeviceToDevice, s);
      if (e == hipSuccess) e = hipMemcpyAsync(b.r2, b.rhs, 2 * n * sizeof(double), hipMemcpyDeviceToDevice, s);
      if (e != hipSuccess) return BIRK_ERR_DEVICE;
      rn = bn;
    } else {
      if (kkt_parts(p, jk, J, b.x, s) != hipSuccess) return BIRK_ERR_DEVICE;
      hipLaunchKernelGGL(k_kkt_out<true>, dim3(nt2), dim3(256), 0, s, b.x, t3, t1, h, b.rhs, b.st, b.r1, b.r2, b.part,
                         sg);
      if (read_norms(rn) != hipSuccess) return BIRK_ERR_DEVICE;
    }
    bool all = true;
    for (int i = 0; i < B; ++i) {
      run[i] = 0;
      if (done[i]) continue;
      if (!std::isfinite(rn[i])) {
        status[i] = BIRK_ERR_NONFINITE;
        done[i] = 1;
      } else if (rn[i] <= o->rtol * bn[i]) {
        status[i] = BIRK_OK;
        done[i] = 1;
      } else if (budget <= 0 || cycle > o->max_iter) {
        status[i] = BIRK_ERR_NOCONV;
        done[i] = 1;
      } else {
        run[i] = 1;
        all = false;
        outer[i] += 1;
        tolv[i] = std::min(0.5, 0.1 * o->rtol * bn[i] / rn[i]);
      }
    }
    if (all) break;
    // cycle start: y = M^{-1} r1, beta1, v = y / beta1
    e = hipMemcpyAsync(b.tol, tolv.data(), B * sizeof(double), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(b.run, run.data(), B * sizeof(int), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = kkt_prec(p, jk, J, h, b.r1, b.y, o->use_precond, false, s);
    if (e != hipSuccess) return BIRK_ERR_DEVICE;
    hipLaunchKernelGGL(k_kv_dot, dim3(nt2), dim3(256), 0, s, b.r1, b.y, b.part, sg);
    hipLaunchKernelGGL(k_mr_scalars<MR_INIT>, dim3(B), dim3(256), 0, s, b.st, b.part, b.tol, b.run, sg);
    hipLaunchKernelGGL(k_mr_update<true>, dim3(nt2), dim3(256), 0, s, b.v, b.y, (double*)nullptr,
                       (const double*)nullptr, (double*)nullptr, b.st, sg);
    // w: w_{k-1}, w1: w_{k-2}
    double *r1 = b.r1, *r2 = b.r2, *y = b.y, *w = b.w, *w1 = b.w1;
    bool cycle_done = false;
    int chunk_no = 0;
    while (!cycle_done && budget > 0) {
      const int want = chunk_no < 2 ? 2 : chunk_no < 3 ? 4 : kChunkIts;
      ++chunk_no;
      const int its = std::min(want, budget);
      for (int k = 0; k < its; ++k) {
        // y = K v - (beta / oldb) r1; alpha = v . y
        if (kkt_parts(p, jk, J, b.v, s) != hipSuccess) return BIRK_ERR_DEVICE;
        hipLaunchKernelGGL(k_kkt_out<false>, dim3(nt2), dim3(256), 0, s, b.v, t3, t1, h, r1, b.st, y, (double*)nullptr,
                           b.part, sg);
        hipLaunchKernelGGL(k_mr_scalars<MR_ALPHA>, dim3(B), dim3(256), 0, s, b.st, b.part, b.tol, b.run, sg);
        // y -= (alpha / beta) r2; then r1 <- r2, r2 <- y, and y = M^{-1} r2 in the buffer of r1
        hipLaunchKernelGGL(k_kkt_orth, dim3(nt2), dim3(256), 0, s, y, r2, h, b.st, o->use_precond ? r1 : nullptr, sg);
        double* t = r1;
        r1 = r2;
        r2 = y;
        y = t;
        if (kkt_prec(p, jk, J, h, r2, y, o->use_precond, true, s) != hipSuccess) return BIRK_ERR_DEVICE;
        // beta = sqrt(r2 . y)
        hipLaunchKernelGGL(k_kv_dot, dim3(nt2), dim3(256), 0, s, r2, y, b.part, sg);
        hipLaunchKernelGGL(k_mr_scalars<MR_GIVENS>, dim3(B), dim3(256), 0, s, b.st, b.part, b.tol, b.run, sg);
        // w_new = (v - eps w1 - delta w2) / gamma into w1's buffer; x += phi w_new; v = y / beta
        hipLaunchKernelGGL(k_mr_update<false>, dim3(nt2), dim3(256), 0, s, b.v, y, w1, w, b.x, b.st, sg);
        double* wn = w1;
        w1 = w;
        w = wn;
      }
      budget -= its;
      e = hipMemcpyAsync(hst.data(), b.st, hst.size() * sizeof(double), hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      if (e != hipSuccess) return BIRK_ERR_DEVICE;
      cycle_done = true;
      for (int i = 0; i < B; ++i)
        if (run[i] && hst[(size_t)i * kSt + S_ACTIVE] != 0.0) cycle_done = false;
    }
    for (int i = 0; i < B; ++i) {
      if (!run[i]) continue;
      inner[i] += (int)hst[(size_t)i * kSt + S_ITERS];
      if (!std::isfinite(hst[(size_t)i * kSt + S_PHIBAR])) {
        status[i] = BIRK_ERR_NONFINITE;
        done[i] = 1;
      }
    }
  }
  e = hipMemcpyAsync(chi, b.x, n * sizeof(double), hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && lam) e = hipMemcpyAsync(lam, b.x + n, n * sizeof(double), hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return BIRK_ERR_DEVICE;
  for (int i = 0; i < B; ++i) {
    if (result == BIRK_OK && status[i] != BIRK_OK) result = (birk_status)status[i];
    if (info) {
      if (info->status) info->status[i] = status[i];
      if (info->inner_iters) info->inner_iters[i] = inner[i];
      if (info->outer_iters) info->outer_iters[i] = outer[i];
      if (info->rel_resid_fp64) info->rel_resid_fp64[i] = bn[i] > 0 ? rn[i] / bn[i] : rn[i];
    }
  }
  return result;
}

}  // namespace birk
