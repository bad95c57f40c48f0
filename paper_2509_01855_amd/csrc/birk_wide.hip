// P^{-1} y and P^{-T} y for 9 <= n_x <= 12 (gfx950): the scans of birk_scan.hip with the maps
// composed on the matrix cores.
//
// At these sizes a node's K_k no longer fits one lane's registers, and carrying a map's columns
// through H_k on the vector unit reads all of H_k from LDS in every lane.  So here
//   * four lanes factor a node: lane q of the quad holds columns q, q + 4, q + 8 of K_k and of
//     w_k J_k (72 doubles); eliminated and substituted a column at a time, that column
//     broadcast to the quad by DPP; a wave forms H_k of sixteen nodes at once, in LDS;
//   * reduce: a tile's map M (columns of A, then b, in one 16 x 16 accumulator) goes through the
//     nodes by M <- M + H_k (M + y_k e^T) in three v_mfma_f64_16x16x4 a node.  Element
//     (l / 16 + 4 i, l % 16) of the accumulator is register i of lane l, which is also where
//     the instruction takes rows 4 i .. 4 i + 3 of its right operand from: M is fed back
//     without moving, and the left operand reads each element of H_k once;
//   * groups: the same product over the maps of 32 tiles, inclusive, in place;
//   * apply: the state (a component per lane) through the group maps before the tile's, its
//     predecessors' map, then node by node through H_k formed again.
// A tile is sixteen nodes times R.  Past an instance's end H_k = 0 and y_k = 0.
//
// Bound: the FP64 vector unit (forming H_k twice: 650 multiply-adds and 290 DPP moves a pass
// of sixteen nodes), then the matrix core (3 x 64 clocks a node).  The former scans (a table of
// H_k written once per J and read twice per product, sixteen lanes a node, five to seven
// levels) took, with one J at n_x = 12, 171 us at 257 nodes, 207 at 4097, 311 at 65537, 336 at
// 131072, and 433 at 65537 with J per node; these 22, 29, 87, 126 and 98.  P^{-T} at 65537
// nodes, J per node (a thread per sixteen nodes): 4070 -> 100.

#include <hip/hip_runtime.h>

#include <type_traits>

#include "birk_dense.h"
#include "birk_internal.h"

namespace birk {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

template <int NX>
struct Wide {
  static constexpr int F = NX * NX + NX;   // a map: columns 0..NX-1 of A, then b
  static constexpr int RS = 12;            // a row of H in a node's record, then 12 values
  // a record is 4 x odd (mod 32) doubles: the sixteen quads' writes fall on different banks
  static constexpr int REC = RS * NX + 12 + (((RS * NX + 12) / 4) % 2 ? 0 : 4);
};

// v of lane S of each quad (DPP quad_perm).
template <int S>
__device__ __forceinline__ double quad_bcast(double v) {
  const unsigned long long x = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)x, S * 0x55, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(x >> 32), S * 0x55, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Node at position pos of the lane's quad: H_k (G_k = H_k^T from J_k^T backwards) row-major
// and y_k into the record, zero past the instance; w_k.  A pivot that is non-finite or not
// above 1e-13 (1 + |w_k / 2| max |J_k|) sets *flag when given.
template <int NX, bool PN, bool BACK, typename T>
__device__ __forceinline__ void form_node(const ScanDesc& d, const double* __restrict__ J, const T* __restrict__ y,
                                          int64_t pos, double* __restrict__ rec, int* flag, double& w) {
  constexpr int NC = 3;
  const int q = (int)(threadIdx.x & 3);
  const int64_t Nn = d.Nn;
  const bool ok = pos < Nn;
  const int64_t p = ok ? pos : 0;
  const int64_t k = BACK ? Nn - 1 - p : p;
  w = d.w[k];
  const double wk = ok ? w : 0.0;
  double K[NC][NX], X[NC][NX], yv[NC], rp[NX];
  // the lane's column q of J (J^T), rows and groups of four columns rs and 4 cs further on;
  // opaque, so that no 36 values or addresses are carried from round to round in registers
  int64_t j0 = PN ? d.joff + k : d.jcoff, es = Nn, yo = d.off + k;
  asm volatile("" : "+v"(j0), "+s"(es), "+v"(yo));
  const int64_t cs = (PN ? es : 1) * (BACK ? NX : 1), rs = (PN ? es : 1) * (BACK ? 1 : NX);
  const double* jq = J + j0 + q * cs;
  const T* yq = y + yo + q * es;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const bool in = 4 * c + 3 < NX || q + 4 * c < NX;
    const double* jc = jq + (in ? 4 * c * cs : 0);
#pragma unroll
    for (int r = 0; r < NX; ++r) X[c][r] = jc[r * rs];
    yv[c] = (double)yq[in ? 4 * c * es : 0];
  }
  double jmax = 0.0;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const bool in = 4 * c + 3 < NX || q + 4 * c < NX;
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const double j = in ? X[c][r] : 0.0;
      jmax = fmax(jmax, fabs(j));
      X[c][r] = wk * j;
      K[c][r] = (r == q + 4 * c ? 1.0 : 0.0) - 0.5 * X[c][r];
    }
    rec[NX * 12 + q + 4 * c] = in && ok ? yv[c] : 0.0;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int r = 0; r < NX; ++r) asm volatile("" : "+v"(K[c][r]), "+v"(X[c][r]));
  double tiny = 0.0;
  bool bad = false;
  if (flag) {
    jmax = fmax(fmax(quad_bcast<0>(jmax), quad_bcast<1>(jmax)), fmax(quad_bcast<2>(jmax), quad_bcast<3>(jmax)));
    tiny = 1e-13 * (1.0 + 0.5 * fabs(wk) * jmax);
  }
  // forward elimination of [K | X], column P of K broadcast from its owner
  static_for<0, NX>([&](auto pc) {
    constexpr int P = decltype(pc)::value, G = P / 4;
    const double piv = quad_bcast<P & 3>(K[G][P]);
    bad = bad || !(fabs(piv) > tiny) || !isfinite(piv);
    rp[P] = recip(piv);
#pragma unroll
    for (int i = P + 1; i < NX; ++i) {
      const double f = quad_bcast<P & 3>(K[G][i]) * rp[P];
      // columns up to P of this group lose entries below their diagonal, which nothing reads
#pragma unroll
      for (int c = G; c < NC; ++c) K[c][i] -= f * K[c][P];
#pragma unroll
      for (int c = 0; c < NC; ++c) X[c][i] -= f * X[c][P];
    }
    // X and K are updated here: left until they are read, they keep every multiplier alive (60
    // values spilt to scratch, 1.4 times the time)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = P + 1; i < NX; ++i) {
        asm volatile("" : "+v"(X[c][i]));
        if (c >= G) asm volatile("" : "+v"(K[c][i]));
      }
  });
  if (flag && ok && bad) atomicOr(flag, 1);
  // back substitution, column P of the upper factor broadcast again
  static_for<0, NX>([&](auto pc) {
    constexpr int P = NX - 1 - decltype(pc)::value, G = P / 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) X[c][P] *= rp[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const double u = quad_bcast<P & 3>(K[G][i]);
#pragma unroll
      for (int c = 0; c < NC; ++c) X[c][i] -= u * X[c][P];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i) asm volatile("" : "+v"(X[c][i]));
  });
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int r = 0; r < NX; ++r) rec[r * 12 + q + 4 * c] = X[c][r];
}

template <int NX, bool PN, bool BACK, typename T>
__global__ __launch_bounds__(64, 2) void k_wide_reduce(const double* __restrict__ J, const T* __restrict__ y,
                                                       const ScanDesc* __restrict__ sd, const int2* __restrict__ tiles,
                                                       double* __restrict__ scan) {
  constexpr int REC = Wide<NX>::REC;
  __shared__ __align__(16) double sm[kWideNodes * REC];
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  if (t.y + 1 >= d.ntile) return;   // the last tile's map is not needed
  const int R = d.rounds, l = (int)threadIdx.x, lr = l & 15, g = l >> 4;
  const int64_t base = (int64_t)t.y * kWideNodes * R + (l >> 2);
  v4d m;
#pragma unroll
  for (int i = 0; i < 4; ++i) m[i] = g + 4 * i == lr && lr < NX ? 1.0 : 0.0;
  const int row = min(lr, NX - 1);
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    double w;
    form_node<NX, PN, BACK, T>(d, J, y, base + kWideNodes * j, sm + (l >> 2) * REC, nullptr, w);
    wave_sync();
#pragma unroll 4
    for (int i = 0; i < kWideNodes; ++i) {
      const double* p = sm + i * REC;
      double a[3], b[3];
      v4d c = m;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const double av = p[row * 12 + 4 * e + g], yv = p[NX * 12 + 4 * e + g];
        a[e] = lr < NX ? av : 0.0;
        const double ye = lr == NX ? yv : 0.0;
        b[e] = m[e] + (BACK ? 0.5 * ye : ye);
        if (BACK) c[e] += ye;
      }
#pragma unroll
      for (int e = 0; e < 3; ++e) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], b[e], c, 0, 0, 0);
      m = c;
    }
    wave_sync();
  }
  double* o = scan + d.tmap + (int64_t)t.y * Wide<NX>::F;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (lr <= NX && g + 4 * i < NX) o[lr * NX + g + 4 * i] = m[i];
}

// kWideGroup tiles of an instance per workgroup: inclusive maps within the group, in place, and
// the group's own map to d.gmap.  Four waves fetch the maps, one composes them (read from
// memory one ahead, every step of the chain waited for it: 34 us at 1024 tiles, now 12).
template <int NX>
__global__ __launch_bounds__(256) void k_wide_groups(double* __restrict__ scan, const ScanDesc* __restrict__ sd,
                                                    const int2* __restrict__ groups) {
  constexpr int F = Wide<NX>::F, PER = (kWideGroup * F + 255) / 256;
  __shared__ double sm[PER * 256];
  const int2 t = groups[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int l = (int)threadIdx.x, lr = l & 15, g = l >> 4;
  const int first = t.y * kWideGroup, n = min(kWideGroup, d.ntile - 1 - first);   // the last tile has no map
  double* tm = scan + d.tmap + (int64_t)first * F;
#pragma unroll
  for (int e = 0; e < PER; ++e) sm[l + 256 * e] = tm[min(l + 256 * e, n * F - 1)];
  __syncthreads();
  if (l >= 64) return;
  v4d m = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (lr <= NX && g + 4 * i < NX) m[i] = sm[lr * NX + g + 4 * i];
  double a[3], b[3];
  auto load = [&](int k) {
    const double* T = sm + k * F;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int x = min(g + 4 * e, NX - 1);
      const double av = T[x * NX + min(lr, NX - 1)], bv = T[NX * NX + x];
      a[e] = lr < NX && g + 4 * e < NX ? av : 0.0;
      b[e] = lr == NX && g + 4 * e < NX ? bv : 0.0;
    }
  };
  if (n > 1) load(1);
  for (int k = 1; k < n; ++k) {
    v4d c = {b[0], b[1], b[2], 0.0};
    const double a0 = a[0], a1 = a[1], a2 = a[2];
    if (k + 1 < n) load(k + 1);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, m[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, m[1], c, 0, 0, 0);
    m = __builtin_amdgcn_mfma_f64_16x16x4f64(a2, m[2], c, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (lr <= NX && g + 4 * i < NX) tm[(int64_t)k * F + lr * NX + g + 4 * i] = m[i];
  }
  double* gm = scan + d.gmap + (int64_t)t.y * F;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (lr <= NX && g + 4 * i < NX) gm[lr * NX + g + 4 * i] = m[i];
}

template <int NX, bool PN, bool BACK, typename T>
__global__ __launch_bounds__(64, 2) void k_wide_apply(const double* __restrict__ J, const T* __restrict__ y,
                                                      const ScanDesc* __restrict__ sd, const int2* __restrict__ tiles,
                                                      const double* __restrict__ scan, T* __restrict__ out,
                                                      T* __restrict__ jout, int* flag) {
  constexpr int REC = Wide<NX>::REC, F = Wide<NX>::F;
  __shared__ __align__(16) double sm[kWideNodes * REC];
  const int2 t = tiles[blockIdx.x];
  const ScanDesc& d = sd[t.x];
  const int R = d.rounds, l = (int)threadIdx.x, lr = l & 15;
  const int64_t base = (int64_t)t.y * kWideNodes * R + (l >> 2);
  const int row = min(lr, NX - 1);
  const bool keep_v = !BACK && jout;
  // the tile's start state: the groups before its own, then its predecessors' map
  double s = 0.0;
  const int ng = t.y / kWideGroup;
#pragma unroll 2
  for (int q = 0; q < ng; ++q) s = advance<NX>(scan + d.gmap + (int64_t)q * F, 1, s);
  if (t.y % kWideGroup) s = advance<NX>(scan + d.tmap + (int64_t)(t.y - 1) * F, 1, s);
#pragma unroll 1
  for (int j = 0; j < R; ++j) {
    double w;
    double* rec = sm + (l >> 2) * REC;
    form_node<NX, PN, BACK, T>(d, J, y, base + kWideNodes * j, rec, flag, w);
    wave_sync();
    double hn[NX], yn;
    auto load = [&](int i) {
      const double* p = sm + i * REC;
#pragma unroll
      for (int q = 0; q < NX; ++q) hn[q] = p[row * 12 + q];
      yn = p[NX * 12 + row];
    };
    load(0);
#pragma unroll 2
    for (int i = 0; i < kWideNodes; ++i) {
      double h[NX], v[2] = {0.0, 0.0};
      const double yi = yn;
#pragma unroll
      for (int q = 0; q < NX; ++q) h[q] = hn[q];
      if (i + 1 < kWideNodes) load(i + 1);
      __builtin_amdgcn_wave_barrier();
      const double u = BACK ? s + 0.5 * yi : s + yi;
      static_for<0, NX>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        v[q & 1] += h[q] * row_bcast<q>(u);
      });
      const double vs = v[0] + v[1];
      const double x = BACK ? yi + vs : u + 0.5 * vs;
      s += BACK ? x : vs;
      if (l < NX) {   // xi (x) in place of y, v in place of the first row of H
        double* p = sm + i * REC;
        p[NX * 12 + l] = x;
        if (keep_v) p[l] = vs;
      }
      __builtin_amdgcn_wave_barrier();
    }
    wave_sync();
    const int64_t pos = base + kWideNodes * j;
    if (pos < d.Nn) {
      int64_t o = d.off + (l & 3) * d.Nn + (BACK ? d.Nn - 1 - pos : pos);
      asm volatile("" : "+v"(o));   // as in form_node
      const double iw = 1.0 / w;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const int col = (l & 3) + 4 * c;
        if (col < NX) {
          out[o + 4 * c * d.Nn] = (T)rec[NX * 12 + col];
          if (keep_v) jout[o + 4 * c * d.Nn] = (T)(rec[col] * iw);
        }
      }
    }
    wave_sync();
  }
}

template <int NX, bool PN, bool BACK, typename T>
void launch(birk_plan* p, const ScanClass& sc, const double* J, const T* y, T* out, T* jout, int* flag, hipStream_t s) {
  const dim3 g(sc.n_tile), b(64);
  if (sc.n_group > 0) {
    hipLaunchKernelGGL((k_wide_reduce<NX, PN, BACK, T>), g, b, 0, s, J, y, sc.dev, sc.tiles, p->scan);
    hipLaunchKernelGGL(k_wide_groups<NX>, dim3(sc.n_group), dim3(256), 0, s, p->scan, sc.dev, sc.groups);
  }
  hipLaunchKernelGGL((k_wide_apply<NX, PN, BACK, T>), g, b, 0, s, J, y, sc.dev, sc.tiles, (const double*)p->scan, out,
                     jout, flag);
}

template <bool PN, bool BACK, typename T>
hipError_t dispatch(birk_plan* p, const ScanClass& sc, const double* J, const T* y, T* out, T* jout, int* flag,
                    hipStream_t s) {
  switch (sc.nx) {
    case 9: launch<9, PN, BACK, T>(p, sc, J, y, out, jout, flag, s); break;
    case 10: launch<10, PN, BACK, T>(p, sc, J, y, out, jout, flag, s); break;
    case 11: launch<11, PN, BACK, T>(p, sc, J, y, out, jout, flag, s); break;
    case 12: launch<12, PN, BACK, T>(p, sc, J, y, out, jout, flag, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// Rounds per tile: up to 1024 tiles, a wave per SIMD.  n_x = 12, one J: 512 tiles take 123 us at
// 65537 nodes and 207 at 131072, 1024 tiles 87 and 126, 2048 tiles 84 and 121; but where a
// batch fills the chip the longer chain of groups before a tile costs more (64 instances, 20 of
// them n_x = 12, mixed precision solve: 4741 us at 1024, 5042 at 2048).
// Longer instances, against a table of H_k made once per J and a hierarchical scan over it:
// P^{-1} at 2^20 + 1 nodes, n_x = 9, 10, 12, one J: 681, 757, 804 us (1057, 1257, 1786), J per
// node: 912, 975, 1006 (2470, 2971, 4157).  A solve of 12 iterations at 2^19 + 1 nodes, where the
// table is made once: n_x = 12, one J 10.5 ms (12.1), J per node 11.7 (13.1); n_x = 9, one J 8.7
// (8.8), but J per node 9.9 against 9.4.
int wide_rounds(int64_t Nn) {
  const int64_t per_round = (int64_t)kWideNodes * 1024;
  return (int)((Nn + per_round - 1) / per_round);
}

template <typename T>
hipError_t wide_inverse(birk_plan* p, const ScanClass& sc, int per_node, const double* J, const T* y, T* out, T* jout,
                        int* flag, hipStream_t s) {
  return per_node ? dispatch<true, false, T>(p, sc, J, y, out, jout, flag, s)
                  : dispatch<false, false, T>(p, sc, J, y, out, jout, flag, s);
}

hipError_t wide_inverse_t(birk_plan* p, const ScanClass& sc, int per_node, const double* J, const double* y,
                          double* out, hipStream_t s) {
  return per_node ? dispatch<true, true, double>(p, sc, J, y, out, nullptr, nullptr, s)
                  : dispatch<false, true, double>(p, sc, J, y, out, nullptr, nullptr, s);
}

template hipError_t wide_inverse<double>(birk_plan*, const ScanClass&, int, const double*, const double*, double*,
                                         double*, int*, hipStream_t);
template hipError_t wide_inverse<float>(birk_plan*, const ScanClass&, int, const double*, const float*, float*, float*,
                                        int*, hipStream_t);

}  // namespace birk
