// Wave helpers: lane broadcasts, the node blocks' LU and affine maps of the preconditioner
// scans, sums.

#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

namespace birk {

// Lane P of each row of sixteen lanes, broadcast across its row (DPP row_newbcast: a VALU
// move, in place of an LDS permute), for a double.
template <int P>
__device__ __forceinline__ double row_bcast(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + P, 0xF, 0xF, true);
}

// f(std::integral_constant<int, P>) for P = B .. E - 1, in order (compile-time lane indices).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// 1 / x from the hardware estimate and two Newton steps (within an ulp of the quotient;
// several times cheaper than a division).
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}

// Unpivoted LU of K = I - (w/2) Jk in place, with reciprocal pivots.  K is strongly
// diagonally dominant on the configurations of interest (w_k <= ~pi/N).  A pivot that
// is non-finite, or not above 1e-13 times the scale 1 + |w/2| max|J_k| of K, marks K as
// numerically singular in *flag.
template <int NX>
__device__ __forceinline__ void lu_kmat(double (&K)[NX][NX], double (&rp)[NX], int* flag, double scale) {
#pragma unroll
  for (int p = 0; p < NX; ++p) {
    const double piv = K[p][p];
    if (flag && (!(fabs(piv) > 1e-13 * scale) || !isfinite(piv))) atomicOr(flag, 1);
    rp[p] = recip(piv);
#pragma unroll
    for (int i = p + 1; i < NX; ++i) {
      const double f = K[i][p] * rp[p];
      K[i][p] = f;
#pragma unroll
      for (int j = p + 1; j < NX; ++j) K[i][j] -= f * K[p][j];
    }
  }
}

template <int NX>
__device__ __forceinline__ void lu_solve(const double (&K)[NX][NX], const double (&rp)[NX], double (&x)[NX]) {
#pragma unroll
  for (int i = 1; i < NX; ++i) {
#pragma unroll
    for (int j = 0; j < i; ++j) x[i] -= K[i][j] * x[j];
  }
#pragma unroll
  for (int i = NX - 1; i >= 0; --i) {
#pragma unroll
    for (int j = i + 1; j < NX; ++j) x[i] -= K[i][j] * x[j];
    x[i] *= rp[i];
  }
}

// LDS written by some lanes of a wave and read by others.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_wave_barrier();
  __threadfence_block();
  __builtin_amdgcn_wave_barrier();
}

// s <- A s + b for the map at m (element (r, c) of [A | b] at m[(c NX + r) fs]); component r
// of the state in lane r of every row of sixteen.
template <int NX>
__device__ __forceinline__ double advance(const double* __restrict__ m, int64_t fs, double s) {
  const int rr = min((int)(threadIdx.x & 15), NX - 1);
  double row[NX], acc = m[(NX * NX + rr) * fs];
#pragma unroll
  for (int q = 0; q < NX; ++q) row[q] = m[(q * NX + rr) * fs];
  static_for<0, NX>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    acc += row[q] * row_bcast<q>(s);
  });
  return acc;
}

template <int NX>
struct Aff {
  double A[NX][NX];
  double b[NX];
};

// v of the lane that DPP control CTRL selects, in the rows that ROWMASK enables
// (row_shr:n = 0x110 + n, row_bcast:15 = 0x142, row_bcast:31 = 0x143); a lane with no
// source keeps its own v.
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long x = __builtin_bit_cast(unsigned long long, v);
  const int lo = (int)(unsigned)x, hi = (int)(unsigned)(x >> 32);
  const int rlo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWMASK, 0xF, false);
  const int rhi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWMASK, 0xF, false);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)rhi << 32) | (unsigned)(unsigned)rlo);
}

// Where take: m <- m o e, e = the map of the source lane (applied first):
// (A_m A_e, A_m b_e + b_m).  e arrives one row at a time.
template <int NX, int CTRL, int ROWMASK>
__device__ __forceinline__ void scan_step(Aff<NX>& m, bool take) {
  double nA[NX][NX], nb[NX];
#pragma unroll
  for (int r = 0; r < NX; ++r) {
    nb[r] = m.b[r];
#pragma unroll
    for (int c = 0; c < NX; ++c) nA[r][c] = 0.0;
  }
#pragma unroll
  for (int q = 0; q < NX; ++q) {
    double er[NX];
#pragma unroll
    for (int c = 0; c < NX; ++c) er[c] = dpp_f64<CTRL, ROWMASK>(m.A[q][c]);
    const double eb = dpp_f64<CTRL, ROWMASK>(m.b[q]);
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const double a = m.A[r][q];
#pragma unroll
      for (int c = 0; c < NX; ++c) nA[r][c] += a * er[c];
      nb[r] += a * eb;
    }
  }
  if (take) {
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      m.b[r] = nb[r];
#pragma unroll
      for (int c = 0; c < NX; ++c) m.A[r][c] = nA[r][c];
    }
  }
}

// Inclusive scan of the lanes' maps in lane order: lane l ends with m_l o ... o m_0.
// Rows of 16 lanes scan by row_shr 1, 2, 4, 8; row_bcast:15 then row_bcast:31 carry the
// totals of the earlier rows.
template <int NX>
__device__ __forceinline__ void wave_scan(Aff<NX>& m) {
  const int l = (int)(threadIdx.x & 63), lr = l & 15;
  scan_step<NX, 0x111, 0xF>(m, lr >= 1);
  scan_step<NX, 0x112, 0xF>(m, lr >= 2);
  scan_step<NX, 0x114, 0xF>(m, lr >= 4);
  scan_step<NX, 0x118, 0xF>(m, lr >= 8);
  scan_step<NX, 0x142, 0xA>(m, ((l >> 4) & 1) != 0);
  scan_step<NX, 0x143, 0xC>(m, l >= 32);
}

// Sum of v over the wave, in its last lane: row_shr 1, 2, 4, 8 (DPP controls 0x110 + n) sum
// each row of 16, row_bcast 15 and 31 (0x142, 0x143) carry the rows' sums up; a lane
// without a source adds zero.  VALU moves, no LDS permutes.
template <int CTRL, int ROWS>
__device__ __forceinline__ double add_dpp(double v) {
  const unsigned long long x = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)x, CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(x >> 32), CTRL, ROWS, 0xF, false);
  return v + __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_sum_last(double v) {
  v = add_dpp<0x111, 0xF>(v);
  v = add_dpp<0x112, 0xF>(v);
  v = add_dpp<0x114, 0xF>(v);
  v = add_dpp<0x118, 0xF>(v);
  v = add_dpp<0x142, 0xA>(v);
  return add_dpp<0x143, 0xC>(v);
}

// v of the wave's last lane, in all.
__device__ __forceinline__ double lane63(double v) {
  const unsigned long long x = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, 63);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), 63);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

}  // namespace birk
