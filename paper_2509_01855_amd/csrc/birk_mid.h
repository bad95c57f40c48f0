// The coefficient stencil between the two DCT-I of a product, on packed component pairs,
// for kernels that form it from the DFT values Y_k of the even extension (C v = Y / 2).
//
// Forward (eq:c_k=bydef with the alias of eq:chatk=): d_k = (-1)^k c^_k / e_k from the
// Chebyshev coefficients a_k = (-1)^k e_k Y_k / N.  d_0 = 0 here: c^_0 adds a constant to
// every output, and is a weighted sum of Y (c0_weight).
// Transpose: q = S M^T S p with p = Y / 2.

#pragma once

#include "birk_dense.h"
#include "birk_fft.h"

namespace birk {

// Reciprocal of a positive integer-valued x: in double the hardware estimate refined by two
// Newton steps (within an ulp of 1/x, several times cheaper than a division), which double-floats
// take too (their own division is two float divisions and a correction); a plain division for
// float.
template <typename T>
__device__ __forceinline__ T recip_int(T x) {
  return T(1) / x;
}
template <>
__device__ __forceinline__ double recip_int<double>(double x) {
  return recip(x);
}
template <>
__device__ __forceinline__ df32 recip_int<df32>(df32 x) {
  return df32(recip((double)x));
}

// p a for p a power of two: exact, and for double-floats two products instead of a rounded one.
template <typename T>
__device__ __forceinline__ T pow2_times(float p, T a) {
  if constexpr (std::is_floating_point<T>::value) return T(p) * a;
  else return T(p * a.hi, p * a.lo);
}

// d_k for 1 <= k <= N from Y_{k-1} and Y_{k+1} (Yp is not used at k = N):
// invN = 1/N, inv4N1 = 1/(4 (N + 1)).  One component, then a pair.
template <typename T>
struct FwdStencil {
  T i2k, cp, sc;
  __device__ __forceinline__ FwdStencil(int k, int N, T invN, T inv4N1) {
    i2k = recip_int<T>(T(2 * k));   // 1/(2k); at k = 1 also e_0 = 1/2
    cp = T(0);
    if (k < N) cp = (k + 1 == N) ? pow2_times(0.5f, i2k) - inv4N1 : i2k;
    sc = pow2_times(k == N ? 2.0f : 1.0f, invN);
  }
  __device__ __forceinline__ T operator()(T Ym, T Yp) const { return (cp * Yp - i2k * Ym) * sc; }
};
template <typename T>
__device__ __forceinline__ cplx<T> mid_fwd(int k, int N, cplx<T> Ym, cplx<T> Yp, T invN, T inv4N1) {
  const FwdStencil<T> f(k, N, invN, inv4N1);
  return fast::mk<T>(f(Ym.x, Yp.x), f(Ym.y, Yp.y));
}

// N times the weight of Y_k in c^_0.
__device__ __forceinline__ double c0_weight(int k, int N) {
  if (k == 0) return 0.5;
  if (k == 1) return 0.25;
  const double r = -recip_int<double>(((double)k - 1.0) * ((double)k + 1.0));
  return k == N ? 0.5 * r : r;
}

// q_j for 0 <= j <= N from Y_0, Y_{j-1}, Y_{j+1} (Yp is not used at j = N
// nor Ym at j <= 1): inv2N1 = 1/(2 (N + 1)).  A pair branches on the two first j once, before the
// reciprocals (N = 100002, six components, double: J^T x 79.7 us with a choice in each component,
// 78.4 so).
template <typename T>
struct TrStencil {
  T cm, cp, c0;
  int j;
  __device__ __forceinline__ TrStencil(int j_, int N, T inv2N1) : j(j_) {
    const T rm = recip_int<T>(T(max(j, 2) - 1)), rp = recip_int<T>(T(j + 1));
    cm = pow2_times(0.5f, rm);
    cp = pow2_times(0.5f, rp);
    if (j == N) {
      cm -= inv2N1;
      cp = T(0);
    }
    c0 = rm * rp;
  }
  __device__ __forceinline__ T operator()(T Y0, T Ym, T Yp) const {
    if (j < 2) return pow2_times(j == 0 ? 0.5f : 0.125f, Y0 - Yp);
    return inner(Y0, Ym, Yp);
  }
  __device__ __forceinline__ T inner(T Y0, T Ym, T Yp) const {   // j >= 2
    return pow2_times(0.5f, cm * Ym - cp * Yp - c0 * Y0);
  }
};
template <typename T>
__device__ __forceinline__ cplx<T> mid_tr(int j, int N, cplx<T> Y0, cplx<T> Ym, cplx<T> Yp, T inv2N1) {
  if (j < 2) {
    const float h = j == 0 ? 0.5f : 0.125f;
    return fast::mk<T>(pow2_times(h, Y0.x - Yp.x), pow2_times(h, Y0.y - Yp.y));
  }
  const TrStencil<T> f(j, N, inv2N1);
  return fast::mk<T>(f.inner(Y0.x, Ym.x, Yp.x), f.inner(Y0.y, Ym.y, Yp.y));
}

}  // namespace birk
