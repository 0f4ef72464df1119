// Device helpers shared by the tendency kernels: reciprocal, the centred
// interpolations of the advecting velocity and the WENO reconstructions of
// orders 5, 7 and 9
// (finite-volume appendix of arXiv 2502.14148: upwind-biased WENO5 with the
// WENO-Z weights of Borges et al. 2008, q = 2; Jiang & Shu 1996 candidate
// stencils and smoothness indicators).
#pragma once

#include <hip/hip_runtime.h>

#include "weno_coeffs.h"

namespace oc {
namespace tz {

enum { SCHEME_NONE = 0, SCHEME_WENOZ = 1, SCHEME_LINEAR = 2 };

__device__ inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double rcp(double x) {
  // hardware estimate refined by two Newton steps (about 1 ulp)
  double r = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, r, 1.0);
  r = __builtin_fma(r, e, r);
  e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, e, r);
}

__device__ inline float fmad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fmad(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <class T>
__device__ inline T interp4(T a0, T a1, T a2, T a3) {
  return ((a1 + a2) * T(7) - (a0 + a3)) * T(1.0 / 12.0);
}

// Reconstruction at the interface between q_{-1} and q_0 from the six values
// q_{-3..2}; `vel` selects the upwind side.
//
// WENO-Z form used here (equal to the textbook form in exact arithmetic):
// with the upwind-ordered stencil (a, b, c, d, e), twice its differences,
// c2 = 2 (c - b), n3 = 2 (c - d), and their differences t0 = c2 + 2 (a - b),
// t1 = -n3 - c2, t2 = 2 (e - d) + n3 (each rounded as its half would be),
//   * candidates as deviations from the upwind neighbour c:
//       4 (r0 - c) = c2 + 2/3 t0, 4 (r1 - c) = c2 + 2/3 t1 = 1/3 (c2 - 2 n3),
//       4 (r2 - c) = -(n3 + 1/3 t2);
//   * four times the Jiang-Shu indicators plus eps, as t (4/3 t + n) + n^2 +
//     4 eps: s0 with (t0, c2), s1 with (t1, c2), s2 with (t2, n3)
//     (the weights only see ratios, so the common factor drops out);
//   * WENO-Z weights d_k (1 + (tau / s_k)^2), tau = |s0 - s2|, multiplied
//     through by 10 s1^2:  a0 = s1^2 + (tau s1 / s0)^2, 6 a1 with a1 = s1^2 +
//     tau^2, 3 a2 with a2 = s1^2 + (tau s1 / s2)^2, both quotients from the one
//     reciprocal of s0 s2;
//   * W = c + (a0 (r0 - c) + 6 a1 (r1 - c) + 3 a2 (r2 - c)) / (a0 + 6 a1 + 3 a2).
// Two reciprocals in 45 operations (46 in FP32, of shorter encodings; 51 and three
// reciprocals with one each for s0 and s2, which cost 2 to 4 % of a whole step).
// FP32 range: next to flat stencils s0 s2 and s1^2 are 16 eps^2, normal for
// eps above 2.72e-20 (with undoubled differences, in 45 operations, eps had to be
// above 1.1e-19); tau s1 / s_k stays below 1.8e19 for indicators up to
// ~1e2 in the field's units squared next to an exactly flat stencil at eps =
// 1e-15.
// Four steps at 256^3 FP32, two at 96x64x128 FP64: 10.04 ms and 671 us; undoubled
// differences 10.07 and 671; both factors in the candidates 10.13 and 669, both
// on the weights 10.04 and 680; indicators scaled by two multiplications 10.15
// and 677.
template <class T, int SCHEME>
__device__ inline T rec6(T m3, T m2, T m1, T p0, T p1, T p2, T vel, T eps) {
  const bool pos = vel > T(0);
  const T a = pos ? m3 : p2;
  const T b = pos ? m2 : p1;
  const T c = pos ? m1 : p0;
  const T d = pos ? p0 : m1;
  const T e = pos ? p1 : m2;
  if (SCHEME == SCHEME_LINEAR)
    return (T(2) * a - T(13) * b + T(47) * c + T(27) * d - T(3) * e) * T(1.0 / 60.0);
  const T cc = T(2) * c, d1 = a - b, d4 = e - d, e4 = T(4) * eps;
  const T c2 = fmad(T(-2), b, cc), n3 = fmad(T(-2), d, cc);
  const T t0 = fmad(T(2), d1, c2), t1 = -n3 - c2, t2 = fmad(T(2), d4, n3);
  const T q2 = fmad(c2, c2, e4), q3 = fmad(n3, n3, e4);
  const T s0 = fmad(t0, fmad(T(4.0 / 3.0), t0, c2), q2);
  const T s1 = fmad(t1, fmad(T(4.0 / 3.0), t1, c2), q2);
  const T s2 = fmad(t2, fmad(T(4.0 / 3.0), t2, n3), q3);
  const T tau = fabs(s0 - s2);
  const T s1s = s1 * s1;
  const T g = tau * s1 * rcp(s0 * s2);
  const T g0 = g * s2, g2 = g * s0;
  const T a0 = fmad(g0, g0, s1s), a1 = fmad(tau, tau, s1s), a2 = fmad(g2, g2, s1s);
  // 4 (W - c); the weights' factors 6 and 3 where the type encodes them best:
  // FP32 multiply-adds carry a literal, FP64 constants take registers
  const T e0 = fmad(T(2.0 / 3.0), t0, c2);
  T num, den;
  if constexpr (sizeof(T) == 4) {
    const T b1 = T(6) * a1, b2 = T(3) * a2;
    const T e1 = fmad(T(2.0 / 3.0), t1, c2), e2 = fmad(T(1.0 / 3.0), t2, n3);
    num = fmad(a0, e0, fmad(b1, e1, -(b2 * e2)));
    den = a0 + b1 + b2;
  } else {
    const T b1 = T(2) * a1;
    const T e1 = fmad(T(-2), n3, c2), e2 = fmad(T(3), n3, t2);
    num = fmad(a0, e0, fmad(-a2, e2, b1 * e1));
    den = fmad(T(3), b1 + a2, a0);
  }
  return fmad(T(0.25), num * rcp(den), c);
}

// Centred reconstruction of order 2R - 2 at the midpoint of a[R-2] and
// a[R-1] from a[0 .. 2R-3] (order 4: interp4).
template <class T, int R>
__device__ inline T interpc(const T* a) {
  if constexpr (R == 3) {
    return interp4(a[0], a[1], a[2], a[3]);
  } else {
    using C = WenoCoef<R>;
    T s = T(0);
#pragma unroll
    for (int o = 0; o < R - 1; ++o) s += T(C::centred[o]) * (a[o] + a[2 * R - 3 - o]);
    return s;
  }
}

// Reconstruction of order 2R - 1 (R = 4, 5) at the interface between q[R-1]
// and q[R] from q[0 .. 2R-1]; `vel` selects the upwind side.  Every
// combination is taken on deviations from the upwind neighbour of the
// interface, and the indicators on differences of neighbouring values, so
// that a large mean of the data does not cost precision.
// A value the optimiser cannot trace back to the load that produced it: a
// choice between two elements of a register array stays a choice between
// two values instead of becoming a dynamically indexed array access.
template <class T>
__device__ inline T opaque(T x) {
  asm("" : "+v"(x));
  return x;
}

template <class T, int SCHEME, int R>
__device__ inline T recw(const T* q, T vel, T eps) {
  using C = WenoCoef<R>;
  constexpr int N = 2 * R - 1;
  const bool pos = vel > T(0);
  T v[N];
#pragma unroll
  for (int t = 0; t < N; ++t) {
    const T a = opaque(q[t]), b = opaque(q[2 * R - 1 - t]);
    v[t] = pos ? a : b;
  }
  const T base = v[R - 1];
  T dv[N];
#pragma unroll
  for (int t = 0; t < N; ++t) dv[t] = v[t] - base;
  if constexpr (SCHEME == SCHEME_LINEAR) {
    T s = T(0);
#pragma unroll
    for (int t = 0; t < N; ++t)
      if (t != R - 1) s += T(C::full[t]) * dv[t];
    return base + s;
  } else {
    T dl[N - 1];
#pragma unroll
    for (int t = 0; t < N - 1; ++t) dl[t] = v[t + 1] - v[t];
    T beta[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      T b = T(0);
#pragma unroll
      for (int m = 0; m < R - 1; ++m) {
        T y = dl[k + m];
#pragma unroll
        for (int t = m + 1; t < R - 1; ++t) y += T(C::Lt[k][m][t]) * dl[k + t];
        b += T(C::D[k][m]) * y * y;
      }
      beta[k] = b;
    }
    T tau = T(0);
#pragma unroll
    for (int k = 0; k < R; ++k) tau += T(C::tau[k]) * beta[k];
    tau = fabs(tau);
    T num = T(0), den = T(0);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      T rk = T(0);
#pragma unroll
      for (int t = 0; t < R; ++t)
        if (k + t != R - 1) rk += T(C::cand[k][t]) * dv[k + t];
      const T qk = tau * rcp(beta[k] + eps);
      const T a = T(C::ideal[k]) * (T(1) + qk * qk);
      num += a * rk;
      den += a;
    }
    return base + num * rcp(den);
  }
}

}  // namespace tz
}  // namespace oc
