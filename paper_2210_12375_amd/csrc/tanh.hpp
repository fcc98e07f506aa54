// tanh of the neural fields, in float and double.  M supplies what the
// hardware does in one instruction (approximate reciprocal and exp2), so that
// the arithmetic around it can be checked on a host.
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define BODE_TANH __device__ __forceinline__
#else
#define BODE_TANH inline
#endif

namespace bode {

// About one ulp: x + x^3 q(x^2) below 1 (q interpolates at Chebyshev nodes,
// the last bits of its first two coefficients chosen for the least mean error
// in float arithmetic), 1 - 2 e / (1 + e) with e = exp(-2 |x|) above.
// Measured over 2^18 points in each of 17 ranges from 0.01 to 100: at most
// 1.24 ulp, rms 0.29 to 0.31 below 1 and 0.36 above, falling to 0.29.  The
// library's tanhf, which the padded widths had: 1.40, 0.29 to 0.43 and 0.34;
// with a polynomial of degree 4 to 0.6 only: 1.61 and 0.46 (1 % of the time of
// 40,000 instances of 65->256->256->64 less).
template <class M>
BODE_TANH float tanh32(float x) {
  const float ax = std::fabs(x), z = x * x;
  const float e = M::exp2(ax * -2.8853900817779268f);
  const float big = std::fma(-2.f * e, M::rcp(1.f + e), 1.f);
  float q = std::fma(0.00014279318565968424f, z, -0.0009235008619725704f);
  q = std::fma(q, z, 0.0032068034633994102f);
  q = std::fma(q, z, -0.008697847835719585f);
  q = std::fma(q, z, 0.021829549223184586f);
  q = std::fma(q, z, -0.05396341532468796f);
  q = std::fma(q, z, 0.13333308696746826f);
  q = std::fma(q, z, -0.3333333134651184f);
  return std::copysign(ax < 1.f ? std::fma(ax, z * q, ax) : big, x);
}

// e^z - 1, z = -2 |x|, as a sum of two doubles and the quotient
// -(e^z - 1) / (2 + (e^z - 1)) corrected by its residual: mean error 0.25
// ulp, largest 0.8 (2^20 points in each of nine ranges of |x| from 1e-300 to
// 700; the library's: 0.25 to 0.28, largest 0.86).  89 instructions for
// its 187, in the two hidden layers of every evaluation: 1000 instances of
// 65->256->256->64 568 -> 521 us, 250 instances of
// 33->128->128->32 with adjoint 1.03 -> 0.99 ms.  The polynomial (e^r - 1 - r) / r^2 on
// |r| <= ln 2 / 2 interpolates at Chebyshev nodes, to 2^-60 of e^r - 1.
template <class M>
BODE_TANH double tanh64(double x) {
#if defined(__clang__)
#pragma clang fp contract(off)
#endif
  const double y = std::fabs(x), z = -2.0 * y;
  const double k = std::rint(z * 1.4426950408889634);
  const double r1 = std::fma(-k, 0.6931471526622772, z);  // exact
  const double r = std::fma(-k, 2.7897668087737545e-08, r1);
  const double rl = std::fma(-k, 2.7897668087737545e-08, r1 - r);
  double q = 2.091468696808688e-09;
  q = std::fma(q, r, 2.5105217004720745e-08);
  q = std::fma(q, r, 2.75572736431103e-07);
  q = std::fma(q, r, 2.7557255400206422e-06);
  q = std::fma(q, r, 2.4801587325547743e-05);
  q = std::fma(q, r, 0.00019841269874820627);
  q = std::fma(q, r, 0.0013888888888883748);
  q = std::fma(q, r, 0.008333333333326136);
  q = std::fma(q, r, 0.04166666666666667);
  q = std::fma(q, r, 0.1666666666666667);
  q = std::fma(q, r, 0.5);
  // e^r - 1 = p + pl, e^z - 1 = m + ml
  const double w = (r * r) * q, p = r + w;
  const double pl = ((r - p) + w) + rl;
  const double s = M::exp2i(int(k)), s1 = s - 1.0, b = s * p, m = s1 + b;
  const double bb = m - s1;
  const double ml =
      std::fma(s, pl, (s1 - (m - bb)) + (b - bb)) + (s - (s1 + 1.0));
  const double d = 2.0 + m, dl = (m - (d - 2.0)) + ml;
  double v = M::rcp(d);
  v = std::fma(std::fma(-d, v, 1.0), v, v);
  v = std::fma(std::fma(-d, v, 1.0), v, v);
  double t = -m * v;
  t = std::fma(std::fma(-dl, t, std::fma(-d, t, -m) - ml), v, t);
  t = y > 40.0 ? 1.0 : t;  // (infinities too)
  return std::copysign(t, x);
}

#if defined(__HIPCC__)
struct HwMath {
  __device__ static __forceinline__ float rcp(float x) {
    return __builtin_amdgcn_rcpf(x);
  }
  __device__ static __forceinline__ double rcp(double x) {
    return __builtin_amdgcn_rcp(x);
  }
  __device__ static __forceinline__ float exp2(float x) {
    return __builtin_amdgcn_exp2f(x);
  }
  __device__ static __forceinline__ double exp2i(int k) {
    return ldexp(1.0, k);
  }
};
#endif

}  // namespace bode
