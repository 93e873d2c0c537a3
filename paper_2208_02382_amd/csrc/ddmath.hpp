// Double-double arithmetic on the device.
//
// A value is an unevaluated sum hi + lo of two doubles (about 106 bits).  Error-free
// transformations: Knuth's TwoSum and the FMA form of the exact product (a*b = p + fma(a,b,-p)).
// Elementary functions (table-driven argument reduction, then short series):
//   log  -- a = 2^e m, m in [1, 2); c = 1 + k/1024 nearest m; log a = e ln2 + log c
//           + 2 atanh(t), t = (m - c)/(m + c), |t| <= 1/4096, atanh by 5 series terms.
//   atan -- a > 1 uses pi/2 - atan(1/a); c = k/1024 nearest the argument x in [0, 1];
//           atan x = atan c + atan(t), t = (x - c)/(1 + x c), |t| <= 1/2048, 5 series terms.
//   sqrt -- from the double reciprocal square root, one correction in double and one beyond it.
// The tables log(1 + k/1024) and atan(k/1024) (dd_tables.hpp) are double pairs from 60-digit
// mpmath; series truncation errors are below 1e-33 relative.
//
// The corner functions are bound by the number of these operations (the float64 vector rate), so
// an operation is left out where it does not carry a bit of the result: the last series terms are
// summed in double and products inside the series are not renormalised, the reciprocals come from
// the hardware's refined ones (each is corrected), the remainder of a quotient or root is one fma
// (exact once the quotient or root is within an ulp), and sums of two numbers of one sign use the
// short addition (whose error bound is then that of the long one; where the two may cancel, the long
// one stays).  Largest relative errors of the host build over 3000 arguments against 60-digit mpmath
// (30000 for the last two), and of the same with every operation carried wide: log 3.9e-32 and
// 3.9e-32, in 1 - [2^-11, 2^-9] 1.8e-30 and 1.8e-30 (the rounding of the table), atan2 2.5e-32 and
// 2.9e-32, sqrt 3.6e-32 and 7.9e-32, quotient 1.3e-32 and 1.5e-32; the corner function F as close or
// closer on six cell shapes, and the same double in every cell of a 64 x 48 x 64 octant up to an aspect
// of 1e5.  The device build is held to the same bounds.  k_igf_corners at 64^3: 28.2 us wide, 15.4 us
// so.
// No fast-math and no contraction: TwoSum and FastTwoSum are exact only if every + and - is
// rounded on its own.  hipcc contracts a*b + c into an fma by default in device code, which
// silently turns these sequences into plain double arithmetic, so contraction is switched off
// for every translation unit that includes this header (and igf.hip is also built with
// -ffp-contract=off).  The only fused multiply-adds are the explicit std::fma calls.
#pragma once
#pragma clang fp contract(off)
#include <hip/hip_runtime.h>
#include <cmath>

#include "dd_tables.hpp"

// Callable from host code as well, so that the arithmetic can be unit-tested on a CPU.
#define PIC_HD __host__ __device__

namespace pic {

struct ddv {
  double hi, lo;
};

PIC_HD __forceinline__ ddv dd_make(double a) { return {a, 0.0}; }

PIC_HD __forceinline__ ddv two_sum(double a, double b) {
  double s = a + b;
  double bb = s - a;
  double e = (a - (s - bb)) + (b - bb);
  return {s, e};
}

PIC_HD __forceinline__ ddv fast_two_sum(double a, double b) {
  double s = a + b;
  double e = b - (s - a);
  return {s, e};
}

PIC_HD __forceinline__ ddv two_prod(double a, double b) {
  double p = a * b;
  return {p, std::fma(a, b, -p)};
}

PIC_HD __forceinline__ ddv dd_add(ddv a, ddv b) {
  ddv s = two_sum(a.hi, b.hi);
  ddv t = two_sum(a.lo, b.lo);
  s.lo += t.hi;
  s = fast_two_sum(s.hi, s.lo);
  s.lo += t.lo;
  return fast_two_sum(s.hi, s.lo);
}

// Short form: the low parts are added in double.  Its error is bounded by 3 2^-106 (|a| + |b|), as
// that of the form above by 3 2^-106 |a + b|: for a and b of one sign.
PIC_HD __forceinline__ ddv dd_add_s(ddv a, ddv b) {
  ddv s = two_sum(a.hi, b.hi);
  s.lo += a.lo + b.lo;
  return fast_two_sum(s.hi, s.lo);
}

// short addition for |a| >= |b|, of one sign or b far smaller
PIC_HD __forceinline__ ddv dd_add_f(ddv a, ddv b) {
  ddv s = fast_two_sum(a.hi, b.hi);
  s.lo += a.lo + b.lo;
  return fast_two_sum(s.hi, s.lo);
}

// the long addition for |a| >= |b| or a = 0
PIC_HD __forceinline__ ddv dd_add_o(ddv a, ddv b) {
  ddv s = fast_two_sum(a.hi, b.hi);
  ddv t = two_sum(a.lo, b.lo);
  s.lo += t.hi;
  s = fast_two_sum(s.hi, s.lo);
  s.lo += t.lo;
  return fast_two_sum(s.hi, s.lo);
}

PIC_HD __forceinline__ ddv dd_neg(ddv a) { return {-a.hi, -a.lo}; }
PIC_HD __forceinline__ ddv dd_sub(ddv a, ddv b) { return dd_add(a, dd_neg(b)); }

PIC_HD __forceinline__ ddv dd_mul(ddv a, ddv b) {
  ddv p = two_prod(a.hi, b.hi);
  p.lo = std::fma(a.hi, b.lo, std::fma(a.lo, b.hi, p.lo));
  return fast_two_sum(p.hi, p.lo);
}

// the product left as it comes, its lo up to an ulp of hi
PIC_HD __forceinline__ ddv dd_mul_u(ddv a, ddv b) {
  ddv p = two_prod(a.hi, b.hi);
  p.lo += std::fma(a.hi, b.lo, a.lo * b.hi);
  return p;
}

PIC_HD __forceinline__ ddv dd_sqr(ddv a) {
  ddv p = two_prod(a.hi, a.hi);
  p.lo = std::fma(a.hi + a.hi, a.lo, p.lo);
  return fast_two_sum(p.hi, p.lo);
}

PIC_HD __forceinline__ ddv dd_mul_d(ddv a, double b) {
  ddv p = two_prod(a.hi, b);
  p.lo = std::fma(a.lo, b, p.lo);
  return fast_two_sum(p.hi, p.lo);
}

// 1 / b to 2^-46 or better for a normal b: the hardware's approximation (some 23 bits) refined by a
// Newton step; 1 / sqrt(b) to about double rounding, by two.  The callers correct for the remainder,
// the quotient twice.
PIC_HD __forceinline__ double recip(double b) {
#ifdef __HIP_DEVICE_COMPILE__
  const double r = __builtin_amdgcn_rcp(b);
  return std::fma(std::fma(-b, r, 1.0), r, r);
#else
  return 1.0 / b;
#endif
}
PIC_HD __forceinline__ double recip_sqrt(double b) {
#ifdef __HIP_DEVICE_COMPILE__
  double r = __builtin_amdgcn_rsq(b);
  r = std::fma(0.5 * r, std::fma(-(b * r), r, 1.0), r);
  return std::fma(0.5 * r, std::fma(-(b * r), r, 1.0), r);
#else
  return 1.0 / std::sqrt(b);
#endif
}

// a / b: three partial quotients, each the current remainder times the double reciprocal of b.hi,
// so that the reciprocal's rounding does not matter.  The first is refined to within an ulp of
// a.hi / b.hi: its remainder a.hi - q1 b.hi is then a double, which the fma gives exactly.
PIC_HD __forceinline__ ddv dd_div(ddv a, ddv b) {
  const double rb = recip(b.hi);
  const double q0 = a.hi * rb;
  const double q1 = std::fma(std::fma(-q0, b.hi, a.hi), rb, q0);
  const ddv r = two_sum(std::fma(-q1, b.hi, a.hi), std::fma(-q1, b.lo, a.lo));
  const double q2 = r.hi * rb;
  const double r2 = std::fma(-q2, b.lo, std::fma(-q2, b.hi, r.hi) + r.lo);
  ddv q = fast_two_sum(q1, q2);
  q.lo = std::fma(r2, rb, q.lo);
  return q;
}

PIC_HD __forceinline__ ddv dd_sqrt(ddv a) {
  if (a.hi <= 0.0) return {0.0, 0.0};
  const double x = recip_sqrt(a.hi), hx = 0.5 * x;
  const double y0 = a.hi * x;
  const double y = std::fma(std::fma(-y0, y0, a.hi), hx, y0);
  // y is within an ulp of the root of a.hi, a.hi - y^2 a double
  return fast_two_sum(y, (std::fma(-y, y, a.hi) + a.lo) * hx);
}

// ln 2 and pi/2 as double pairs (hi = the double nearest the constant, lo = the remainder).
constexpr double kLn2Hi = 6.93147180559945286e-01;
constexpr double kLn2Lo = 2.31904681384629956e-17;
constexpr double kPi2Hi = 1.57079632679489656e+00;
constexpr double kPi2Lo = 6.12323399573676604e-17;

// 1/3 and 1/5 as double pairs
constexpr double kThirdHi = 0.3333333333333333;
constexpr double kThirdLo = 1.850371707708594e-17;
constexpr double kFifthHi = 0.2;
constexpr double kFifthLo = -1.1102230246251566e-17;

// t + SIGN t^3/3 + t^5/5 + SIGN t^7/7 + t^9/9: atanh t for SIGN = 1 (|t| <= 2^-12), atan t for
// -1 (|t| <= 2^-11).  The fourth and fifth terms, below 2^-68 t, are summed in double: their
// rounding is 2^-121 t.
template <int SIGN>
PIC_HD __forceinline__ ddv odd_series(ddv t) {
  const ddv t2 = dd_sqr(t);
  const double z = SIGN * t2.hi;
  ddv w = fast_two_sum(kFifthHi, z * std::fma(z, 1.0 / 9.0, 1.0 / 7.0));
  w.lo += kFifthLo;
  const ddv q = dd_mul_u(t2, w);
  ddv p = fast_two_sum(kThirdHi, SIGN * q.hi);
  p.lo += kThirdLo + SIGN * q.lo;
  const ddv u = dd_mul_u(t, dd_mul_u(t2, p));  // the second and later terms, below 2^-23 t
  return dd_add_f(t, SIGN > 0 ? u : dd_neg(u));
}

// natural log of a positive double-double.
PIC_HD inline ddv dd_log(ddv a) {
  int e;
  std::frexp(a.hi, &e);  // a.hi = f 2^e, f in [1/2, 1)
  e -= 1;
  const ddv m = {std::ldexp(a.hi, -e), std::ldexp(a.lo, -e)};  // exact; m.hi in [1, 2)
  const int k = (int)std::rint((m.hi - 1.0) * 1024.0);         // 0..1024
  const double c = 1.0 + (double)k * 0.0009765625;
  ddv den = two_sum(m.hi, c);
  den.lo += m.lo;
  // m.hi - c is exact; the quotient takes den unnormalised (its lo is below an ulp of hi)
  const ddv at = odd_series<1>(dd_div(two_sum(m.hi - c, m.lo), den));
  ddv el2 = two_prod((double)e, kLn2Hi);
  el2.lo = std::fma((double)e, kLn2Lo, el2.lo);
  // just below 1 (e = -1, c near 2) these cancel, and with c near 1 so may the last two
  const ddv base = dd_add_o(el2, ddv{kLogTab[k][0], kLogTab[k][1]});
  return dd_add_o(base, ddv{at.hi + at.hi, at.lo + at.lo});
}

// arctangent of p/q for double-doubles p >= 0, q > 0, without forming p/q: the ratio or its
// inverse, whichever is at most about 1, picks the table entry c = k/1024 from the leading
// parts, and atan(num/den) = atan c + atan(t) with t = (num - c den)/(den + c num) (the
// (x - c)/(1 + x c) of x = num/den), so one division serves both the ratio and the reduction.
// The identity holds for any c >= 0, so the entry is chosen with the unrefined reciprocal: that
// only widens |t| by a rounding error beyond 1/2048.
PIC_HD inline ddv dd_atan2(ddv p, ddv q) {
  const bool inv = p.hi > q.hi;
  const ddv num = inv ? q : p, den = inv ? p : q;
#ifdef __HIP_DEVICE_COMPILE__
  const double ratio = num.hi * __builtin_amdgcn_rcp(den.hi);
#else
  const double ratio = num.hi / den.hi;
#endif
  const int k = (int)std::rint(ratio * 1024.0);  // 0..1024
  const double c = (double)k * 0.0009765625;
  const ddv t = dd_div(dd_sub(num, dd_mul_d(den, c)), dd_add_f(den, dd_mul_d(num, c)));
  ddv r = dd_add_o(ddv{kAtanTab[k][0], kAtanTab[k][1]}, odd_series<-1>(t));
  if (inv) r = dd_add_o(ddv{kPi2Hi, kPi2Lo}, dd_neg(r));
  return r;
}

// arctangent of a non-negative double-double.
PIC_HD inline ddv dd_atan(ddv a) { return dd_atan2(a, dd_make(1.0)); }

}  // namespace pic
