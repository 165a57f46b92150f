// Double-double arithmetic (Dekker 1971; Knuth, TAOCP vol. 2, 4.2.2).
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define EPRL_DD __host__ __device__ __forceinline__
#else  // (the host compiler, for tests)
#define EPRL_DD inline
#endif

// The error-free transformations below need every product and sum rounded exactly as
// written: fusing p = a*b into a later p + e (the default contraction of device code) would
// destroy the error terms.
#ifdef __clang__
#pragma clang fp contract(off)
#endif

namespace eprl {

struct dd {
  double hi, lo;
};

EPRL_DD dd two_sum(double a, double b) {
  double s = a + b;
  double bb = s - a;
  double e = (a - (s - bb)) + (b - bb);
  return {s, e};
}

EPRL_DD dd fast_two_sum(double a, double b) {
  double s = a + b;
  return {s, b - (s - a)};
}

EPRL_DD dd dd_add(dd a, dd b) {
  dd s = two_sum(a.hi, b.hi);
  dd t = two_sum(a.lo, b.lo);
  s.lo += t.hi;
  s = fast_two_sum(s.hi, s.lo);
  s.lo += t.lo;
  return fast_two_sum(s.hi, s.lo);
}

EPRL_DD dd dd_mul(dd a, dd b) {
  double p = a.hi * b.hi;
  double e = __builtin_fma(a.hi, b.hi, -p);
  e += a.hi * b.lo + a.lo * b.hi;
  return fast_two_sum(p, e);
}

// Quotient of two integers below 2^50 as a double-double, both words rounded to nearest but for about
// 2^-50 of an ulp (2^-106 of the quotient in all, as with two divisions).  One division: each word is a
// product with the reciprocal, corrected by its remainder, which is exact (a multiple of the product's
// last place, of fewer than 53 bits).
EPRL_DD dd dd_ratio(double num, double den) {
  const double inv = 1.0 / den;
  double q = num * inv;
  q = __builtin_fma(__builtin_fma(-q, den, num), inv, q);
  const double r = __builtin_fma(-q, den, num);
  double lo = r * inv;
  lo = __builtin_fma(__builtin_fma(-lo, den, r), inv, lo);
  return fast_two_sum(q, lo);
}

// sqrt(q) of a small integer q as a double-double.
EPRL_DD dd dd_sqrt_int(double q) {
  double s = __builtin_sqrt(q);
  double r = __builtin_fma(-s, s, q);
  return fast_two_sum(s, r / (2.0 * s));
}

}  // namespace eprl
