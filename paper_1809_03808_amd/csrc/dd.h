// Double-double arithmetic on the device (about 106 significant bits: Knuth's
// two-sum and the exact product of a fused multiply-add), real and complex.
//
// The error-free transformations need every product rounded on its own: a
// product contracted into the following addition (a fused multiply-add) leaves
// the error term computed from a different rounding, which loses the low half
// of every double-double value.
#pragma once

#include <hip/hip_runtime.h>

namespace helm {

struct dd {
  double hi, lo;
};
__device__ inline dd two_sum(double a, double b) {
  const double s = a + b, bb = s - a;
  return {s, (a - (s - bb)) + (b - bb)};
}
__device__ inline dd fast_two_sum(double a, double b) {  // |a| >= |b|
  const double s = a + b;
  return {s, b - (s - a)};
}
__device__ inline dd dd_of(double a) { return {a, 0.0}; }
__device__ inline dd dd_neg(dd x) { return {-x.hi, -x.lo}; }
__device__ inline dd dd_add(dd x, dd y) {
  dd s = two_sum(x.hi, y.hi);
  const dd t = two_sum(x.lo, y.lo);
  s = fast_two_sum(s.hi, s.lo + t.hi);
  return fast_two_sum(s.hi, s.lo + t.lo);
}
__device__ inline dd dd_sub(dd x, dd y) { return dd_add(x, dd_neg(y)); }
__device__ inline dd dd_mul(dd x, dd y) {
#pragma clang fp contract(off)
  const double p = x.hi * y.hi;
  double e = fma(x.hi, y.hi, -p);
  e = fma(x.hi, y.lo, e);
  e = fma(x.lo, y.hi, e);
  return fast_two_sum(p, e);
}
__device__ inline dd dd_mul_d(dd x, double y) {
#pragma clang fp contract(off)
  const double p = x.hi * y;
  double e = fma(x.hi, y, -p);
  e = fma(x.lo, y, e);
  return fast_two_sum(p, e);
}
// x / y: three quotient digits, each from the remainder of the previous ones
__device__ inline dd dd_div(dd x, dd y) {
  const double q1 = x.hi / y.hi;
  dd r = dd_sub(x, dd_mul_d(y, q1));
  const double q2 = r.hi / y.hi;
  r = dd_sub(r, dd_mul_d(y, q2));
  const double q3 = r.hi / y.hi;
  return dd_add(fast_two_sum(q1, q2), dd_of(q3));
}

struct cdd {
  dd re, im;
};
__device__ inline cdd cdd_of(double2 a) { return {dd_of(a.x), dd_of(a.y)}; }
__device__ inline cdd cdd_zero() { return {dd_of(0.0), dd_of(0.0)}; }
__device__ inline cdd cdd_add(cdd a, cdd b) { return {dd_add(a.re, b.re), dd_add(a.im, b.im)}; }
__device__ inline cdd cdd_sub(cdd a, cdd b) { return {dd_sub(a.re, b.re), dd_sub(a.im, b.im)}; }
__device__ inline cdd cdd_neg(cdd a) { return {dd_neg(a.re), dd_neg(a.im)}; }
__device__ inline cdd cdd_mul(cdd a, cdd b) {
  return {dd_sub(dd_mul(a.re, b.re), dd_mul(a.im, b.im)), dd_add(dd_mul(a.re, b.im), dd_mul(a.im, b.re))};
}
__device__ inline cdd cdd_scale(cdd a, dd s) { return {dd_mul(a.re, s), dd_mul(a.im, s)}; }
__device__ inline cdd cdd_scale_d(cdd a, double s) { return {dd_mul_d(a.re, s), dd_mul_d(a.im, s)}; }
__device__ inline cdd cdd_div(cdd a, cdd b) {
  const dd den = dd_add(dd_mul(b.re, b.re), dd_mul(b.im, b.im));
  const dd nr = dd_add(dd_mul(a.re, b.re), dd_mul(a.im, b.im));
  const dd ni = dd_sub(dd_mul(a.im, b.re), dd_mul(a.re, b.im));
  return {dd_div(nr, den), dd_div(ni, den)};
}
__device__ inline double cdd_abs2_hi(cdd a) { return a.re.hi * a.re.hi + a.im.hi * a.im.hi; }
__device__ inline bool cdd_is_zero(cdd a) { return a.re.hi == 0.0 && a.im.hi == 0.0; }
__device__ inline double4 pack(cdd a) { return make_double4(a.re.hi, a.re.lo, a.im.hi, a.im.lo); }
__device__ inline cdd unpack(double4 v) { return {{v.x, v.y}, {v.z, v.w}}; }

}  // namespace helm
