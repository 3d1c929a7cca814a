// Double-double arithmetic (value = hi + lo, |lo| <= ulp(hi)/2) for the fold.
//
// The unpivoted cluster elimination of Algorithm 1 forms Schur complements
// whose entries mix large (1/sigma_min of a nearly singular block) and O(1)
// parts; carrying the fold in double-double keeps the O(1) parts exact to
// FP64 level.  Built from the classic error-free transformations:
//   two_sum (Knuth): s + e == a + b exactly,
//   two_prod via fused multiply-add: p + e == a * b exactly.
// Every function body turns floating-point contraction off: hipcc contracts by
// default, and fusing the product a * b of two_prod into the sum that follows
// (s = p + e becomes fma(a, b, e)) counts the product's rounding error twice,
// leaving the result only about as accurate as plain FP64.
#pragma once

#include <hip/hip_runtime.h>

namespace hsc {

struct dd {
  double hi, lo;
};

struct zdd {   // complex double-double, 32 bytes
  dd re, im;
};

__device__ __forceinline__ dd two_sum(double a, double b) {
#pragma clang fp contract(off)
  const double s = a + b;
  const double bb = s - a;
  const double e = (a - (s - bb)) + (b - bb);
  return dd{s, e};
}

__device__ __forceinline__ dd quick_two_sum(double a, double b) {   // |a| >= |b|
#pragma clang fp contract(off)
  const double s = a + b;
  return dd{s, b - (s - a)};
}

__device__ __forceinline__ dd two_prod(double a, double b) {
#pragma clang fp contract(off)
  const double p = a * b;
  return dd{p, fma(a, b, -p)};
}

// sum with error bounded by ~2^-104 (|x| + |y|) (the "sloppy" double-double add):
// absolute accuracy relative to the operands, which is what the fold needs.
__device__ __forceinline__ dd dd_add(dd x, dd y) {
#pragma clang fp contract(off)
  dd s = two_sum(x.hi, y.hi);
  s.lo += x.lo + y.lo;
  return quick_two_sum(s.hi, s.lo);
}

__device__ __forceinline__ dd dd_neg(dd x) { return dd{-x.hi, -x.lo}; }
__device__ __forceinline__ dd dd_sub(dd x, dd y) { return dd_add(x, dd_neg(y)); }

__device__ __forceinline__ dd dd_mul(dd x, dd y) {
#pragma clang fp contract(off)
  dd p = two_prod(x.hi, y.hi);
  p.lo = fma(x.hi, y.lo, p.lo);
  p.lo = fma(x.lo, y.hi, p.lo);
  return quick_two_sum(p.hi, p.lo);
}

__device__ __forceinline__ dd dd_from(double a) { return dd{a, 0.0}; }

__device__ __forceinline__ zdd zdd_from(double2 v) { return zdd{dd{v.x, 0.0}, dd{v.y, 0.0}}; }
__device__ __forceinline__ double2 zdd_round(zdd v) { return make_double2(v.re.hi + v.re.lo, v.im.hi + v.im.lo); }
__device__ __forceinline__ zdd zdd_zero() { return zdd{dd{0.0, 0.0}, dd{0.0, 0.0}}; }
__device__ __forceinline__ zdd zdd_add(zdd a, zdd b) { return zdd{dd_add(a.re, b.re), dd_add(a.im, b.im)}; }
__device__ __forceinline__ zdd zdd_sub(zdd a, zdd b) { return zdd{dd_sub(a.re, b.re), dd_sub(a.im, b.im)}; }
__device__ __forceinline__ zdd zdd_neg(zdd a) { return zdd{dd_neg(a.re), dd_neg(a.im)}; }

__device__ __forceinline__ zdd zdd_mul(zdd a, zdd b) {
  return zdd{dd_sub(dd_mul(a.re, b.re), dd_mul(a.im, b.im)), dd_add(dd_mul(a.re, b.im), dd_mul(a.im, b.re))};
}

// acc + a * b
__device__ __forceinline__ zdd zdd_fma(zdd acc, zdd a, zdd b) { return zdd_add(acc, zdd_mul(a, b)); }

// 1 / a = conj(a) / |a|^2, scaled by the power of two of the larger component (0 for a = 0).  |a|^2 as d.hi + d.lo + f
// with the roundings of its low part in f, each component as an FP64 quotient and its residual, so that little but
// the result's own rounding remains; the FP64 reciprocal y of d.hi is on its way meanwhile.  Error in units of 2^-106 of
// |1 / a|, mean and worst: 0.43 and 3.4 (0.68 and 5.3 with one Newton step of |a|^-2, 0.48 and 3.5 with three FP64
// quotients a component); an inverse of order 64 to 512 takes 2 to 4 % longer than with the Newton step.
__device__ __forceinline__ zdd zdd_rcp(zdd a) {
#pragma clang fp contract(off)
  const double s = fmax(fabs(a.re.hi), fabs(a.im.hi));
  if (s == 0.0) return zdd_zero();
  const int k = -ilogb(s);
  const dd x{ldexp(a.re.hi, k), ldexp(a.re.lo, k)}, z{ldexp(a.im.hi, k), ldexp(a.im.lo, k)};
  const dd p = two_prod(x.hi, x.hi), q = two_prod(z.hi, z.hi), d = two_sum(p.hi, q.hi);   // in [1, 8)
  double y = __builtin_amdgcn_rcp(d.hi);
  y = fma(y, fma(-d.hi, y, 1.0), y);
  y = fma(y, fma(-d.hi, y, 1.0), y);
  const dd c = two_sum(p.lo, fma(2.0 * x.hi, x.lo, q.lo)), g = two_sum(d.lo, 2.0 * z.hi * z.lo), l = two_sum(c.hi, g.hi);
  const double f = l.lo + (c.lo + g.lo + fma(x.lo, x.lo, z.lo * z.lo)), e = fma(-l.hi, y, fma(-d.hi, y, 1.0));
  auto over = [&](dd v) {
    const double h = v.hi * y;
    const dd r = two_sum(fma(-h, d.hi, v.hi), fma(-h, l.hi, v.lo));
    const double w = r.hi * y;
    const dd t = quick_two_sum(h, w + (fma(r.hi, y, -w) + fma(w, e, fma(-h, f, r.lo) * y)));
    return dd{ldexp(t.hi, k), ldexp(t.lo, k)};
  };
  return zdd{over(x), over(dd_neg(z))};
}

// Pointers loaded from a descriptor are generic to the compiler; as global ones they give global loads and
// stores instead of flat ones (which also wait for LDS).
typedef double v2d __attribute__((ext_vector_type(2)));
template <class T> using global_ptr = __attribute__((address_space(1))) T*;

__device__ __forceinline__ zdd load_zdd(const zdd* q) {
  const global_ptr<const v2d> p = (global_ptr<const v2d>)q;
  const v2d re = p[0], im = p[1];
  return zdd{dd{re.x, re.y}, dd{im.x, im.y}};
}
__device__ __forceinline__ void store_zdd(zdd* q, zdd v) {
  const global_ptr<v2d> p = (global_ptr<v2d>)q;
  p[0] = v2d{v.re.hi, v.re.lo};
  p[1] = v2d{v.im.hi, v.im.lo};
}

// Lazy accumulation of a sum of double-double products (the GEMM inner loop): hi
// holds the running FP64 sum, lo collects the exact rounding errors of the hi
// additions (two_sum) and the products' low parts in plain FP64.  renorm() folds
// lo back into hi; called every few terms it keeps the result double-double
// accurate while each product-accumulate costs 12 FP64 operations instead of 18.
struct ddacc {
  double hi, lo;
};

struct zddacc {
  ddacc re, im;
};

__device__ __forceinline__ void ddacc_add_prod(ddacc& a, dd x, dd y) {
#pragma clang fp contract(off)
  const double ph = x.hi * y.hi;
  double pl = fma(x.hi, y.hi, -ph);
  pl = fma(x.hi, y.lo, pl);
  pl = fma(x.lo, y.hi, pl);
  const double s = a.hi + ph;
  const double bb = s - a.hi;
  const double e = (a.hi - (s - bb)) + (ph - bb);
  a.hi = s;
  a.lo += e + pl;
}

__device__ __forceinline__ void ddacc_renorm(ddacc& a) {
  const dd s = two_sum(a.hi, a.lo);
  a.hi = s.hi;
  a.lo = s.lo;
}

// c += a * b
__device__ __forceinline__ void zddacc_fma(zddacc& c, zdd a, zdd b) {
  ddacc_add_prod(c.re, a.re, b.re);
  ddacc_add_prod(c.re, dd_neg(a.im), b.im);
  ddacc_add_prod(c.im, a.re, b.im);
  ddacc_add_prod(c.im, a.im, b.re);
}

__device__ __forceinline__ void zddacc_renorm(zddacc& c) {
  ddacc_renorm(c.re);
  ddacc_renorm(c.im);
}

__device__ __forceinline__ zddacc zddacc_from(zdd v) { return zddacc{{v.re.hi, v.re.lo}, {v.im.hi, v.im.lo}}; }
__device__ __forceinline__ zdd zddacc_value(zddacc c) { return zdd{two_sum(c.re.hi, c.re.lo), two_sum(c.im.hi, c.im.lo)}; }

__device__ __forceinline__ double zdd_cabs1(zdd a) { return fabs(a.re.hi) + fabs(a.im.hi); }

}  // namespace hsc
