// Reciprocals of complex double-double numbers, read as four hexadecimal doubles a line: csrc/dd.h's, then the
// same by three FP64 quotients per component of operands scaled by the larger one.
#include <cstdio>

#include "../../paper_1702_05167_amd/csrc/dd.h"

using namespace hsc;

static dd quotient(dd x, dd y) {
  const double q1 = x.hi / y.hi;
  dd r = dd_sub(x, dd_mul(dd_from(q1), y));
  const double q2 = r.hi / y.hi;
  r = dd_sub(r, dd_mul(dd_from(q2), y));
  const double q3 = r.hi / y.hi;
  return dd_add(quick_two_sum(q1, q2), dd_from(q3));
}

static zdd by_quotients(zdd a) {
  const dd s = dd_from(1.0 / fmax(fabs(a.re.hi), fabs(a.im.hi)));
  const dd re = dd_mul(a.re, s), im = dd_mul(a.im, s);
  const dd den = dd_add(dd_mul(re, re), dd_mul(im, im));
  return zdd{dd_mul(quotient(re, den), s), dd_mul(quotient(dd_neg(im), den), s)};
}

int main() {
  double v[4];
  while (std::scanf("%la %la %la %la", v, v + 1, v + 2, v + 3) == 4) {
    const zdd a{{v[0], v[1]}, {v[2], v[3]}}, x = zdd_rcp(a), y = by_quotients(a);
    std::printf("%a %a %a %a %a %a %a %a\n", x.re.hi, x.re.lo, x.im.hi, x.im.lo, y.re.hi, y.re.lo, y.im.hi, y.im.lo);
  }
  return 0;
}
