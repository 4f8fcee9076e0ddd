// Host build of the table-driven FP64 2^t and e^-q, the reduction of a phase
// to a fraction of a revolution, and the quarter-turn form of the sine,
// against long double libm: prints the largest relative error of each of the
// first two, the largest error of the other two, and the count of wrong edges.
#include <math.h>
#include <stdio.h>

#include "zmc_device.hpp"

int main() {
  double worst_e = 0, worst_q = 0, worst_t = 0, worst_s = 0;
  const long double pi = 3.14159265358979323846264338327950288L;
  for (int i = -400000; i <= 400000; ++i) {
    const double t = i * (64.0 / 400000.0) + i * 1e-9;
    const long double ref = exp2l((long double)t);
    const double e = (double)fabsl(((long double)zmc::exp2_fp64(t) - ref) / ref);
    if (e > worst_e) worst_e = e;
    const double q = t < 0 ? -t : t;
    const long double rq = expl(-(long double)q);
    // q log2 e is formed with one rounding of log2 e: an error of q 2^-53
    const double eq = (double)(fabsl(((long double)zmc::exp_minus_fp64<true>(q) - rq) / rq) / (1 + q));
    if (eq > worst_q) worst_q = eq;
    const double x = i * 0.0025;  // radians, up to 1000
    const long double r = (long double)x / (2 * pi);
    const double f = zmc::turns_fraction(x);
    const long double d = r - (long double)f;
    const double et = (double)fabsl(d - rintl(d));
    if (et > worst_t) worst_t = et;
    const double es = (double)fabsl((long double)zmc::cos_turns(f - 0.25) - sinl((long double)x));
    if (es > worst_s) worst_s = es;
  }
  int bad = 0;
  bad += !(zmc::exp_minus_fp64<true>(INFINITY) == 0.0 && zmc::exp_minus_fp64<true>(1e300) == 0.0);
  bad += !(zmc::exp_minus_fp64<false>(-INFINITY) == INFINITY && zmc::exp_minus_fp64<false>(-1e300) == INFINITY);
  bad += !(zmc::exp_minus_fp64<true>(0.0) == 1.0 && zmc::exp_minus_fp64<true>(NAN) == 0.0);
  for (int j = 0; j < 256; ++j)  // the table's own points
    bad += !(fabsl(zmc::exp2_fp64(j / 256.0) - exp2l(j / 256.0L)) <= 1.2e-16L * exp2l(j / 256.0L));
  for (int k = -1074; k < 1024; ++k) bad += !(zmc::exp2_fp64(k) == ldexp(1.0, k));
  printf("%.3e %.3e %.3e %.3e %d\n", worst_e, worst_q, worst_t, worst_s, bad);
  return 0;
}
