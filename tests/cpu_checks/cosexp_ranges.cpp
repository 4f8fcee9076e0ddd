// Host build of the FP64 COSEXP integrand against long double: prints the largest
// error of a sample whose cosine and offset are 1 and 0 (x1 = x2 = x4 = 0), as a
// share of the roundings of the exponent E (four of 2^-53, which move 2^E by E times
// that) and of 2^t (1.2e-16), over boxes where y1 y2 >= 0 and x3 up to 1000; the
// largest error of a sample's cosine (x3 = x4 = 0) as a share of the roundings of its
// phase; and the count of wrong values where x3^2 is huge or overflows.
#include <math.h>
#include <stdio.h>

#include <random>

#include "zmc_device.hpp"

struct Point {
  zmc::ScanParams p{};
  double x[4];
  Point(double lo, double hi, double x1, double x2, double x3, double x4, int N) : x{x1, x2, x3, x4} {
    p.M = 4;
    p.small_index = 1;
    for (int l = 0; l < 4; ++l) p.axis_len[l] = 1, p.axis_off[l] = l, p.axis_stride[l] = 1, p.axis_inv[l] = 1.0;
    for (int k = 0; k < N; ++k) p.lo[k] = lo, p.hi[k] = hi;
    p.axis = x;
  }
};

constexpr long double kPiL = 3.14159265358979323846264338327950288L;

int main() {
  std::mt19937 rng(8);
  double worst_e = 0, worst_c = 0;
  const double boxes[][2] = {{0, 1}, {-1, 0}, {-3, -0.5}, {0.5, 3}};
  for (const auto& bx : boxes)
    for (double x3 : {0.5, 3.0, 30.0, 1000.0}) {
      Point pt(bx[0], bx[1], 0, 0, x3, 0, 2);
      zmc::CosExp<double, 2> f;
      f.setup(pt.p, 0);
      for (int i = 0; i < 20000; ++i) {
        double t[2];
        long double y[2];
        for (int k = 0; k < 2; ++k) {
          const uint32_t r = rng() >> (i % 24);  // small words too
          t[k] = zmc::Unif<double>::t(k && i % 2 ? r : ~r);
          const uint32_t w = k && i % 2 ? r : ~r;
          y[k] = bx[0] + ((long double)bx[1] - bx[0]) * ((long double)w + 0.5L) * 0x1p-32L;
        }
        const long double q = (long double)x3 * x3 * y[0] * y[1], ref = expl(-q);
        if (ref < 1e-30L) continue;
        // y1 and y2 carry the rounding of their box offset besides their own
        long double dy = 0;
        for (int k = 0; k < 2; ++k) dy += 0x1p-53L * (1 + fabsl(bx[0] / y[k]) * (bx[0] == -1 || bx[0] == 0 ? 0 : 1));
        const long double may = ref * (1.2e-16L + q * (4 * 0x1p-53L + dy));
        const double d = (double)(fabsl((long double)f.value(t) - ref) / may);
        if (!(d <= worst_e)) worst_e = d;
      }
    }
  for (const auto& bx : {boxes[0], boxes[1]})
    for (double X : {1.0, 30.0, 1000.0}) {
      Point pt(bx[0], bx[1], X, 0.7 * X, 0, 0, 3);
      zmc::CosExp<double, 3> f;
      f.setup(pt.p, 0);
      for (int i = 0; i < 20000; ++i) {
        double t[3];
        long double y[3];
        for (int k = 0; k < 3; ++k) {
          const uint32_t r = rng();
          t[k] = zmc::Unif<double>::t(r);
          y[k] = bx[0] + ((long double)bx[1] - bx[0]) * ((long double)r + 0.5L) * 0x1p-32L;
        }
        const long double a = pt.x[0] * y[0], b = pt.x[1] * y[1], ph = a + b + y[2];
        const long double red = ph - 2 * kPiL * rintl(ph / (2 * kPiL));
        // per term: 1/(2 pi), its product with x, y's own rounding, the product and
        // the sums; y3's map rounds A and B
        const long double may = 2.8e-16L + 2 * kPiL * 0x1p-54L +
                                0x1p-53L * (4 * fabsl(a) + 4 * fabsl(b) + 3 + fabsl(a + b) + fabsl(ph)) + 1e-18L * X;
        const double d = (double)(fabsl((long double)f.value(t) - cosl(red)) / may);
        if (!(d <= worst_c)) worst_c = d;
      }
    }
  int bad = 0;
  for (double x3 : {1e152, 1e153, 1.3e154, 1e155}) {
    Point pt(-1, 1, 0, 0, x3, 0, 2);
    zmc::CosExp<double, 2> f;
    f.setup(pt.p, 0);
    const double quarter = 0x1p30, upper = 0x1.8p31;  // y = -1/2 and +1/2
    const double grow[2] = {quarter, upper}, fall[2] = {upper, upper};
    bad += !(f.value(grow) == INFINITY) + !(f.value(fall) == 0.0);
  }
  printf("%.3e %.3e %d\n", worst_e, worst_c, bad);
  return 0;
}
