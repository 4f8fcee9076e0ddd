// Host build of the FP64 SIN_SUM integrand on boxes [0, w] with w down to 1e-17
// and sum x = 0, where sin is as small as its phase: prints for N = 1 and N = 3 the
// largest error of a sample against long double, as a share of what the roundings
// of the phase s (2 + N of 2^-53 each, which move sin s by s cos s times that) and
// the sine polynomial (2.8e-16) may add up to; the count of phases
// whose reduction is not v = t or copysign(1/2, t) - t exactly, and the count of
// values outside [-1, 1] at phases up to 1e300.
#include <math.h>
#include <stdio.h>

#include <random>

#include "zmc_device.hpp"

template <int N>
double worst(double w, std::mt19937& rng) {
  zmc::ScanParams p{};
  for (int k = 0; k < N; ++k) p.hi[k] = w;
  zmc::SinSum<double, N> f;
  f.setup(p, 0);
  double e = 0;
  for (int i = 0; i < 4000; ++i) {
    double t[N];
    long double s = 0;
    for (int k = 0; k < N; ++k) {
      const uint32_t r = rng();
      t[k] = zmc::Unif<double>::t(r);
      s += (long double)w * ((long double)r + 0.5L) * 0x1p-32L;
    }
    const long double ref = sinl(s);
    const long double may = 2.8e-16L * fabsl(ref) + (2 + N) * 0x1p-53L * fabsl(s * cosl(s));
    const double d = (double)(fabsl((long double)f.value(t) - ref) / may);
    if (!(d <= e)) e = d;
  }
  return e;
}

int main() {
  std::mt19937 rng(3);
  double e1 = 0, e3 = 0;
  for (double w : {1.0, 1e-2, 1e-4, 1e-6, 1e-8, 1e-12, 1e-17}) {
    e1 = fmax(e1, worst<1>(w, rng));
    e3 = fmax(e3, worst<3>(w, rng));
  }
  long bad = 0, out = 0;
  for (int i = -200000; i <= 200000; ++i) {
    const double r = i * (3.7 / 200000.0) * (i % 3 ? 1.0 : 1e-9);
    const double t = r - rint(r);
    const double v = fabs(t) > 0.25 ? copysign(0.5, t) - t : t;
    bad += zmc::sin_turns(r) != zmc::sin_2pi_quarter(v);
  }
  for (int k = 0; k < 1000; ++k) {
    const double s = zmc::sin_turns(0.37 * pow(2.0, k));
    out += !(fabs(s) <= 1.0 + 4e-16);
  }
  printf("%.3e %.3e %ld %ld\n", e1, e3, bad, out);
  return 0;
}
