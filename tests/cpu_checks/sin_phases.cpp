// Host build of the FP64 SIN_SUM integrand on boxes up to 10 wide and sums up to 1000:
// prints the largest error of a sample against long double, as a share of the
// roundings of the phase's sum and reduction and of the sine polynomial; the largest
// ratio of the integrand's mean square error to that of the same sum whose product
// with 1/(2 pi) is rounded before its reduction; and, for phases from 2^40 to 1e300,
// the count of values outside [-1, 1] and of boxes whose mean square is not near 1/2.
#include <math.h>
#include <stdio.h>

#include <random>

#include "zmc_device.hpp"

constexpr long double kPiL = 3.14159265358979323846264338327950288L;
constexpr long double kTwoPiLo = -1.00331152253366640475e-19L;  // 2 pi - (long double)2 pi

template <int N>
void point(double lo, double hi, double x, std::mt19937& rng, double* worst, double* ratio) {
  zmc::ScanParams p{};
  p.M = 1;
  p.small_index = 1;
  p.axis_len[0] = 1, p.axis_stride[0] = 1, p.axis_inv[0] = 1.0;
  p.axis = &x;
  for (int k = 0; k < N; ++k) p.lo[k] = lo, p.hi[k] = hi;
  zmc::fold_sin_box(N, p.lo, p.hi);
  zmc::SinSum<double, N> f;
  f.setup(p, 0);
  long double sq = 0, sq_rounded = 0;
  for (int i = 0; i < 20000; ++i) {
    double t[N], sy = 0;
    long double s = x, sum = 0;
    for (int k = 0; k < N; ++k) {
      const uint32_t r = rng();
      t[k] = zmc::Unif<double>::t(r);
      s += lo + ((long double)hi - lo) * ((long double)r + 0.5L) * 0x1p-32L;
      const double y = __builtin_fma(f.A[k], t[k], f.B[k]);
      sy = k ? sy + y : y;
      sum += fabsl(sy) + fabsl(y);
    }
    const long double n = rintl(s / (2 * kPiL));
    const long double e = sinl((s - n * (2 * kPiL)) - n * kTwoPiLo);
    const long double d = f.value(t) - e;
    const double r = (x + sy) * zmc::kInv2Pi, fr = r - rint(r);
    const long double dr = zmc::sin_2pi_quarter(fabs(fr) > 0.25 ? copysign(0.5, fr) - fr : fr) - e;
    sq += d * d;
    sq_rounded += dr * dr;
    // B, y and the partial sums; x + sum; the reduced phase and 1/(2 pi)
    const long double may = 2.8e-16L + 0x1p-53L * (sum + N * fabs(lo) + fabsl(s) + kPiL + 0.57L * fabsl(s));
    const double share = (double)(fabsl(d) / may);
    if (!(share <= *worst)) *worst = share;
  }
  const double q = (double)sqrtl(sq / sq_rounded);
  if (!(q <= *ratio)) *ratio = q;
}

int main() {
  std::mt19937 rng(4);
  double worst = 0, ratio = 0;
  for (double x : {0.3, 7.7, 51.0, 1000.0})
    for (double w : {1.0, 10.0}) {
      point<1>(0, w, x, rng, &worst, &ratio);
      point<2>(-w, 0.5 * w, x, rng, &worst, &ratio);
      point<4>(0, w, x, rng, &worst, &ratio);
      point<12>(0, w, x, rng, &worst, &ratio);
    }
  long out = 0, flat = 0;
  for (double w = 0x1p40; w < 1e300; w *= 37.0) {
    zmc::ScanParams p{};
    p.hi[0] = p.hi[1] = w;
    const double x = w > 1e100 ? w : 0.0;  // both, the box alone, the sum alone
    if (w > 1e200) p.hi[0] = p.hi[1] = 1.0;
    p.M = 1;
    p.small_index = 1;
    p.axis_len[0] = 1, p.axis_stride[0] = 1, p.axis_inv[0] = 1.0;
    p.axis = &x;
    zmc::fold_sin_box(2, p.lo, p.hi);
    zmc::SinSum<double, 2> f;
    f.setup(p, 0);
    double sq = 0;
    for (int i = 0; i < 4000; ++i) {
      const double t[2] = {zmc::Unif<double>::t(rng()), zmc::Unif<double>::t(rng())};
      const double v = f.value(t);
      out += !(fabs(v) <= 1.0 + 4e-16);
      sq += v * v;
    }
    flat += w < 0x1p80 && !(fabs(sq / 4000 - 0.5) < 0.04);
  }
  printf("%.3e %.3f %ld %ld\n", worst, ratio, out, flat);
  return 0;
}
