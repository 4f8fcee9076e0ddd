// Host build of the kernels' grid decoding: every axis index of a set of grid
// points against 64-bit division, on grids up to 2^32 points with lengths and
// indices at the edges (exact multiples of the strides, one less, one more) and
// beyond 2^32 (the 64-bit path).  Prints the number of wrong indices.
#include <cstdint>
#include <cstdio>
#include <random>

#include "zmc_device.hpp"

int main() {
  std::mt19937_64 rng(99);
  long bad = 0, total = 0;
  for (int it = 0; it < 4000; ++it) {
    zmc::ScanParams p{};
    p.M = 1 + (int)(rng() % 16);
    uint64_t G = 1;
    const uint64_t cap = it % 10 == 0 ? (uint64_t)1 << 45 : (uint64_t)1 << 32;
    for (int l = 0; l < p.M; ++l) {
      uint64_t L = it % 7 == 0 && l == 0 ? cap / 3 : 1 + rng() % (it % 3 ? 7 : 4000);
      if (G * L > cap) L = 1;
      p.axis_len[l] = (int64_t)L;
      G *= L;
    }
    uint64_t stride = 1;
    for (int l = p.M - 1; l >= 0; --l) {
      p.axis_stride[l] = stride;
      p.axis_inv[l] = 1.0 / (double)stride;
      stride *= (uint64_t)p.axis_len[l];
    }
    p.small_index = G <= ((uint64_t)1 << 32);
    for (int k = 0; k < 200; ++k) {
      uint64_t g = rng() % G;
      if (k % 2) {
        const uint64_t s = p.axis_stride[rng() % (uint64_t)p.M];
        g = g / s * s + (k % 3) - 1;
      }
      if (k < 2) g = k ? G - 1 : 0;
      if (g >= G) g = G - 1;
      zmc::ParamCursor c(p, g);
      for (int l = 0; l < p.M; ++l) {
        bad += c.index(l) != (g / p.axis_stride[l]) % (uint64_t)p.axis_len[l];
        ++total;
      }
    }
  }
  std::printf("%ld %ld\n", bad, total);
  return bad != 0;
}
