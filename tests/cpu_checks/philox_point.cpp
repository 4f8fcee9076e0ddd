// Host build of the sample-major Philox blocks (the point's part shared, the
// word block per lane; batches of 1, 2 and 3); prints the blocks that differ
// from the generic path over a seeded set of (seed, g, b), edges included.
#include <cstdint>
#include <cstdio>
#include <random>

#include "zmc_device.hpp"

template <int NB> long check(uint64_t seed, uint32_t g, uint32_t b) {
  zmc::Words4 w[NB];
  zmc::philox_blocks_sm<NB>(b, zmc::philox_point(g, seed), w);
  long bad = 0;
  for (int i = 0; i < NB; ++i) {
    const zmc::Words4 a = zmc::philox_block((uint64_t)b + i, g, seed);
    for (int k = 0; k < 4; ++k) bad += a.r[k] != w[i].r[k];
  }
  return bad;
}

int main() {
  std::mt19937_64 rng(4242);
  long bad = 0, total = 0;
  for (int i = 0; i < 60000; ++i) {
    const uint64_t seed = rng();
    uint32_t g = (uint32_t)rng(), b = (uint32_t)rng();
    if (i % 5 == 0) g = i % 2 ? 0u : 0xFFFFFFFFu;
    if (i % 7 == 0) b = i % 2 ? 0u : 0xFFFFFFFFu - 2u;
    if (b > 0xFFFFFFFFu - 2u) b = 0xFFFFFFFFu - 2u;
    bad += check<1>(seed, g, b) + check<2>(seed, g, b) + check<3>(seed, g, b);
    ++total;
  }
  std::printf("%ld %ld\n", bad, total);
  return bad != 0;
}
