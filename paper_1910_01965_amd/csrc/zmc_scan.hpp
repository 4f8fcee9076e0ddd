// zmc_scan.hpp -- the scan loops on gfx950, device code only (no host
// dependencies), so that both the compiled-in kernels and the kernels built at
// run time for user integrands use them.
//
// Point-major: a lane owns one grid point and all lanes of a wave walk the
// same groups of four samples in step, so the Philox counter words that
// depend only on the sample index (the word block b) are wave-uniform and
// live in scalar registers; only the grid-index half of the counter differs
// between lanes.  A point's sample range may be cut into `splits` pieces run
// by different blocks; their FP64 partials are merged by a second pass.
//
// Sample-major: a block owns one grid point and its lanes share the samples
// (lane t takes groups t, t+T, ...); lane sums are merged over the wave by DPP,
// then over the block's waves through LDS, then (for several blocks per point)
// by the same second pass.
//
// Method: direct Monte Carlo per grid point, ZMCintegral-v5 Sec. 2, Eq. (1);
// the paper gives each point to one GPU thread (Sec. 2, Fig. 1), which is the
// point-major layout without splits.
#pragma once

#include "zmc_device.hpp"

namespace zmc {

// Groups j0 .. jfull-1 in full, then (when `ragged`) the scan's short last
// group; every lane of the wave walks the same j.
// The lane's sums are shifted by its first sample, so that the final
// M2 = S2 - S1^2 / n does not cancel even when the samples are close to each
// other and far from the integrand's typical value.
template <class Fam, typename T, int N, class Gen>
__device__ __forceinline__ void lane_groups(const Fam& fam, const Gen& gen, uint64_t j0,
                                            uint64_t jfull, bool ragged, int tail,
                                            LaneAcc<T>& acc) {
  uint64_t j = j0;
  if (j < jfull) {
    T v[4];
    eval_group<Fam, T, N>(fam, j, gen, v);
    acc.init(v[0]);
    acc.add4(v);
    ++j;
  }
  // j <= jfull here; the inequality test keeps the (wave-uniform) loop
  // control on the scalar unit, which has no unsigned 64-bit "less than"
  for (; j != jfull; ++j) {
    T v[4];
    eval_group<Fam, T, N>(fam, j, gen, v);
    acc.add4(v);
  }
  if (ragged) {
    T v[4];
    eval_group<Fam, T, N>(fam, jfull, gen, v);
    if (jfull == j0) acc.init(v[0]);
    acc.add_partial(v, tail);
  }
}

// One point-major tile: the block's lanes take grid points first,
// first + 1, ... (one each) over sample piece sp.
template <class Fam, typename T, int N>
__device__ __forceinline__ void pm_tile(const ScanParams& p, uint64_t first, uint64_t sp) {
  const uint64_t j0 = sp * p.gps;
  const uint64_t j1 = (j0 + p.gps < p.n_groups) ? j0 + p.gps : p.n_groups;
  const bool ragged = (j1 == p.n_groups) && ((p.n & 3u) != 0);
  const uint64_t jfull = ragged ? j1 - 1 : j1;
  const int tail = (int)(p.n - 4 * (p.n_groups - 1));
  const uint64_t g = first + threadIdx.x;  // local index: outputs
  if (g >= p.G) return;
  const uint64_t gg = p.g_base + g;        // global index: parameters and stream
  Fam fam;
  fam.setup(p, gg);
  LaneAcc<T> acc;
  acc.init((T)0);
  with_form(fam, [&](const auto& f) {
    using F = std::decay_t<decltype(f)>;
    if (p.fast_counter) {
      using Gen = std::conditional_t<Phased<F>::value, GenPointMajorPhased, GenPointMajor>;
      const Gen gen = Gen::make((uint32_t)gg, p.seed);
      lane_groups<F, T, N>(f, gen, j0, jfull, ragged, tail, acc);
    } else {
      const GenAny gen{gg, p.seed};
      lane_groups<F, T, N>(f, gen, j0, jfull, ragged, tail, acc);
    }
  });
  const Moments m = to_moments(acc, (double)split_samples(p.n, p.n_groups, p.gps, sp));
  if (p.splits == 1) {
    finalize(p, g, m);
  } else {
    p.part_mean[sp * p.G + g] = m.mean;
    p.part_m2[sp * p.G + g] = m.m2;
  }
}

// The lane's groups j, j + step, ... of a piece whose rows of `step` groups
// (one per lane) number `rows`: every row but the last is full, and only the
// last can hold the scan's short last group (`tail` samples) or stop before the
// lane (`in_last` false).  The lane's sums are shifted by its first sample.
// Returns the lane's sample count.
template <class Fam, typename T, int N, class Gen>
__device__ __forceinline__ double strided_groups(const Fam& fam, const Gen& gen, uint64_t j,
                                                 uint64_t step, uint64_t rows, bool in_last,
                                                 uint64_t last, int tail, LaneAcc<T>& acc) {
  if (rows > 1) {
    T v[4];
    eval_group<Fam, T, N>(fam, j, gen, v);
    acc.init(v[0]);
    acc.add4(v);
    j += step;
    for (uint64_t i = 2; i != rows; ++i) {
      T u[4];
      eval_group<Fam, T, N>(fam, j, gen, u);
      acc.add4(u);
      j += step;
    }
  }
  double count = 4.0 * (double)(rows - 1);
  if (in_last) {
    T v[4];
    eval_group<Fam, T, N>(fam, j, gen, v);
    if (rows == 1) acc.init(v[0]);
    if (j == last && tail != 4) {
      acc.add_partial(v, tail);
      count += (double)tail;
    } else {
      acc.add4(v);
      count += 4.0;
    }
  }
  return count;
}

// Sample-major work on grid point g (local index; its global index is p.g_base +
// g) over sample piece sp by the `waves` waves of the block from wave w0 on: lane
// t of them takes groups j0 + t, j0 + t + T, ... (T: the lanes of the whole block;
// fewer waves than the block's are used for pieces of at most as many groups as
// they have lanes).  Then the lanes are merged: the mean of all samples as the first
// lane's plus the sum of the lanes' differences from it, each weighted by its share
// of the samples (a sum of n_lane mean_lane would overflow for means above the
// largest double / n), the waves' likewise, and M2 = sum_lanes (M2_lane + n_lane
// (mean_lane - mean)^2).  Sums over the block replace a tree of pairwise
// merges of three doubles, each with a division (about 1.3 us of a block's
// time; a 10^4-point FP64 scan of 1024 samples, N = 4: 86 -> 55 us).
// Every thread of the block must call it, those with no point to work on with
// `active` false (it synchronises unless `waves` is 1); `lds` holds kSmLds doubles.
constexpr int kSmLds = 4 * 16;  // four values of each of a block's waves

template <class Fam, typename T, int N>
__device__ __forceinline__ void sm_work(const ScanParams& p, uint64_t g, uint64_t sp, double* lds,
                                        unsigned w0, unsigned waves, bool active) {
  const unsigned lane = threadIdx.x - 64 * w0;
  const uint64_t j0 = sp * p.gps;
  const uint64_t j1 = (j0 + p.gps < p.n_groups) ? j0 + p.gps : p.n_groups;
  const uint64_t last = p.n_groups - 1;
  const int tail = (int)(p.n - 4 * last);  // samples in the scan's last group
  const uint64_t len = j1 - j0;
  const uint64_t rows = (len + blockDim.x - 1) / blockDim.x;
  const bool in_last = lane < (unsigned)(len - (rows - 1) * blockDim.x);
  LaneAcc<T> acc;
  acc.init((T)0);
  double count = 0.0;
  if (active) {
    Fam fam;
    fam.setup(p, p.g_base + g);
    with_form(fam, [&](const auto& f) {
      using F = std::decay_t<decltype(f)>;
      if constexpr (Phased<F>::value) {
        if (p.fast_counter) {
          const GenSampleMajorPhased gen{philox_point((uint32_t)(p.g_base + g), p.seed)};
          count = strided_groups<F, T, N>(f, gen, j0 + lane, blockDim.x, rows, in_last, last, tail, acc);
          return;
        }
      }
      const GenAny gen{p.g_base + g, p.seed};
      if constexpr (Phased<F>::value) {
        count = strided_groups<F, T, N>(f, gen, j0 + lane, blockDim.x, rows, in_last, last, tail, acc);
      } else {
        for (uint64_t j = j0 + lane; j < j1; j += blockDim.x) {
          T v[4];
          eval_group<F, T, N>(f, j, gen, v);
          if (count == 0.0) acc.init(v[0]);  // shift by the lane's first sample
          if (j == last && tail != 4) {
            acc.add_partial(v, tail);
            count += (double)tail;
          } else {
            acc.add4(v);
            count += 4.0;
          }
        }
      }
    });
  }
  const Moments m = to_moments(acc, count);
  const double n = (double)split_samples(p.n, p.n_groups, p.gps, sp);
  const double wt = m.n / n;
  double ref = first_lane(m.mean);
  double s = wave_sum(m.n > 0.0 ? wt * (m.mean - ref) : 0.0);
  const unsigned w = threadIdx.x >> 6;
  if (waves > 1) {
    const double wave_wt = wave_sum(wt);
    if ((threadIdx.x & 63u) == 0) {
      lds[w] = s;
      lds[16 + w] = ref;
      lds[32 + w] = wave_wt;
    }
    __syncthreads();
    s = lds[w0];
    ref = lds[16 + w0];
    for (unsigned i = 1; i < waves; ++i) s += lds[w0 + i] + lds[32 + w0 + i] * (lds[16 + w0 + i] - ref);
  }
  const double mean = ref + s;
  const double d = m.mean - mean;
  double m2 = wave_sum(m.n > 0.0 ? m.m2 + m.n * d * d : 0.0);
  if (waves > 1) {
    if ((threadIdx.x & 63u) == 0) lds[48 + w] = m2;
    __syncthreads();
    m2 = lds[48 + w0];
    for (unsigned i = 1; i < waves; ++i) m2 += lds[48 + w0 + i];
  }
  if (lane == 0 && active) {
    if (p.splits == 1) {
      finalize(p, g, Moments{n, mean, m2});
    } else {
      p.part_mean[sp * p.G + g] = mean;
      p.part_m2[sp * p.G + g] = m2;
    }
  }
  if (waves > 1) __syncthreads();
}

// The whole block on one point.
template <class Fam, typename T, int N>
__device__ __forceinline__ void sm_tile(const ScanParams& p, uint64_t g, uint64_t sp, double* lds) {
  sm_work<Fam, T, N>(p, g, sp, lds, 0, blockDim.x >> 6, true);
}

// A sample-major tile of a batch: `p.sm_points` consecutive points from `first`
// over sample piece sp, by a block of four waves.  A piece that fits the lanes of
// one or two waves gives each wave, or each pair, its own points.  A tile of one
// point costs its block a queue pop, the tile and scan records and the set-up one
// after another, latency that short pieces do not cover: a mix of 30 FP32 scans
// takes 2.63 ms, and took 4.27 with one point a tile.
template <class Fam, typename T, int N>
__device__ __forceinline__ void sm_tile_points(const ScanParams& p, uint64_t first, uint64_t sp, double* lds) {
  const uint64_t j0 = sp * p.gps;
  const uint64_t j1 = (j0 + p.gps < p.n_groups) ? j0 + p.gps : p.n_groups;
  const unsigned waves = j1 - j0 <= 64 ? 1 : j1 - j0 <= 128 ? 2 : 4;
  const unsigned teams = 4 / waves, w = threadIdx.x >> 6;
  const unsigned team = __builtin_amdgcn_readfirstlane(w / waves);
  const uint64_t left = p.G - first;
  const unsigned count = left < p.sm_points ? (unsigned)left : p.sm_points;
  for (unsigned i = 0; i < count; i += teams) {
    const unsigned at = i + team;
    const bool active = at < count;
    sm_work<Fam, T, N>(p, first + (active ? at : 0), sp, lds, team * waves, waves, active);
  }
}

// Merge of point g's pieces s0 .. s1-1 in order; loads run four pieces ahead of
// the merges.
__device__ __forceinline__ Moments merge_pieces(const ScanParams& p, uint64_t g, int s0, int s1) {
  Moments t{0.0, 0.0, 0.0};
  for (int s = s0; s < s1; s += 4) {
    double mean[4], m2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t at = (uint64_t)(s + i < s1 ? s + i : s1 - 1) * p.G + g;
      mean[i] = p.part_mean[at];
      m2[i] = p.part_m2[at];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (s + i < s1)
        t = merge(t, Moments{(double)split_samples(p.n, p.n_groups, p.gps, (uint64_t)(s + i)), mean[i], m2[i]});
  }
  return t;
}

// Second pass: merge of every point's pieces, then f and sigma.  Few pieces are
// merged by one thread a point; from kMergeTreeSplits on, 16 threads take
// consecutive runs of pieces and a tree over LDS joins them in order (one thread
// waits on its loads in turn: a scan of 1000 points in 128 pieces took 200 us, of
// which 73 after the main kernel, and takes 153 with the tree).  The choice depends on the piece count alone, so a
// point's result does not depend on the grid it is part of.  `lds` holds 3 x
// 256 doubles; blocks of 256 threads.
constexpr int kMergeTreeSplits = 16;

__device__ __forceinline__ void merge_body(const ScanParams& p, double* lds) {
  if (p.splits < kMergeTreeSplits) {
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t g = (uint64_t)blockIdx.x * 256u + threadIdx.x; g < p.G; g += stride)
      finalize(p, g, merge_pieces(p, g, 0, p.splits));
    return;
  }
  const unsigned pt = threadIdx.x & 15u, run = threadIdx.x >> 4;
  const int per = (p.splits + 15) / 16;
  const int s0 = (int)run * per, s1 = s0 + per < p.splits ? s0 + per : p.splits;
  for (uint64_t base = (uint64_t)blockIdx.x * 16u; base < p.G; base += (uint64_t)gridDim.x * 16u) {
    const uint64_t g = base + pt;
    Moments t{0.0, 0.0, 0.0};
    if (g < p.G && s0 < s1) t = merge_pieces(p, g, s0, s1);
    lds[threadIdx.x] = t.n;
    lds[256 + threadIdx.x] = t.mean;
    lds[512 + threadIdx.x] = t.m2;
    for (unsigned step = 1; step < 16; step <<= 1) {
      __syncthreads();
      if ((run & (2 * step - 1)) == 0) {
        const unsigned o = threadIdx.x + 16 * step;
        t = merge(t, Moments{lds[o], lds[256 + o], lds[512 + o]});
        lds[threadIdx.x] = t.n;
        lds[256 + threadIdx.x] = t.mean;
        lds[512 + threadIdx.x] = t.m2;
      }
    }
    if (run == 0 && g < p.G) finalize(p, g, t);
    __syncthreads();  // the next points reuse lds
  }
}

// Kernel bodies: the point-major scan (grid.x = point blocks, grid.y = sample
// pieces), the sample-major scan (grid.x = points, grid.y = pieces; `lds`
// holds 3 x 16 doubles) and per-sample integrand values of global point g
// (debugging, parity).
template <class Fam, typename T, int N>
__device__ __forceinline__ void point_major_body(const ScanParams& p) {
  load_tables<Fam>();
  for (uint64_t pb = blockIdx.x; pb < p.point_blocks; pb += gridDim.x)
    pm_tile<Fam, T, N>(p, pb * blockDim.x, blockIdx.y);
}

template <class Fam, typename T, int N>
__device__ __forceinline__ void sample_major_body(const ScanParams& p, double* lds) {
  load_tables<Fam>();
  for (uint64_t g = blockIdx.x; g < p.G; g += gridDim.x) sm_tile<Fam, T, N>(p, g, blockIdx.y, lds);
}

// Persistent batch body: the block pops tiles [begin, end) of the tile table
// through one atomic counter and runs them until the table is exhausted;
// every block reaches that exit.  `next` and `lds` are the kernel's shared
// memory (one word, 3 x 16 doubles).
template <class Fam, typename T, int N>
__device__ __forceinline__ void batch_body(const ScanParams* __restrict__ scans,
                                           const Tile* __restrict__ tiles, uint32_t begin,
                                           uint32_t end, uint32_t* counter, uint32_t* next,
                                           double* lds) {
  load_tables<Fam>();
  // far from the end of the table thread 0 pops the next tile while the block
  // runs the last one; near it a tile that waits for a busy block would keep the
  // device waiting (12 small FP64 scans: 507 us when it did, 388 without)
  uint32_t popped = 0;
  bool have = false;
  for (;;) {
    __syncthreads();  // the previous tile is done with `next` and `lds`
    if (threadIdx.x == 0) *next = have ? popped : begin + atomicAdd(counter, 1u);
    __syncthreads();
    const uint32_t t = *next;
    if (t >= end) break;
    have = end - t > 4u * gridDim.x;
    if (have && threadIdx.x == 0) popped = begin + atomicAdd(counter, 1u);
    const Tile tl = tiles[t];
    const ScanParams& p = scans[tl.scan];
    const uint64_t sp = tl.split_mode & ~kTileSampleMajor;
    if (tl.split_mode & kTileSampleMajor) {
      sm_tile_points<Fam, T, N>(p, tl.first, sp, lds);
    } else {
      pm_tile<Fam, T, N>(p, tl.first, sp);
    }
  }
}

template <class Fam, typename T, int N>
__device__ __forceinline__ void debug_values_body(const ScanParams& p, uint64_t g, uint64_t s0,
                                                  int64_t count, double* out) {
  load_tables<Fam>();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint64_t s = s0 + (uint64_t)i;
  Fam fam;
  fam.setup(p, g);
  T v[4];
  eval_group<Fam, T, N>(fam, s >> 2, GenAny{g, p.seed}, v);
  const unsigned k = (unsigned)(s & 3u);
  out[i] = (double)(k == 0 ? v[0] : k == 1 ? v[1] : k == 2 ? v[2] : v[3]);
}

}  // namespace zmc
