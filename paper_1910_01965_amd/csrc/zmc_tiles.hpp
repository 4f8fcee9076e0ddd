// zmc_tiles.hpp -- the compiled-in scan kernels for gfx950 (templates over
// the integrand family, working precision and dimension) and the per-family
// launchers that each family translation unit instantiates.  The loops they
// run are in zmc_scan.hpp.
#pragma once

#include "zmc_internal.hpp"
#include "zmc_scan.hpp"

namespace zmc {

// Waves per SIMD asked of the kernels: enough for the issue phases to pair (two
// waves pair 60 % as often as four), unless what they then spill in the set-up and
// around the loops costs more.  Chosen from timings of each kernel at one and two
// waves less, N = 3..16, SIN_SUM, GAUSS and COSEXP.  GAUSS, whose kernels hold a
// general and a reduced form, spills first.
template <class Fam> constexpr bool kTwoForms = HasUnitForm<Fam>::value;

// Point-major.  FP32 at 5 against 4: SIN_SUM N = 16 4 % faster, COSEXP 3 %, Gaussian
// N = 8 0.98 vs 1.05 ms (5e5 points x 1024 samples), but Gaussian N = 13 467 vs 418 us,
// N = 16 1140 vs 483 us (10^5 points x 1024 samples; 608 at the compiler's own choice
// of unphased kernels).  FP64 at 4 up to N = 8 (Gaussian N = 8 1.48 vs 1.63 ms) and 3
// beyond (Gaussian N = 12 2.07 vs 2.30 ms).
template <class Fam, typename T, int N>
constexpr int kMinWaves = sizeof(T) == 4 ? (kTwoForms<Fam> && N > kAnyMaxDims ? 4 : 5) : N <= kAnyMaxDims ? 4 : 3;

// Batch kernels hold the point-major and the sample-major loops.  FP32 at 5, 4 and 3:
// 12 scans of 600 to 1000 points, N = 8, 119 : 100 : 100 for the Gaussian and 113 : 100 :
// 103 for SIN_SUM, 4 scans of 40000 points 128 : 100 : 113 and 104 : 100 : 118; N = 16
// Gaussian 206 : 100 : 77.  Five stay for N = 7, where small scans would gain 11 % and
// large ones lose 3 % (a batch of 512 scans: 5.80 s, 5.84 with four from N = 7 on, 5.75
// with five up to N = 8).  FP64 at 4 against 3: COSEXP N = 8 121 : 100, N = 7 97 : 100; at 3
// against 2: N = 16 118 to 137 : 100 in small scans, 85 to 93 : 100 in large ones.
template <class Fam, typename T, int N>
constexpr int kBatchWaves = sizeof(T) == 4 ? (N <= (kTwoForms<Fam> ? 6 : 7) ? 5 : kTwoForms<Fam> && N == 16 ? 3 : 4)
                                           : (N < kAnyMaxDims ? 4 : N < 16 ? 3 : 2);

template <class Fam, typename T, int N>
__global__ __launch_bounds__(256, (kMinWaves<Fam, T, N>)) void k_point_major(ScanParams p) {
  point_major_body<Fam, T, N>(p);
}

// Sample-major kernels: blocks of up to 256 threads (every automatic plan), or
// up to 1024 for N <= kAnyMaxDims (explicit plans), whose bound of 128 VGPRs a
// lane makes the FP64 kernels spill.  One or two waves per SIMD less than for
// the point-major kernels: the lane's word block and the point's Philox constants
// take some 20 VGPRs more, and what short scans spill in the set-up is most of them:
// Gaussian FP32, 1000 points x 1000 samples, at 4, 3 and 2 waves N = 8 20.8, 17.7 and
// 17.8 us, N = 12 32.6, 23.6 and 20.4, N = 16 47.4, 47.2 and 25.3 (unphased 18.1, 21.5, 27.1);
// 1500 points x 32768 samples N = 10 105 : 100 : 107.  Others FP32 at 4 and 3: N = 16
// 116 to 123 : 100 in such short scans, 97 to 101 : 100 in long ones.  FP64 Gaussian at 2 and 1:
// N = 16 52 and 39.5 us (36.9 unphased), long scans 83 : 100.
template <class Fam, typename T, int N>
constexpr int kSmMinWaves = sizeof(T) == 8 ? (N <= 5 ? 3 : kTwoForms<Fam> && N >= 15 ? 1 : 2)
                            : kTwoForms<Fam> ? (N <= 6 ? 4 : N <= 10 ? 3 : 2)
                                             : (N <= 12 ? 4 : 3);

template <class Fam, typename T, int N, int MaxThreads>
__global__ __launch_bounds__(MaxThreads, (MaxThreads > 256 ? 1 : kSmMinWaves<Fam, T, N>))
void k_sample_major(ScanParams p) {
  __shared__ double lds[kSmLds];
  sample_major_body<Fam, T, N>(p, lds);
}

// Batched scans: a persistent kernel per (family, precision, N) variant.  Its
// blocks pop tiles [begin, end) of the batch's tile table through one atomic
// counter (tiles are sorted longest first) and exit once the table is
// exhausted; every block reaches that exit.
template <class Fam, typename T, int N>
__global__ __launch_bounds__(256, (kBatchWaves<Fam, T, N>)) void k_batch(const ScanParams* __restrict__ scans,
                                               const Tile* __restrict__ tiles, uint32_t begin,
                                               uint32_t end, uint32_t* counter) {
  __shared__ uint32_t next;
  __shared__ double lds[kSmLds];
  batch_body<Fam, T, N>(scans, tiles, begin, end, counter, &next, lds);
}

// One tile of any family with N <= kAnyMaxDims in working precision T: the
// switch picks the template instance from the scan's own (family, N).  Scans
// of more dimensions run in their own per-variant kernels (k_batch), so that
// this kernel's register use stays that of its N <= 8 branches.
template <typename T>
__device__ __forceinline__ void run_tile_any(const ScanParams& p, const Tile& tl, double* lds) {
  const uint64_t sp = tl.split_mode & ~kTileSampleMajor;
  const bool sm = (tl.split_mode & kTileSampleMajor) != 0;
#define ZMC_TILE_CASE(FAM, NN)                                  \
  case FAM##_ID * 32 + NN:                                      \
    if (sm)                                                     \
      sm_tile_points<FAM<T, NN>, T, NN>(p, tl.first, sp, lds);  \
    else                                                        \
      pm_tile<FAM<T, NN>, T, NN>(p, tl.first, sp);              \
    break;
#define ZMC_TILE_CASES(FAM)                                                                  \
  ZMC_TILE_CASE(FAM, 1) ZMC_TILE_CASE(FAM, 2) ZMC_TILE_CASE(FAM, 3) ZMC_TILE_CASE(FAM, 4) \
  ZMC_TILE_CASE(FAM, 5) ZMC_TILE_CASE(FAM, 6) ZMC_TILE_CASE(FAM, 7) ZMC_TILE_CASE(FAM, 8)
  constexpr int SinSum_ID = ZMC_SIN_SUM, Gauss_ID = ZMC_GAUSS, Const_ID = ZMC_CONST,
                Linear_ID = ZMC_LINEAR, CosExp_ID = ZMC_COSEXP;
  static_assert(kAnyMaxDims == 8 && kMaxDims < 32, "the cases list N = 1..8");
  switch (p.family * 32 + p.N) {
    ZMC_TILE_CASES(SinSum)
    ZMC_TILE_CASES(Gauss)
    ZMC_TILE_CASES(Const)
    ZMC_TILE_CASES(Linear)
    ZMC_TILE_CASE(CosExp, 2) ZMC_TILE_CASE(CosExp, 3) ZMC_TILE_CASE(CosExp, 4)
    ZMC_TILE_CASE(CosExp, 5) ZMC_TILE_CASE(CosExp, 6) ZMC_TILE_CASE(CosExp, 7)
    ZMC_TILE_CASE(CosExp, 8)
    default:
      break;
  }
#undef ZMC_TILE_CASES
#undef ZMC_TILE_CASE
}

// Batched scans, one kernel for every family (N <= kAnyMaxDims) of one
// working precision: the blocks pop tiles of all scans from one queue.  FP32 at
// four waves per SIMD spills 49 VGPRs, none of them inside a loop over groups (a build
// that spilled 5 served 7.07e11 samples/s of the mix that this one serves at 7.05e11;
// at five waves 2 % less); FP64 spills in the loops beyond two (at four waves a
// served FP64 mix took 3.8 ms instead of 3.1).
template <typename T>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 2) void k_batch_any(const ScanParams* __restrict__ scans,
                                                   const Tile* __restrict__ tiles, uint32_t begin,
                                                   uint32_t end, uint32_t* counter) {
  __shared__ uint32_t next;
  __shared__ double lds[kSmLds];
  if constexpr (sizeof(T) == 8) exp2_table_load();
  uint32_t popped = 0;  // as in batch_body
  bool have = false;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) next = have ? popped : begin + atomicAdd(counter, 1u);
    __syncthreads();
    const uint32_t t = next;
    if (t >= end) break;
    have = end - t > 4u * gridDim.x;
    if (have && threadIdx.x == 0) popped = begin + atomicAdd(counter, 1u);
    const Tile tl = tiles[t];
    run_tile_any<T>(scans[tl.scan], tl, lds);
  }
}

template <class Fam, typename T, int N>
__global__ void k_debug_values(ScanParams p, uint64_t g, uint64_t s0, int64_t count,
                               double* out) {
  debug_values_body<Fam, T, N>(p, g, s0, count, out);
}

// ---------------------------------------------------------------------------
// Launchers of one family F in working precision T for N = Lo .. Lo + 7
// (Lo = 1 or 9); each (family, precision, N range) triple is instantiated in
// its own translation unit.
// ---------------------------------------------------------------------------
constexpr int kDimsPerUnit = 8;

template <template <typename, int> class F, typename T, int Lo>
struct FamilyOps {
  template <int N>
  static hipError_t main_n(const ScanParams& p, const Plan& plan, hipStream_t stream) {
    const dim3 block((unsigned)plan.block);
    const dim3 grid((unsigned)plan.grid_x, (unsigned)plan.splits);
    if (plan.mode == ZMC_MODE_POINT_MAJOR) {
      hipLaunchKernelGGL((k_point_major<F<T, N>, T, N>), grid, block, 0, stream, p);
    } else if (plan.block <= 256) {
      hipLaunchKernelGGL((k_sample_major<F<T, N>, T, N, 256>), grid, block, 0, stream, p);
    } else if constexpr (N <= kAnyMaxDims) {
      hipLaunchKernelGGL((k_sample_major<F<T, N>, T, N, 1024>), grid, block, 0, stream, p);
    } else {
      return hipErrorInvalidValue;  // the planner refuses such blocks
    }
    return hipGetLastError();
  }
  template <int N>
  static hipError_t values_n(const ScanParams& p, uint64_t g, uint64_t s0, int64_t count,
                             double* out, hipStream_t stream) {
    const unsigned blocks = (unsigned)((count + 255) / 256);
    hipLaunchKernelGGL((k_debug_values<F<T, N>, T, N>), dim3(blocks), dim3(256), 0, stream, p, g,
                       s0, count, out);
    return hipGetLastError();
  }
  template <int N>
  static hipError_t occupancy_n(int* blocks_per_cu) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_batch<F<T, N>, T, N>, 256, 0);
  }
  template <int N>
  static hipError_t batch_n(const ScanParams* scans, const Tile* tiles, uint32_t begin,
                            uint32_t end, uint32_t* counter, unsigned blocks, hipStream_t stream) {
    hipLaunchKernelGGL((k_batch<F<T, N>, T, N>), dim3(blocks), dim3(256), 0, stream, scans, tiles,
                       begin, end, counter);
    return hipGetLastError();
  }

  // Dispatch on N.  Defined out of line (not inline), so that the explicit
  // instantiation declarations below keep every other translation unit from
  // instantiating the kernels again.
  static hipError_t main(int N, const ScanParams& p, const Plan& plan, hipStream_t stream);
  static hipError_t values(int N, const ScanParams& p, uint64_t g, uint64_t s0, int64_t count,
                           double* out, hipStream_t stream);
  static hipError_t occupancy(int N, int* blocks_per_cu);
  static hipError_t batch(int N, const ScanParams* scans, const Tile* tiles, uint32_t begin,
                          uint32_t end, uint32_t* counter, unsigned blocks, hipStream_t stream);
};

// Instances below a family's smallest N (COSEXP needs two dimensions) are
// never built; validation rejects those descriptors before dispatch.
#define ZMC_BY_DIMS(CALL)                                                                 \
  switch (N - Lo) {                                                                       \
    case 0: if constexpr (Lo >= F<T, Lo>::kMinDims) return CALL(Lo); else break;          \
    case 1: return CALL(Lo + 1);                                                          \
    case 2: return CALL(Lo + 2);                                                          \
    case 3: return CALL(Lo + 3);                                                          \
    case 4: return CALL(Lo + 4);                                                          \
    case 5: return CALL(Lo + 5);                                                          \
    case 6: return CALL(Lo + 6);                                                          \
    case 7: return CALL(Lo + 7);                                                          \
    default: break;                                                                       \
  }                                                                                       \
  return hipErrorInvalidValue;
static_assert(kDimsPerUnit == 8, "ZMC_BY_DIMS lists eight dimensions");

template <template <typename, int> class F, typename T, int Lo>
hipError_t FamilyOps<F, T, Lo>::main(int N, const ScanParams& p, const Plan& plan, hipStream_t stream) {
#define ZMC_CALL(NN) main_n<NN>(p, plan, stream)
  ZMC_BY_DIMS(ZMC_CALL)
#undef ZMC_CALL
}

template <template <typename, int> class F, typename T, int Lo>
hipError_t FamilyOps<F, T, Lo>::values(int N, const ScanParams& p, uint64_t g, uint64_t s0,
                                       int64_t count, double* out, hipStream_t stream) {
#define ZMC_CALL(NN) values_n<NN>(p, g, s0, count, out, stream)
  ZMC_BY_DIMS(ZMC_CALL)
#undef ZMC_CALL
}

template <template <typename, int> class F, typename T, int Lo>
hipError_t FamilyOps<F, T, Lo>::occupancy(int N, int* blocks_per_cu) {
#define ZMC_CALL(NN) occupancy_n<NN>(blocks_per_cu)
  ZMC_BY_DIMS(ZMC_CALL)
#undef ZMC_CALL
}

template <template <typename, int> class F, typename T, int Lo>
hipError_t FamilyOps<F, T, Lo>::batch(int N, const ScanParams* scans, const Tile* tiles,
                                      uint32_t begin, uint32_t end, uint32_t* counter,
                                      unsigned blocks, hipStream_t stream) {
#define ZMC_CALL(NN) batch_n<NN>(scans, tiles, begin, end, counter, blocks, stream)
  ZMC_BY_DIMS(ZMC_CALL)
#undef ZMC_CALL
}
#undef ZMC_BY_DIMS

// Launchers of the any-family batch kernel in working precision T.
template <typename T>
struct AnyOps {
  static hipError_t occupancy(int* blocks_per_cu);
  static hipError_t batch(const ScanParams* scans, const Tile* tiles, uint32_t begin, uint32_t end,
                          uint32_t* counter, unsigned blocks, hipStream_t stream);
};

template <typename T>
hipError_t AnyOps<T>::occupancy(int* blocks_per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_batch_any<T>, 256, 0);
}

template <typename T>
hipError_t AnyOps<T>::batch(const ScanParams* scans, const Tile* tiles, uint32_t begin,
                            uint32_t end, uint32_t* counter, unsigned blocks, hipStream_t stream) {
  hipLaunchKernelGGL(k_batch_any<T>, dim3(blocks), dim3(256), 0, stream, scans, tiles, begin, end,
                     counter);
  return hipGetLastError();
}

#define ZMC_DECLARE_FAMILY_OPS(F)                                \
  extern template struct FamilyOps<F, float, 1>;                 \
  extern template struct FamilyOps<F, double, 1>;                \
  extern template struct FamilyOps<F, float, 1 + kDimsPerUnit>;  \
  extern template struct FamilyOps<F, double, 1 + kDimsPerUnit>;
ZMC_DECLARE_FAMILY_OPS(SinSum)
ZMC_DECLARE_FAMILY_OPS(Gauss)
ZMC_DECLARE_FAMILY_OPS(CosExp)
ZMC_DECLARE_FAMILY_OPS(Const)
ZMC_DECLARE_FAMILY_OPS(Linear)
#undef ZMC_DECLARE_FAMILY_OPS
extern template struct AnyOps<float>;
extern template struct AnyOps<double>;

}  // namespace zmc
