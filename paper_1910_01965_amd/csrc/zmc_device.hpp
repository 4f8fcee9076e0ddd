// zmc_device.hpp -- device building blocks of the parameter-scan kernels
// (gfx950, wave64): the counter-based generator, the uniform maps, the
// integrand families, per-lane accumulators and the FP64 merges.
//
// Method: direct Monte Carlo at every grid point (ZMCintegral-v5, Sec. 2,
// Eq. (1)); the paper leaves the generator, the sample layout and the error
// estimate open, and the library fixes them as stated in include/zmc.h.
#pragma once

#if defined(__HIPCC_RTC__)
// hipRTC (user integrands): its runtime header keeps the fixed-width types
// in its own namespace
using __hip_internal::int32_t;
using __hip_internal::int64_t;
using __hip_internal::uint32_t;
using __hip_internal::uint64_t;
#else
#include <hip/hip_runtime.h>
#include <stdint.h>
#endif

#include <type_traits>

#include "zmc_exp2_table.hpp"

namespace zmc {

constexpr int kMaxParams = 16;
constexpr int kMaxDims = 16;
constexpr int kAnyMaxDims = 8;  // integration dimensions of the any-family batch kernel
constexpr int kMaxUserParams = 16;  // constants passed to a user integrand

// Everything a scan kernel needs, passed by value as the kernel argument.
struct ScanParams {
  uint64_t G;            // grid points of this launch (local indices 0..G-1)
  uint64_t g_base;       // global flat index of local point 0 (chunked scans)
  uint64_t n;            // samples per point
  uint64_t n_groups;     // ceil(n / 4)
  uint64_t gps;          // groups per split
  uint64_t seed;
  uint64_t point_blocks; // ceil(G / block) (point-major)
  int32_t M, N, splits, family;
  int32_t fast_counter;  // 1 when every word block b and global index g is < 2^32
  int32_t small_index;   // 1 when every global index g is < 2^32
  int32_t n_params;      // user integrands: entries of params in use
  uint32_t sm_points;    // points of a sample-major tile (batches, server)
  int64_t axis_len[kMaxParams];
  int64_t axis_off[kMaxParams];
  uint64_t axis_stride[kMaxParams];  // prod of the lengths of later axes
  double axis_inv[kMaxParams];       // 1 / axis_stride
  double lo[kMaxDims], hi[kMaxDims];
  double vol;
  double params[kMaxUserParams];
  const double* axis;    // device: concatenated value lists
  double* f;             // device outputs [G]
  double* sigma;
  double* part_mean;     // device split partials [splits][G] (or null)
  double* part_m2;
};

// One unit of batched work: a point-major tile (256 consecutive grid points
// of one scan over one sample piece) or a sample-major tile (ScanParams::sm_points
// consecutive grid points, one sample piece, the whole block).
struct Tile {
  uint32_t scan;        // index into the batch's scan table
  uint32_t split_mode;  // bits 0..30: sample piece; bit 31: 1 = sample-major
  uint64_t first;       // point-major: first grid point; sample-major: its first point
};

constexpr uint32_t kTileSampleMajor = 0x80000000u;

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).  A round takes the high
// and low halves of the products of words 0 and 2 with the two multipliers
// and mixes the highs with words 1, 3 and the round key; the key advances by
// the two Weyl increments.  On gfx950 a 32x32->64 product is one full-rate
// v_mad_u64_u32 and the three-way xor is one v_bitop3_b32 (truth table 0x96).
// ---------------------------------------------------------------------------
constexpr uint32_t kPhiloxM0 = 0xD2511F53u;
constexpr uint32_t kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u;
constexpr uint32_t kPhiloxW1 = 0xBB67AE85u;

__host__ __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
  return a ^ b ^ c;
#endif
}

struct Words4 {
  uint32_t r[4];
};

// One Philox round on (c0, c1, c2, c3) with round key (k0, k1).
__host__ __device__ __forceinline__ void philox_round(uint32_t& c0, uint32_t& c1, uint32_t& c2,
                                                      uint32_t& c3, uint32_t k0, uint32_t k1) {
  const uint64_t p0 = (uint64_t)kPhiloxM0 * c0;
  const uint64_t p1 = (uint64_t)kPhiloxM1 * c2;
  const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
  const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
  c1 = (uint32_t)p1;
  c3 = (uint32_t)p0;
  c0 = n0;
  c2 = n2;
}

__host__ __device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                                         uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    philox_round(c0, c1, c2, c3, k0, k1);
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
  }
  Words4 w;
  w.r[0] = c0; w.r[1] = c1; w.r[2] = c2; w.r[3] = c3;
  return w;
}

// Block b of grid point g: counter (b lo, b hi, g lo, g hi), key = seed.
__host__ __device__ __forceinline__ Words4 philox_block(uint64_t b, uint64_t g, uint64_t seed) {
  return philox4x32_10((uint32_t)b, (uint32_t)(b >> 32), (uint32_t)g, (uint32_t)(g >> 32),
                       (uint32_t)seed, (uint32_t)(seed >> 32));
}

// ---------------------------------------------------------------------------
// Issue phases.  A CU's SIMD issues one wave64 VALU instruction every four
// cycles (a slot), or two from different waves when both are of the pairing
// kind.  Measured on the MI355X (loops of one or two instruction forms, 4 to 8
// waves per SIMD, cycles per instruction):
//   xor, and, shift, 32-bit add, bitop3, FP32 add/mul/fma    2.1 (pairs)
//   the same with an SGPR operand                            4.1 (of a pair, only
//                                                            one may read an SGPR)
//   v_mad_u64_u32, v_alignbit, conversions, FP64             4.1 (v_mad_u64_u32
//                                                            pairs with FP32 only)
//   v_exp_f32, v_sin_f32                                     8.2
// Philox alternates the two kinds: two wide products, then two three-way xors
// per round.  Left alone the waves drift apart, the xors of one meet the
// products of the others, and nothing pairs (4.1 cycles per instruction over a
// whole block).  So the wave priority is raised for the products and for the
// floating-point work of a group and lowered for the xors: a wave that reaches
// its xors waits there until the others have reached theirs, and the xors
// issue in pairs (3.1 per instruction, 297 cycles for three blocks instead of
// 393).  For this the round keys live in vector registers.
// The phases are empty asm statements through which the phase's values pass,
// so that data flow alone keeps the order and unused blocks still vanish.
// Effect (kernel times, start -> here): Gaussian 10^6 points x 4096 samples,
// N = 3, FP32 3.53 -> 2.97 ms, FP64 6.19 -> 5.68 ms; COSEXP 32^4 points x 4096,
// N = 2, FP32 3.12 -> 2.72 ms, FP64 6.99 -> 6.75 ms.
// ---------------------------------------------------------------------------

// Blocks whose phases run together: enough xors at a time to pair well, few
// enough values to keep five FP32 waves per SIMD (1, 2, 3, 4 blocks: 3.13,
// 3.06, 3.03, 3.04 ms for the FP32 Gaussian above).
constexpr int kMaxBatch = 3;
constexpr int kKeyRounds = 7;  // rounds 4..10, whose keys are kept in VGPRs

// x in a vector register (a wave-uniform value would go to an SGPR).
template <typename T> __host__ __device__ __forceinline__ T in_vgpr(T x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(x));
#endif
  return x;
}

#if defined(__HIP_DEVICE_COMPILE__)
#define ZMC_PHASE(NAME, T, PRIO)                                                              \
  template <int NB>                                                                           \
  __device__ __forceinline__ void NAME(T (&a)[NB], T (&b)[NB]) {                              \
    static_assert(NB >= 1 && NB <= kMaxBatch, "phases of one to three blocks");               \
    if constexpr (NB == 1)                                                                    \
      asm("s_setprio " PRIO : "+v"(a[0]), "+v"(b[0]));                                        \
    else if constexpr (NB == 2)                                                               \
      asm("s_setprio " PRIO : "+v"(a[0]), "+v"(b[0]), "+v"(a[1]), "+v"(b[1]));                \
    else                                                                                      \
      asm("s_setprio " PRIO                                                                   \
          : "+v"(a[0]), "+v"(b[0]), "+v"(a[1]), "+v"(b[1]), "+v"(a[2]), "+v"(b[2]));          \
  }
#else
#define ZMC_PHASE(NAME, T, PRIO) \
  template <int NB> __host__ __device__ inline void NAME(T (&)[NB], T (&)[NB]) {}
#endif
ZMC_PHASE(phase_mul, uint32_t, "2")
ZMC_PHASE(phase_int, uint64_t, "0")
ZMC_PHASE(phase_float, uint32_t, "3")
#undef ZMC_PHASE

// ---------------------------------------------------------------------------
// The same blocks for the point-major layout when b < 2^32 and g < 2^32 (the
// host checks both for the whole scan).  All lanes of a wave then share b and
// differ in g only, so the first two rounds split into a per-lane part that
// does not change from block to block (computed once per point) and a
// wave-uniform part that the compiler keeps in scalar registers:
//   round 1: (hi, lo)(M1 g) is per lane and fixed; (hi, lo)(M0 b) is uniform;
//   round 2: M0 times the round-1 word 0 = hi(M1 g) ^ k0 is per lane and
//            fixed; M1 times the round-1 word 2 = hi(M0 b) ^ k1 is uniform.
// Only rounds 3..10 multiply per-lane, per-block values.
// ---------------------------------------------------------------------------
struct PhiloxLane {
  uint32_t r1;   // round-1 output word 1: lo(M1 g)
  uint32_t h2;   // hi(M0 * round-1 word 0)
  uint32_t l2;   // lo(M0 * round-1 word 0)
  uint32_t k0, k1;
};

__host__ __device__ __forceinline__ PhiloxLane philox_lane(uint32_t g, uint64_t seed) {
  PhiloxLane L;
  L.k0 = (uint32_t)seed;
  L.k1 = (uint32_t)(seed >> 32);
  const uint64_t p1 = (uint64_t)kPhiloxM1 * g;
  const uint32_t w0 = (uint32_t)(p1 >> 32) ^ L.k0;  // counter word 1 (b hi) is 0
  L.r1 = (uint32_t)p1;
  const uint64_t p2 = (uint64_t)kPhiloxM0 * w0;
  L.h2 = (uint32_t)(p2 >> 32);
  L.l2 = (uint32_t)p2;
  return L;
}

__host__ __device__ __forceinline__ Words4 philox_block_pm(uint32_t b, const PhiloxLane& L) {
  // round 1 (key k): words 0, 1 per lane and fixed; words 2, 3 uniform
  const uint64_t q0 = (uint64_t)kPhiloxM0 * b;
  const uint32_t u2 = (uint32_t)(q0 >> 32) ^ L.k1;  // counter word 3 (g hi) is 0
  const uint32_t u3 = (uint32_t)q0;
  // round 2 (key k + W): the product with word 2 is uniform
  const uint32_t k0b = L.k0 + kPhiloxW0, k1b = L.k1 + kPhiloxW1;
  const uint64_t q1 = (uint64_t)kPhiloxM1 * u2;
  uint32_t c0 = L.r1 ^ ((uint32_t)(q1 >> 32) ^ k0b);
  uint32_t c1 = (uint32_t)q1;
  uint32_t c2 = L.h2 ^ (u3 ^ k1b);
  uint32_t c3 = L.l2;
  uint32_t k0 = k0b + kPhiloxW0, k1 = k1b + kPhiloxW1;
  {
    // round 3: word 1 and the key are uniform, word 3 is per lane and fixed,
    // so each new word is one per-lane product high half and one xor
    const uint64_t p0 = (uint64_t)kPhiloxM0 * c0;
    const uint64_t p1 = (uint64_t)kPhiloxM1 * c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ (c1 ^ k0);
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ (c3 ^ k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
  }
#pragma unroll
  for (int round = 3; round < 10; ++round) {
    philox_round(c0, c1, c2, c3, k0, k1);
    k0 += kPhiloxW0;
    k1 += kPhiloxW1;
  }
  Words4 w;
  w.r[0] = c0; w.r[1] = c1; w.r[2] = c2; w.r[3] = c3;
  return w;
}

// Rounds 4..10 of NB blocks in phases: words 0 and 2 in c0, c2, words 1 and 3 in
// the low halves of round 3's products q, p; kv as in_vgpr keys.
template <int NB>
__host__ __device__ __forceinline__ void philox_key_rounds(uint32_t (&c0)[NB], uint32_t (&c2)[NB],
                                                           uint64_t (&p)[NB], uint64_t (&q)[NB],
                                                           const uint32_t* kv, Words4 w[NB]) {
#pragma unroll
  for (int r = 0; r < kKeyRounds; ++r) {
    uint64_t pp[NB], qq[NB];
    phase_mul<NB>(c0, c2);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      pp[i] = (uint64_t)kPhiloxM0 * c0[i];
      qq[i] = (uint64_t)kPhiloxM1 * c2[i];
    }
    phase_int<NB>(pp, qq);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      c0[i] = xor3((uint32_t)(qq[i] >> 32), (uint32_t)q[i], kv[2 * r]);
      c2[i] = xor3((uint32_t)(pp[i] >> 32), (uint32_t)p[i], kv[2 * r + 1]);
      p[i] = pp[i];
      q[i] = qq[i];
    }
  }
  phase_float<NB>(c0, c2);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    w[i].r[0] = c0[i];
    w[i].r[1] = (uint32_t)q[i];
    w[i].r[2] = c2[i];
    w[i].r[3] = (uint32_t)p[i];
  }
}

__host__ __device__ __forceinline__ void philox_vgpr_keys(uint64_t seed, uint32_t* kv) {
#pragma unroll
  for (int i = 0; i < kKeyRounds; ++i) {
    kv[2 * i] = in_vgpr((uint32_t)seed + (uint32_t)(3 + i) * kPhiloxW0);
    kv[2 * i + 1] = in_vgpr((uint32_t)(seed >> 32) + (uint32_t)(3 + i) * kPhiloxW1);
  }
}

// The same with what the issue phases need.
struct PhiloxPhasedLane {
  PhiloxLane L;
  uint32_t l2k;                 // l2 ^ round 3's second key
  uint32_t kv[2 * kKeyRounds];  // keys of rounds 4..10, in vector registers
};

__host__ __device__ __forceinline__ PhiloxPhasedLane philox_phased_lane(uint32_t g, uint64_t seed) {
  PhiloxPhasedLane P;
  P.L = philox_lane(g, seed);
  P.l2k = P.L.l2 ^ (P.L.k1 + 2 * kPhiloxW1);
  philox_vgpr_keys(seed, P.kv);
  return P;
}

// Blocks b0 .. b0 + NB - 1 of the lane's grid point, NB <= kMaxBatch.
template <int NB>
__host__ __device__ __forceinline__ void philox_blocks_pm(uint32_t b0, const PhiloxPhasedLane& P,
                                                             Words4 w[NB]) {
  const PhiloxLane& L = P.L;
  uint32_t c0[NB], c2[NB], u1[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const uint32_t b = b0 + (uint32_t)i;
    // round 1 (key k): words 0, 1 per lane and fixed; words 2, 3 uniform
    const uint64_t q0 = (uint64_t)kPhiloxM0 * b;
    const uint32_t u2 = (uint32_t)(q0 >> 32) ^ L.k1;  // counter word 3 (g hi) is 0
    const uint32_t u3 = (uint32_t)q0;
    // round 2 (key k + W): the product with word 2 is uniform
    const uint32_t k0b = L.k0 + kPhiloxW0, k1b = L.k1 + kPhiloxW1;
    const uint64_t q1 = (uint64_t)kPhiloxM1 * u2;
    c0[i] = L.r1 ^ ((uint32_t)(q1 >> 32) ^ k0b);
    c2[i] = L.h2 ^ (u3 ^ k1b);
    u1[i] = (uint32_t)q1 ^ (L.k0 + 2 * kPhiloxW0);
  }
  uint64_t p[NB], q[NB];
  phase_mul<NB>(c0, c2);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    p[i] = (uint64_t)kPhiloxM0 * c0[i];
    q[i] = (uint64_t)kPhiloxM1 * c2[i];
  }
  phase_int<NB>(p, q);
  // round 3: word 1 and the key are uniform, word 3 is per lane and fixed,
  // so each new word is one per-lane product high half and one xor
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    c0[i] = (uint32_t)(q[i] >> 32) ^ u1[i];
    c2[i] = (uint32_t)(p[i] >> 32) ^ P.l2k;
  }
  philox_key_rounds<NB>(c0, c2, p, q, P.kv, w);
}

// ---------------------------------------------------------------------------
// The sample-major mirror (b < 2^32, g < 2^32): the wave shares g and its lanes
// differ in b, so round 1's M1 g and round 2's M0 product are wave-uniform.
// 18 products per lane and block instead of 20, and the xors in phases.  Uniform
// values sit in vector registers (see the issue phases).
// ---------------------------------------------------------------------------
struct PhiloxPoint {
  uint32_t k1;                  // the second key of round 1
  uint32_t u1;                  // round-1 word 1 ^ round 2's first key
  uint32_t x0;                  // hi(M0 * round-1 word 0) ^ round 2's second key
  uint32_t x3;                  // lo(M0 * round-1 word 0) ^ round 3's second key
  uint32_t k03;                 // round 3's first key
  uint32_t kv[2 * kKeyRounds];  // keys of rounds 4..10
};

__host__ __device__ __forceinline__ PhiloxPoint philox_point(uint32_t g, uint64_t seed) {
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  const uint64_t p1 = (uint64_t)kPhiloxM1 * g;
  const uint64_t p2 = (uint64_t)kPhiloxM0 * ((uint32_t)(p1 >> 32) ^ k0);  // counter word 1 is 0
  PhiloxPoint P;
  P.k1 = in_vgpr(k1);
  P.u1 = in_vgpr((uint32_t)p1 ^ (k0 + kPhiloxW0));
  P.x0 = in_vgpr((uint32_t)(p2 >> 32) ^ (k1 + kPhiloxW1));
  P.x3 = in_vgpr((uint32_t)p2 ^ (k1 + 2 * kPhiloxW1));
  P.k03 = in_vgpr(k0 + 2 * kPhiloxW0);
  philox_vgpr_keys(seed, P.kv);
  return P;
}

// Blocks b0 .. b0 + NB - 1 (b0 per lane), NB <= kMaxBatch.
template <int NB>
__host__ __device__ __forceinline__ void philox_blocks_sm(uint32_t b0, const PhiloxPoint& P, Words4 w[NB]) {
  uint32_t c0[NB], c2[NB];
  uint64_t p[NB], q[NB], r2[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    p[i] = (uint64_t)kPhiloxM0 * (b0 + (uint32_t)i);               // round 1
    r2[i] = (uint64_t)kPhiloxM1 * ((uint32_t)(p[i] >> 32) ^ P.k1);  // round 2 (counter word 3 is 0)
  }
  phase_int<NB>(p, r2);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    c0[i] = (uint32_t)(r2[i] >> 32) ^ P.u1;
    c2[i] = (uint32_t)p[i] ^ P.x0;
  }
  phase_mul<NB>(c0, c2);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    p[i] = (uint64_t)kPhiloxM0 * c0[i];  // round 3
    q[i] = (uint64_t)kPhiloxM1 * c2[i];
  }
  phase_int<NB>(p, q);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    c0[i] = xor3((uint32_t)(q[i] >> 32), (uint32_t)r2[i], P.k03);
    c2[i] = (uint32_t)(p[i] >> 32) ^ P.x3;
  }
  philox_key_rounds<NB>(c0, c2, p, q, P.kv, w);
}

// ---------------------------------------------------------------------------
// Uniform variates.  The per-dimension affine map y = A t + B is folded into
// each family; t is
//   FP64: u = (r + 1/2) 2^-32 exactly, A = hi - lo, B = lo (y = fma(A, u, B));
//   FP32: v = 1 + (r >> 9) 2^-23 in [1, 2) built from the bits (one
//         v_alignbit_b32), A = hi - lo, B = lo - A (1 - 2^-24), so that
//         A v + B = lo + A ((r >> 9) + 1/2) 2^-23.
// ---------------------------------------------------------------------------
template <typename T> struct Unif;

// FP64: the variate is the word itself, t = r (exact), and the affine
// constants carry the scale and the half-step offset of u = (r + 1/2) 2^-32:
// y = lo + h u = (h 2^-32) r + (lo + h 2^-33).  The power-of-two scalings are
// exact; the one rounding of B moves y by at most half an ulp from
// fma(h, u, lo), and the map costs a conversion and one fma per coordinate.
template <> struct Unif<double> {
  static __host__ __device__ __forceinline__ double t(uint32_t r) { return (double)r; }
  static __host__ __device__ inline void affine(double lo, double hi, double* A, double* B) {
    const double h = hi - lo;
    *A = h * 0x1p-32;
    *B = lo + h * 0x1p-33;
  }
};

template <> struct Unif<float> {
  static __device__ __forceinline__ float t(uint32_t r) {
    // (0x7F : r) >> 9 = 0x3F800000 | (r >> 9): a float in [1, 2)
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, r, 9u));
  }
  static __host__ __device__ inline void affine(double lo, double hi, double* A, double* B) {
    *A = hi - lo;
    *B = lo - (hi - lo) * (1.0 - 0x1p-24);
  }
};

template <typename T> __host__ __device__ __forceinline__ T fmaT(T a, T b, T c);
template <> __host__ __device__ __forceinline__ double fmaT(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}
template <> __host__ __device__ __forceinline__ float fmaT(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}

constexpr double kLog2e = 1.4426950408889634074;

// FP32 sine and cosine through the hardware units, which take their argument
// in revolutions.  The FP32 families carry phases in revolutions throughout:
// the per-point constants are multiplied by 1/(2 pi) in FP64 at set-up, before
// rounding, so a sample's phase r carries the same relative rounding as the
// phase in radians would, and r - rint(r) reduces it to [-1/2, 1/2] exactly
// (for |r| >= 2^23 an FP32 phase no longer resolves a revolution and the
// reduced phase is 0).
constexpr double kInv2Pi = 0.15915494309189533577;
constexpr double kPi = 3.14159265358979323846;
constexpr double kInv2PiLo = -9.839338337591243e-18;  // 1/(2 pi) - kInv2Pi

__device__ __forceinline__ float sin_turns(float r) {
  return __builtin_amdgcn_sinf(r - __builtin_rintf(r));
}

__device__ __forceinline__ float cos_turns(float r) {
  return __builtin_amdgcn_cosf(r - __builtin_rintf(r));
}

// FP64 sine and cosine of a phase r in revolutions.  t = r - rint(r) lies in
// [-1/2, 1/2] exactly.  Both reduce to sin(2 pi v) with v in [-1/4, 1/4]:
//   sin: v = t for |t| <= 1/4, else v = copysign(1/2, t) - t (sin(pi - a) =
//        sin a; exact, since 1/4 <= |t| <= 1/2): |v| = min(|t|, 1/2 - |t|),
//        whose minimum is one instruction where a compare and two selects are three;
//   cos: v = 1/4 - |t| (cos a = sin(pi/2 - a); exact for |t| >= 1/8, else
//        one rounding of at most 2^-55 revolutions).
// sin(2 pi v) = v P(v^2) with P of degree 8, from Chebyshev economization of
// the Taylor series on [-1/4, 1/4] (paper_1910_01965_amd/fp64_poly.py: the
// dropped terms are below 1.7e-19, the FP64 Horner evaluation within 2.2e-16
// relative of a 60-digit reference on a dense grid).  One polynomial serves
// both functions, with no octant selection.
__host__ __device__ __forceinline__ double sin_2pi_quarter(double v) {
  const double v2 = v * v;
  double p = 0.10071467531221244;
  p = __builtin_fma(p, v2, -0.7176853699001249);
  p = __builtin_fma(p, v2, 3.8199227975201033);
  p = __builtin_fma(p, v2, -15.094641368684599);
  p = __builtin_fma(p, v2, 42.05869391526577);
  p = __builtin_fma(p, v2, -76.70585975263434);
  p = __builtin_fma(p, v2, 81.60524927607172);
  p = __builtin_fma(p, v2, -41.34170224039975);
  p = __builtin_fma(p, v2, 6.283185307179586);
  return v * p;
}

// FP64 2^t.  n = rint(256 t) and f = 256 t - n in [-1/2, 1/2] (exact); with
// j = n mod 256, 2^t = 2^(n div 256) 2^(j/256) 2^(f/256).  2^(j/256) comes from
// a table in LDS as T (1 + eps), T rounded to double; 2^(f/256) - 1 is a
// degree-4 polynomial from Chebyshev economization (fp64_poly.py: dropped terms
// below 2.4e-18); T + T (f P(f) + eps) then carries one rounding (1.113e-16
// relative at most), and ldexp applies 2^(n div 256).  n is read from the low
// word of 256 t + 1.5 2^52, whose addition rounds to an integer.
// FP64 instructions never pair with anything (see the issue phases), so what
// counts is their number: 11, with three shifts and masks that pair, against 16
// for a polynomial on [-1/2, 1/2] without a table; the LDS reads (16 bytes a
// lane, their bank conflicts included) run beside them.  Table size: 64
// entries need one more fma, 512 save none.
// t is first clamped to [-2100, 2100], beyond which 2^t is 0 or inf in double:
// -inf then gives 0 and +inf gives inf, as exp does, and n always fits 32 bits
// (a NaN t is clamped too and gives 0; the parameter values it would come from
// must be finite).
constexpr int kExp2Entries = 256;
constexpr double kExp2Scale = 256.0;
constexpr double kRoundMagic = 0x1.8p52;  // x + kRoundMagic: rint(x) in the low word

#if defined(__HIP_DEVICE_COMPILE__)
static __device__ const double kExp2Table[2 * kExp2Entries] = {ZMC_EXP2_TABLE};

// The block's copy of the table (LDS); exp2_table_load fills it, and every
// thread of the block must call that before the first 2^t.
__device__ __forceinline__ double* exp2_table() {
  __shared__ __align__(16) double table[2 * kExp2Entries];
  return table;
}

__device__ __forceinline__ void exp2_table_load() {
  double* t = exp2_table();
  for (unsigned i = threadIdx.x; i < 2 * kExp2Entries; i += blockDim.x) t[i] = kExp2Table[i];
  __syncthreads();
}
#else
inline const double* exp2_table() {
  static const double table[2 * kExp2Entries] = {ZMC_EXP2_TABLE};
  return table;
}
__host__ __device__ inline void exp2_table_load() {}
#endif

// 2^(u / 256), u = n + f, m = n + kRoundMagic.
__host__ __device__ __forceinline__ double exp2_parts(double m, double f) {
  const int n = (int)(uint32_t)__builtin_bit_cast(uint64_t, m);
  const double* e = exp2_table() + 2 * (n & (kExp2Entries - 1));
  const double T = e[0], eps = e[1];
  double p = 2.239395396091414e-12;
  p = __builtin_fma(p, f, 3.3083030595039036e-09);
  p = __builtin_fma(p, f, 3.6655655969100867e-06);
  p = __builtin_fma(p, f, 0.002707606174062263);
  p = __builtin_fma(p, f, eps);
  return __builtin_ldexp(__builtin_fma(T, p, T), n >> 8);
}

// 2^t.  kNonPositive: the caller guarantees t <= 0 (or NaN), so only the lower
// clamp is needed.  256 t is exact, so it takes no instruction of its own.
template <bool kNonPositive = false>
__host__ __device__ __forceinline__ double exp2_fp64(double t) {
  t = __builtin_fmax(t, -2100.0);
  if constexpr (!kNonPositive) t = __builtin_fmin(t, 2100.0);
  const double m = __builtin_fma(t, kExp2Scale, kRoundMagic);
  return exp2_parts(m, __builtin_fma(t, kExp2Scale, -(m - kRoundMagic)));
}

// e^(-q) = 2^(-q log2 e).  kNonNegative: q >= 0 (or NaN, which gives 0).
template <bool kNonNegative = false>
__host__ __device__ __forceinline__ double exp_minus_fp64(double q) {
  q = __builtin_fmin(q, 2100.0 / kLog2e);
  if constexpr (!kNonNegative) q = __builtin_fmax(q, -2100.0 / kLog2e);
  constexpr double cs = -kExp2Scale * kLog2e;
  const double m = __builtin_fma(q, cs, kRoundMagic);
  return exp2_parts(m, __builtin_fma(q, cs, -(m - kRoundMagic)));
}

__host__ __device__ __forceinline__ double sin_turns(double r) {
  const double t = r - __builtin_rint(r);
  const double a = __builtin_fabs(t);
  return sin_2pi_quarter(__builtin_copysign(__builtin_fmin(a, 0.5 - a), t));
}

__host__ __device__ __forceinline__ double cos_turns(double r) {
  const double t = r - __builtin_rint(r);
  return sin_2pi_quarter(0.25 - __builtin_fabs(t));
}

// sin(s) in FP64, s in radians below 2^51: with c = 1 / pi, n = rint(s c), by adding
// kRoundMagic, and u = s c - n with one rounding, at u's own magnitude, so that neither a
// small phase nor a reduced one carries the rounding of the whole (a product rounded
// before its reduction has 5 to 20 % more error on boxes of 1 to 10); then (-1)^n
// sin(pi u) with the quarter-turn polynomial's coefficients scaled by powers of two.
// n's parity is the low bit of s c + kRoundMagic, shifted into the sign.
__host__ __device__ __forceinline__ double sin_radians(double s) {
  constexpr double c = 2.0 * kInv2Pi;
  const double m = __builtin_fma(s, c, kRoundMagic);
  const double u = __builtin_fma(s, c, -(m - kRoundMagic));
  const double u2 = u * u;
  double p = 0.10071467531221244 * 0x1p-17;
  p = __builtin_fma(p, u2, -0.7176853699001249 * 0x1p-15);
  p = __builtin_fma(p, u2, 3.8199227975201033 * 0x1p-13);
  p = __builtin_fma(p, u2, -15.094641368684599 * 0x1p-11);
  p = __builtin_fma(p, u2, 42.05869391526577 * 0x1p-9);
  p = __builtin_fma(p, u2, -76.70585975263434 * 0x1p-7);
  p = __builtin_fma(p, u2, 81.60524927607172 * 0x1p-5);
  p = __builtin_fma(p, u2, -41.34170224039975 * 0x1p-3);
  p = __builtin_fma(p, u2, 6.283185307179586 * 0x1p-1);
  const uint64_t odd = __builtin_bit_cast(uint64_t, m) << 63;
  return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, u * p) ^ odd);
}

// r less whole turns, in radians.  The product is rounded before its reduction: fused
// with it, its rounding error, of any size for a large r, would be the result.
__host__ __device__ inline double fold_turns(double r) {
#pragma clang fp contract(off)
  const double h = r * kInv2Pi;
  return (h - __builtin_rint(h)) * (2.0 * kPi);
}

// Phases of 2^48 and more, of which FP64 resolves a few hundredths of a turn and less:
// a box that reaches them is replaced by one whose map y = A t + B has A and B modulo
// 2 pi (t is a whole number), which keeps the phases that sin_radians gets below 2^50.
// On the host, once per scan.
inline void fold_sin_box(int N, double* lo, double* hi) {
  double reach = 0.0;
  for (int k = 0; k < N; ++k) reach += __builtin_fmax(__builtin_fabs(lo[k]), __builtin_fabs(hi[k]));
  if (reach < 0x1p48) return;
  for (int k = 0; k < N; ++k) {
    const double h = hi[k] - lo[k], a = fold_turns(h * 0x1p-32), b = fold_turns(lo[k] + h * 0x1p-33);
    lo[k] = b - 0.5 * a;
    hi[k] = lo[k] + a * 0x1p32;
  }
}

// Radians to a fraction of a revolution in [-1/2, 1/2], without the rounding of
// the whole revolutions: |error| below 2^-54 plus 2^-106 |s| (host checks of the
// phase reductions).
__host__ __device__ __forceinline__ double turns_fraction(double s) {
  const double r = s * kInv2Pi;
  const double e = __builtin_fma(s, kInv2Pi, -r) + s * kInv2PiLo;
  return (r - __builtin_rint(r)) + e;
}

// Families whose FP64 form takes 2^t from the block's table: the kernels load
// it first.
template <class Fam, class = void> struct UsesExp2Table : std::false_type {};
template <class Fam>
struct UsesExp2Table<Fam, std::void_t<decltype(Fam::kExp2Table)>>
    : std::integral_constant<bool, Fam::kExp2Table> {};

template <class Fam> __device__ __forceinline__ void load_tables() {
  if constexpr (UsesExp2Table<Fam>::value) exp2_table_load();
}

// Parameter x_l of grid point g (C order: stride_l = prod_{j>l} L_j), for the
// FP32 user integrands, which keep the code they had (see Phased).
__device__ __forceinline__ double param_x(const ScanParams& p, uint64_t g, int l) {
  const uint64_t i = (g / p.axis_stride[l]) % (uint64_t)p.axis_len[l];
  return p.axis[p.axis_off[l] + (int64_t)i];
}

// Parameters x_0, x_1, ... of grid point g in turn (C order: stride_l = prod_{j>l}
// L_j): with q_l = floor(g / stride_l), index i_l = q_l - q_(l-1) L_l.  For g < 2^32
// floor((g + 1/2) (1 / stride)) in FP64 is exact: the quotient stays 1 / (2 stride)
// away from an integer, far above the product's error of q 2^-52.  Six
// instructions a parameter instead of two 64-bit divisions of some 130 each
// (10^7 points x 16 samples over three parameters: 167 -> 145 us).
struct ParamCursor {
  const ScanParams& p;
  uint64_t g;
  double gh;
  uint32_t q = 0;
  __host__ __device__ __forceinline__ ParamCursor(const ScanParams& sp, uint64_t gg)
      : p(sp), g(gg), gh((double)(uint32_t)gg + 0.5) {}
  __host__ __device__ __forceinline__ uint64_t index(int l) {
    if (!p.small_index) return (g / p.axis_stride[l]) % (uint64_t)p.axis_len[l];
    const uint32_t ql = (uint32_t)(gh * p.axis_inv[l]);
    const uint32_t i = ql - q * (uint32_t)p.axis_len[l];
    q = ql;
    return i;
  }
  __host__ __device__ __forceinline__ double next(int l) { return p.axis[p.axis_off[l] + (int64_t)index(l)]; }
};

// ---------------------------------------------------------------------------
// Integrand families.  Each one holds the per-point constants (set up once
// per point in FP64, then rounded to T) and evaluates one sample from its N
// variates t[0..N-1].
// ---------------------------------------------------------------------------

// sin(sum_l x_l + sum_k y_k): the paper's test integrand, Eq. (2) and Eq. (4).
// FP64: the phase is summed in radians, coordinate by coordinate, as the formula
// states it (folding the box offsets into the point's constant, or carrying the
// coordinates in turns, adds up to 60 % to its error), and reduced as it is: a
// quarter turn taken off first, for a cosine without the sine's parity, rounds a
// phase of w radians to 2^-55 of a revolution, a relative error of 2e-16 / w in f (1.0,
// f = 0, on a box of 1e-17).  Boxes that reach 2^48 come folded (fold_sin_box).
template <typename T, int N> struct SinSum {
  static constexpr int kMinDims = 1;
  T A[N], B[N];
  T sx;        // FP64: sum of x; FP32: sum x + sum B (A and sx in revolutions)
  __host__ __device__ void setup(const ScanParams& p, uint64_t g) {
    double s = 0.0, sb = 0.0;
    ParamCursor x(p, g);
    for (int l = 0; l < p.M; ++l) s += x.next(l);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      double a, b;
      Unif<T>::affine(p.lo[k], p.hi[k], &a, &b);
      A[k] = sizeof(T) == 8 ? (T)a : (T)(a * kInv2Pi);
      B[k] = (T)b;
      sb += b;
    }
    if constexpr (sizeof(T) == 8)
      sx = __builtin_fabs(s) < 0x1p48 ? s : fold_turns(s);
    else
      sx = (T)((s + sb) * kInv2Pi);
  }
  __host__ __device__ __forceinline__ T value(const T* t) const {
    if constexpr (sizeof(T) == 8) {
      double sy = fmaT(A[0], t[0], B[0]);
#pragma unroll
      for (int k = 1; k < N; ++k) sy += fmaT(A[k], t[k], B[k]);
      return sin_radians(sx + sy);
    } else {
      float ph = sx;
#pragma unroll
      for (int k = 0; k < N; ++k) ph = fmaT(A[k], t[k], ph);
      return sin_turns(ph);
    }
  }
};

// exp(-(sum_{k<=M} x_k y_k^2 + sum_{k>M} y_k^2)).
// With every coefficient c_k of a point finite and >= 0 (c_k = x_k for k <= M,
// 1 beyond; times log2(e) in FP32), sqrt(c_k) is folded into that point's
// affine map, z_k = sqrt(c_k) y_k, and the point stores c_k = 1, so that the
// one formula fma(c_k y, y, q) gives sum_k z_k^2.  The tile loops run waves
// whose points are all folded on GaussUnit, which drops the product with
// c_k = 1 and so changes no bit: a point's value depends on that point alone.
template <typename T, int N> struct GaussUnit {
  T A[N], B[N];
  __device__ __forceinline__ T value(const T* t) const {
    // the first square is a plain product: fma(z, z, +0) would be the same
    // value but a three-operand instruction, which cannot dual-issue
    T q;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const T z = fmaT(A[k], t[k], B[k]);
      q = k == 0 ? z * z : fmaT(z, z, q);
    }
    if constexpr (sizeof(T) == 8) {
      return exp_minus_fp64<true>(q);  // q, a sum of squares, is >= 0
    } else {
      return __builtin_amdgcn_exp2f(-q);
    }
  }
};

template <typename T, int N> struct Gauss {
  static constexpr int kMinDims = 1;
  static constexpr bool kExp2Table = sizeof(T) == 8;
  using UnitForm = GaussUnit<T, N>;
  T A[N], B[N], c[N];   // FP32: c carries log2(e) for exp2
  bool unit;            // wave-uniform: c_k = 1 on every active lane of the wave
  __device__ void setup(const ScanParams& p, uint64_t g) {
    double x[N];
    bool fold = true;
    ParamCursor cursor(p, g);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      x[k] = (k < p.M) ? cursor.next(k) : 1.0;
      fold = fold && x[k] >= 0.0 && x[k] <= 0x1.fffffffffffffp+1023;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
      double a, b;
      Unif<T>::affine(p.lo[k], p.hi[k], &a, &b);
      const double ck = sizeof(T) == 8 ? x[k] : x[k] * kLog2e;
      const double s = fold ? sqrt(ck) : 1.0;
      A[k] = (T)(a * s);
      B[k] = (T)(b * s);
      c[k] = fold ? (T)1 : (T)ck;
    }
    unit = __builtin_amdgcn_ballot_w64(!fold) == 0;
  }
  __device__ __forceinline__ UnitForm unit_form() const {
    UnitForm u;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      u.A[k] = A[k];
      u.B[k] = B[k];
    }
    return u;
  }
  __device__ __forceinline__ T value(const T* t) const {
    T q;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const T y = fmaT(A[k], t[k], B[k]);
      q = k == 0 ? (c[k] * y) * y : fmaT(c[k] * y, y, q);
    }
    if constexpr (sizeof(T) == 8) {
      return exp_minus_fp64(q);
    } else {
      return __builtin_amdgcn_exp2f(-q);
    }
  }
};

// cos(x1 y1 + x2 y2 + sum_{k>=3} y_k) exp(-x3^2 y1 y2) + x4.
template <typename T, int N> struct CosExp;

template <int N> struct CosExp<float, N> {
  static constexpr int kMinDims = 2;
  float A[N], B[N];
  float x1, x2, nx3sq, x4;  // nx3sq = -x3^2 log2(e): the exponential is evaluated as 2^t
  float rest;               // sum of B_k for k >= 3, folded into the phase
  // x1, x2, rest and A_k, B_k (k >= 3) in revolutions (times 1/(2 pi))
  __device__ void setup(const ScanParams& p, uint64_t g) {
    const double turn = kInv2Pi;
    double sb = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      double a, b;
      Unif<float>::affine(p.lo[k], p.hi[k], &a, &b);
      A[k] = (float)(k >= 2 ? a * turn : a);
      B[k] = (float)b;
      if (k >= 2) sb += b;
    }
    ParamCursor x(p, g);
    x1 = (float)(x.next(0) * turn);
    x2 = (float)(x.next(1) * turn);
    const double x3 = x.next(2);
    nx3sq = (float)(-(x3 * x3) * kLog2e);
    x4 = (float)x.next(3);
    rest = (float)(sb * turn);
  }
  __device__ __forceinline__ float value(const float* t) const {
    const float y1 = fmaT(A[0], t[0], B[0]);
    const float y2 = fmaT(A[1], t[1], B[1]);
    float ph;
    if constexpr (N == 2) {
      ph = fmaT(x1, y1, x2 * y2);  // no further terms: no zero addend
    } else {
      ph = rest;
#pragma unroll
      for (int k = 2; k < N; ++k) ph = fmaT(A[k], t[k], ph);
      ph = fmaT(x1, y1, fmaT(x2, y2, ph));
    }
    const float e = __builtin_amdgcn_exp2f(nx3sq * y1 * y2);
    return fmaT(cos_turns(ph), e, x4);
  }
};

// FP64: the box coordinates y1, y2 are formed first, each with one rounding, and
// the exponent is their product.  Folding x3^2 into y1's map would save an
// instruction, but lets its two coefficients' roundings meet where y1 is near 0:
// on [-1, 0]^2 with x3 = 1000 the exponent of a sample is then off by 1e-11 instead of
// 1e-14, and for |x3| from 7e152 an infinite offset hides a finite one.  Folding
// x1, x2 and the other offsets into the phase's coefficients doubles the phase's
// error on boxes around 0.
template <int N> struct CosExp<double, N> {
  static constexpr int kMinDims = 2;
  static constexpr bool kExp2Table = true;
  double A[N], B[N];            // k >= 3: in revolutions (times 1/(2 pi))
  double x1, x2, nx3sq, x4;     // x1, x2 in revolutions; nx3sq = -x3^2 log2(e)
  __host__ __device__ void setup(const ScanParams& p, uint64_t g) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      double a, b;
      Unif<double>::affine(p.lo[k], p.hi[k], &a, &b);
      A[k] = k >= 2 ? a * kInv2Pi : a;
      B[k] = k >= 2 ? b * kInv2Pi : b;
    }
    ParamCursor x(p, g);
    x1 = x.next(0) * kInv2Pi;
    x2 = x.next(1) * kInv2Pi;
    const double x3 = x.next(2);
    nx3sq = -(x3 * x3) * kLog2e;
    x4 = x.next(3);
  }
  __host__ __device__ __forceinline__ double value(const double* t) const {
    const double y1 = fmaT(A[0], t[0], B[0]);
    const double y2 = fmaT(A[1], t[1], B[1]);
    double ph = fmaT(x1, y1, x2 * y2);
#pragma unroll
    for (int k = 2; k < N; ++k) ph += fmaT(A[k], t[k], B[k]);
    return __builtin_fma(cos_turns(ph), exp2_fp64(nx3sq * y1 * y2), x4);
  }
};

// 1: the sampler must reproduce the box volume exactly.
template <typename T, int N> struct Const {
  static constexpr int kMinDims = 1;
  __device__ void setup(const ScanParams&, uint64_t) {}
  __device__ __forceinline__ T value(const T*) const { return (T)1; }
};

// sum_k y_k.
template <typename T, int N> struct Linear {
  static constexpr int kMinDims = 1;
  T A[N], B[N];
  __device__ void setup(const ScanParams& p, uint64_t) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      double a, b;
      Unif<T>::affine(p.lo[k], p.hi[k], &a, &b);
      A[k] = (T)a;
      B[k] = (T)b;
    }
  }
  __device__ __forceinline__ T value(const T* t) const {
    T s = (T)0;
#pragma unroll
    for (int k = 0; k < N; ++k) s += fmaT(A[k], t[k], B[k]);
    return s;
  }
};

// ---------------------------------------------------------------------------
// One group of four consecutive samples s = 4j .. 4j+3 of point g uses the N
// Philox blocks b = jN .. jN+N-1 (words 4Nj .. 4Nj+4N-1, word i of the group
// being coordinate i mod N of sample 4j + i / N).
// ---------------------------------------------------------------------------
// Word-block generators of one grid point: any counter, or the point-major
// fast path (b < 2^32, g < 2^32, b shared by the wave).
struct GenAny {
  uint64_t g, seed;
  __device__ __forceinline__ Words4 block(uint64_t b) const { return philox_block(b, g, seed); }
  template <int NB>
  __device__ __forceinline__ void blocks(uint64_t b, Words4 w[NB]) const {
#pragma unroll
    for (int i = 0; i < NB; ++i) w[i] = block(b + (uint64_t)i);
  }
  template <typename T> __device__ __forceinline__ GenAny after(T&) const { return *this; }
};

struct GenPointMajor {
  PhiloxLane L;
  static __device__ __forceinline__ GenPointMajor make(uint32_t g, uint64_t seed) {
    return {philox_lane(g, seed)};
  }
  __device__ __forceinline__ Words4 block(uint64_t b) const {
    return philox_block_pm((uint32_t)b, L);
  }
};

struct GenPointMajorPhased {
  PhiloxPhasedLane P;
  static __device__ __forceinline__ GenPointMajorPhased make(uint32_t g, uint64_t seed) {
    return {philox_phased_lane(g, seed)};
  }
  template <int NB>
  __device__ __forceinline__ void blocks(uint64_t b, Words4 w[NB]) const {
    philox_blocks_pm<NB>((uint32_t)b, P, w);
  }
  // the same generator, whose blocks wait for v
  template <typename T> __device__ __forceinline__ GenPointMajorPhased after(T& v) const {
    GenPointMajorPhased g = *this;
    asm("" : "+v"(g.P.L.r1), "+v"(v));
    return g;
  }
};

struct GenSampleMajorPhased {
  PhiloxPoint P;
  template <int NB>
  __device__ __forceinline__ void blocks(uint64_t b, Words4 w[NB]) const {
    philox_blocks_sm<NB>((uint32_t)b, P, w);
  }
  template <typename T> __device__ __forceinline__ GenSampleMajorPhased after(T& v) const {
    GenSampleMajorPhased g = *this;
    asm("" : "+v"(g.P.k1), "+v"(v));
    return g;
  }
};

// Families whose groups run in issue phases: all but those that set
// kPhased = false (the FP32 user integrands: the order in which the compiler
// contracts a user's own products and sums into FMAs changes with the code
// around them, by up to 1e-8 of the result, so they keep the code they had).
template <class Fam, class = void> struct Phased : std::true_type {};
template <class Fam>
struct Phased<Fam, std::void_t<decltype(Fam::kPhased)>> : std::integral_constant<bool, Fam::kPhased> {};

// Word blocks drawn together (see the issue phases), in equal batches.
template <int N>
constexpr int kBatchBlocks = (N + (N + kMaxBatch - 1) / kMaxBatch - 1) / ((N + kMaxBatch - 1) / kMaxBatch);

// Blocks C .. of the group in batches; a sample is evaluated as soon as the
// batch that holds its last word (word sN + N - 1) has been drawn, and before
// the next batch starts (gen.after), so that in many dimensions only the
// variates of about one sample are live at a time.
template <class Fam, typename T, int N, class Gen, int C = 0>
__device__ __forceinline__ void eval_blocks(const Fam& fam, uint64_t b0, const Gen& gen, T t[4 * N],
                                            T v[4]) {
  if constexpr (C < N) {
    constexpr int NB = N - C < kBatchBlocks<N> ? N - C : kBatchBlocks<N>;
    Words4 w[NB];
    gen.template blocks<NB>(b0 + C, w);
#pragma unroll
    for (int i = 0; i < 4 * NB; ++i) t[4 * C + i] = Unif<T>::t(w[i / 4].r[i % 4]);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int last = (s * N + N - 1) / 4;
      if (last >= C && last < C + NB) v[s] = fam.value(t + s * N);
    }
    constexpr int done = 4 * (C + NB) / N;  // samples evaluated so far
    if constexpr (C + NB < N && done > 0 && done > 4 * C / N) {
      eval_blocks<Fam, T, N, Gen, C + NB>(fam, b0, gen.after(v[done - 1]), t, v);
    } else {
      eval_blocks<Fam, T, N, Gen, C + NB>(fam, b0, gen, t, v);
    }
  }
}

template <class Fam, typename T, int N, class Gen>
__device__ __forceinline__ void eval_group(const Fam& fam, uint64_t j, const Gen& gen, T v[4]) {
  if constexpr (Phased<Fam>::value) {
    T t[4 * N];
    eval_blocks<Fam, T, N, Gen>(fam, j * (uint64_t)N, gen, t, v);
  } else {
    T t[4 * N];
    const uint64_t b0 = j * (uint64_t)N;
    if constexpr (N <= kAnyMaxDims) {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const Words4 w = gen.block(b0 + c);
#pragma unroll
        for (int i = 0; i < 4; ++i) t[4 * c + i] = Unif<T>::t(w.r[i]);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) v[s] = fam.value(t + s * N);
    } else {
      // many dimensions: sample s is evaluated right after the block that holds
      // its last word (word sN + N - 1), so that only the variates of about one
      // sample are live at a time; the values are the same
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const Words4 w = gen.block(b0 + c);
#pragma unroll
        for (int i = 0; i < 4; ++i) t[4 * c + i] = Unif<T>::t(w.r[i]);
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if ((s * N + N - 1) / 4 == c) v[s] = fam.value(t + s * N);
      }
    }
  }
}

// Runs body(f) with f = the family's reduced form (Fam::UnitForm) when the
// family has one and its wave-uniform `unit` flag is set, else with fam
// itself; the two give the same bits, the reduced form in fewer instructions.
template <class Fam, class = void> struct HasUnitForm : std::false_type {};
template <class Fam>
struct HasUnitForm<Fam, std::void_t<typename Fam::UnitForm>> : std::true_type {};

template <class Fam, class Body>
__device__ __forceinline__ void with_form(const Fam& fam, Body&& body) {
  if constexpr (HasUnitForm<Fam>::value) {
    if (fam.unit) {
      body(fam.unit_form());
      return;
    }
  }
  body(fam);
}

// ---------------------------------------------------------------------------
// Per-lane accumulation: shifted sums of d = v - c and d^2 in T, each with a
// Kahan compensation term, four samples at a time.  c is one of the lane's own
// samples, which keeps the final M2 = S2 - S1^2 / n well conditioned.
// ---------------------------------------------------------------------------
template <typename T> struct LaneAcc {
  T c;
  T s1, e1, s2, e2;
  __device__ __forceinline__ void init(T shift) {
    c = shift;
    s1 = e1 = s2 = e2 = (T)0;
  }
  __device__ __forceinline__ static void kahan(T& s, T& e, T x) {
    const T y = x - e;
    const T tt = s + y;
    e = (tt - s) - y;
    s = tt;
  }
  __device__ __forceinline__ void add4(const T v[4]) {
    const T d0 = v[0] - c, d1 = v[1] - c, d2 = v[2] - c, d3 = v[3] - c;
    const T s = (d0 + d1) + (d2 + d3);
    const T q = fmaT(d0, d0, d1 * d1) + fmaT(d2, d2, d3 * d3);
    kahan(s1, e1, s);
    kahan(s2, e2, q);
  }
  // the first `valid` of the four values count (ragged last group)
  __device__ __forceinline__ void add_partial(const T v[4], int valid) {
    T w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (i < valid) ? v[i] : c;
    add4(w);
  }
};

// Welford state (count, mean, M2) in FP64.
struct Moments {
  double n, mean, m2;
};

template <typename T>
__device__ __forceinline__ Moments to_moments(const LaneAcc<T>& a, double count) {
  Moments m;
  m.n = count;
  if (count > 0.0) {
    const double S1 = (double)a.s1 - (double)a.e1;
    const double S2 = (double)a.s2 - (double)a.e2;
    m.mean = (double)a.c + S1 / count;
    m.m2 = S2 - S1 * (S1 / count);
    if (m.m2 < 0.0) m.m2 = 0.0;
  } else {
    m.mean = 0.0;
    m.m2 = 0.0;
  }
  return m;
}

// Chan, Golub, LeVeque pairwise merge; `a` is always the lower-indexed part
// so that every merge order is fixed.
__device__ __forceinline__ Moments merge(const Moments& a, const Moments& b) {
  if (b.n == 0.0) return a;
  if (a.n == 0.0) return b;
  Moments m;
  m.n = a.n + b.n;
  const double d = b.mean - a.mean;
  const double wb = b.n / m.n;
  m.mean = a.mean + d * wb;
  m.m2 = a.m2 + b.m2 + d * d * a.n * wb;
  return m;
}

// Sum over the 64 lanes in a fixed tree; every lane gets it.  Levels 1 to 8 move
// the value by DPP within rows of 16 lanes, 16 and 32 by a shuffle.
template <int Ctrl> __device__ __forceinline__ double dpp_move(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, Ctrl, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), Ctrl, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ double wave_sum(double x) {
  x += dpp_move<0xB1>(x);   // quad_perm [1,0,3,2]
  x += dpp_move<0x4E>(x);   // quad_perm [2,3,0,1]
  x += dpp_move<0x141>(x);  // row_half_mirror: the other quad of eight lanes
  x += dpp_move<0x140>(x);  // row_mirror: the other half of sixteen
  x += __shfl_xor(x, 16, 64);
  x += __shfl_xor(x, 32, 64);
  return x;
}

// The first lane's value (wave-uniform).
__device__ __forceinline__ double first_lane(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Samples in split sp (groups [sp*gps, min((sp+1)*gps, n_groups)), the last
// group of the scan possibly short).
__host__ __device__ __forceinline__ uint64_t split_samples(uint64_t n, uint64_t n_groups,
                                                           uint64_t gps, uint64_t sp) {
  const uint64_t j0 = sp * gps;
  uint64_t j1 = j0 + gps;
  if (j1 > n_groups) j1 = n_groups;
  if (j0 >= j1) return 0;
  uint64_t s1 = 4 * j1;
  if (s1 > n) s1 = n;
  return s1 - 4 * j0;
}

__device__ __forceinline__ void finalize(const ScanParams& p, uint64_t g, const Moments& m) {
  p.f[g] = p.vol * m.mean;
  p.sigma[g] = p.vol * sqrt(m.m2 / (m.n * (m.n - 1.0)));
}

}  // namespace zmc
