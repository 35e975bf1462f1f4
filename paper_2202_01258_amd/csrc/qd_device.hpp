// qd_device.hpp -- device-side arithmetic of the generation kernels (gfx950).
//
// Counter-based random numbers, the Gaussian sampler and the fp32
// transcendental functions the kernels use.  Every function here is evaluated
// with explicit fused multiply-adds in a fixed order and the library is built
// with -ffp-contract=off, so each result is a fixed function of its inputs,
// independent of launch shape or scheduling.  That makes a generation
// reproducible bit for bit, which the insertion step needs: which elite keeps
// a cell is decided by comparing fp32 objectives.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/qd.h"

namespace qd {

// ---------------------------------------------------------------------------
// Philox4x32 with 10 rounds (Salmon et al., SC'11).  Counter words:
// (item, individual, generation, stream tag); key = the 64-bit seed.
// ---------------------------------------------------------------------------
enum : uint32_t { kTagInit = 0, kTagSelect = 1, kTagIso = 2, kTagCentroid = 3, kTagEnv = 4,
                  kTagCvtSample = 5, kTagInitLevel = 6 };

struct Key {
  uint32_t k0, k1;
};

// a ^ b ^ c in one v_bitop3_b32 (truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                        Key key) {
  uint32_t k0 = key.k0, k1 = key.k1;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint64_t m0 = (uint64_t)0xD2511F53u * c0;   // one v_mad_u64_u32 each
    const uint64_t m1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = xor3((uint32_t)(m1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(m0 >> 32), c3, k1);
    c0 = n0;
    c1 = (uint32_t)m1;
    c2 = n2;
    c3 = (uint32_t)m0;
    k0 += 0x9E3779B9u;                                 // Weyl schedule; the key is
    k1 += 0xBB67AE85u;                                 // wave-uniform (scalar unit)
  }
  return make_uint4(c0, c1, c2, c3);
}

// philox() for many individuals at the same items: what does not depend on the
// individual (counter word 1) -- one product in each of the first three rounds
// -- is worked out once per item, the rest is finished per individual.
struct PhiloxItem {
  uint32_t a, b, h, l;
};
struct PhiloxIndividual {
  uint32_t hi, lo;                                     // of round 2's first product
};

__device__ __forceinline__ PhiloxItem philox_item(uint32_t c0, uint32_t c2, uint32_t c3, Key key) {
  const uint64_t m0 = (uint64_t)0xD2511F53u * c0;
  const uint64_t m1 = (uint64_t)0xCD9E8D57u * c2;
  const uint64_t m1b = (uint64_t)0xCD9E8D57u * xor3((uint32_t)(m0 >> 32), c3, key.k1);
  const uint64_t m0c = (uint64_t)0xD2511F53u *
                       xor3((uint32_t)(m1b >> 32), (uint32_t)m1, key.k0 + 0x9E3779B9u);
  PhiloxItem v;
  v.a = (uint32_t)m0 ^ (key.k1 + 0xBB67AE85u);
  v.b = (uint32_t)m1b ^ (key.k0 + 2u * 0x9E3779B9u);
  v.h = (uint32_t)(m0c >> 32) ^ (key.k1 + 2u * 0xBB67AE85u);
  v.l = (uint32_t)m0c;
  return v;
}

__device__ __forceinline__ PhiloxIndividual philox_individual(uint32_t c1, uint32_t c2, Key key) {
  const uint64_t m1 = (uint64_t)0xCD9E8D57u * c2;
  const uint64_t m0 = (uint64_t)0xD2511F53u * ((uint32_t)(m1 >> 32) ^ c1 ^ key.k0);
  return PhiloxIndividual{(uint32_t)(m0 >> 32), (uint32_t)m0};
}

__device__ __forceinline__ uint4 philox_finish(const PhiloxItem& v, const PhiloxIndividual& w, Key key) {
  const uint64_t m1c = (uint64_t)0xCD9E8D57u * (v.a ^ w.hi);
  uint32_t c0 = (uint32_t)(m1c >> 32) ^ v.b, c1 = (uint32_t)m1c, c2 = v.h ^ w.lo, c3 = v.l;
  uint32_t k0 = key.k0 + 3u * 0x9E3779B9u, k1 = key.k1 + 3u * 0xBB67AE85u;
#pragma unroll
  for (int round = 3; round < 10; ++round) {
    const uint64_t m0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t m1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = xor3((uint32_t)(m1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(m0 >> 32), c3, k1);
    c0 = n0;
    c1 = (uint32_t)m1;
    c2 = n2;
    c3 = (uint32_t)m0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return make_uint4(c0, c1, c2, c3);
}

__device__ __forceinline__ float unit24(uint32_t x) {        // [0, 1)
  return (float)(x >> 8) * 0x1p-24f;
}

// ---------------------------------------------------------------------------
// fp32 functions from +, -, *, fma and IEEE division.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float fma32(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}

constexpr float kLn2Hi = 0x1.62e4p-1f;      // ln 2, 16 leading bits
constexpr float kLn2Lo = 0x1.7f7d1cp-20f;   // remainder of ln 2
constexpr float kLog2e = 0x1.715476p+0f;

// ---------------------------------------------------------------------------
// Gaussian sampler: one standard normal per Philox word x by inversion.
// k = (x & 0xffffff) + 1 (exact in fp32), p = k 2^-24; the magnitude is the
// half-normal quantile Phi^-1(1 - p/2), read from the table of cubics that
// qd_archive_init builds on the host (QD_NORMAL_ROWS rows of (c0, c1, c2,
// c3)): row = binary exponent of k times 16 plus its next four bits, taken
// straight from the fp32 bits of k; u = its remaining 19 bits as an integer;
// z = c0 + u (c1 + u (c2 + u c3)) by fma from the cubic term.  Bit 31 of x
// is the sign (bits 24..30 are not used).  Ten VALU instructions and one
// 16-byte LDS read per normal.  Every workgroup that draws normals stages the
// table in LDS (6160 bytes).
// ---------------------------------------------------------------------------
constexpr int kNormalRows = QD_NORMAL_ROWS;

struct Tables {
  const float4* ntab;   // LDS copy of the table
};

__device__ __forceinline__ void stage_normal_table(float4* dst, const float4* src, int tid,
                                                   int nthreads) {
  for (int i = tid; i < kNormalRows; i += nthreads) dst[i] = src[i];
}

__device__ __forceinline__ float normal(uint32_t x, const Tables& tb) {
  // k = (x & 0xffffff) + 1 as one 24-bit multiply-add (k * 1 + 1)
  uint32_t k;
  asm("v_mad_u32_u24 %0, %1, 1, 1" : "=v"(k) : "v"(x));
  const uint32_t b = __float_as_uint((float)k);
  // row = (b >> 19) - 127 * 16: a bit-field extract (kept as one instruction:
  // the compiler would rewrite it into a shift and a mask), then the scaled
  // index and the bias go into one shift-and-add of the address
  uint32_t e4;
  asm("v_bfe_u32 %0, %1, 19, 12" : "=v"(e4) : "v"(b));
  const float4 c = (tb.ntab - (127 << 4))[e4];
  const float u = (float)(b & 0x7ffffu);
  const float z = fma32(u, fma32(u, fma32(u, c.w, c.z), c.y), c.x);
  return __uint_as_float(__float_as_uint(z) ^ (x & 0x80000000u));   // one v_bitop3
}

// sqrt(20) sin(pi x) up to sign (the sign may differ by (-1)^rint(x)):
// r = x - rint(x) in [-1/2, 1/2] (exact), then r P(r^2), P the Taylor series
// of sqrt(20) sin(pi r) / r in u = r^2 through u^5 by Horner's rule.  Its
// coefficient k, sqrt(20) (-1)^k pi^(2k+1) / (2k+1)!, is worked out in double
// at compile time and rounded once to fp32.
constexpr float rsin_coef(int k) {
  double c = 4.47213595499957939282;   // sqrt(20)
  for (int i = 1; i <= 2 * k + 1; ++i) c *= 3.14159265358979323846 / (double)i;
  return (float)((k & 1) ? -c : c);
}
__device__ __forceinline__ float rsinpi(float x) {
  constexpr float c0 = rsin_coef(0), c1 = rsin_coef(1), c2 = rsin_coef(2);
  constexpr float c3 = rsin_coef(3), c4 = rsin_coef(4), c5 = rsin_coef(5);
  const float r = x - __builtin_rintf(x);
  const float u = r * r;
  float q = fma32(u, c5, c4);
  q = fma32(u, q, c3);
  q = fma32(u, q, c2);
  q = fma32(u, q, c1);
  q = fma32(u, q, c0);
  return r * q;
}

// e^x, input clamped to [-87, 88]: k = rint(x log2 e), r = x - k ln 2 in two
// fma steps, Taylor through r^7, times 2^k assembled in the exponent field.
__device__ __forceinline__ float exp32(float x) {
  const float y = x < -87.0f ? -87.0f : (x > 88.0f ? 88.0f : x);
  const float k = __builtin_rintf(y * kLog2e);
  float r = fma32(-k, kLn2Hi, y);
  r = fma32(-k, kLn2Lo, r);
  float p = fma32(r, 1.0f / 5040.0f, 1.0f / 720.0f);
  p = fma32(r, p, 1.0f / 120.0f);
  p = fma32(r, p, 1.0f / 24.0f);
  p = fma32(r, p, 1.0f / 6.0f);
  p = fma32(r, p, 0.5f);
  p = fma32(r, p, 1.0f);
  p = fma32(r, p, 1.0f);
  const float scale = __uint_as_float((uint32_t)((int32_t)k + 127) << 23);
  const float e = p * scale;
  return x == x ? e : x;
}

// a / b by the hardware reciprocal and one residual correction.  Used where
// the library has checked, over every input the caller can pass, that the
// result equals the IEEE quotient (qd_check_fast_arith).
__device__ __forceinline__ float div_rcp(float a, float b) {
  const float y = __builtin_amdgcn_rcpf(b);
  const float q = a * y;
  const float r = fma32(-q, b, a);
  return fma32(r, y, q);
}

// tanh: odd Taylor polynomial through x^11 for |x| < 0.3,
// else 1 - 2 / (e^{2|x|} + 1) with e^y by exp32's formula and an IEEE division;
// the sign is copied back.  The definition, which qd_check_fast_arith compares
// tanh32 with over all 2^32 inputs.
__device__ __forceinline__ float tanh32_plain(float x) {
  const float a = __builtin_fabsf(x);
  float r;
  if (a < 0.3f) {
    const float a2 = a * a;
    float p = fma32(a2, -1382.0f / 155925.0f, 62.0f / 2835.0f);
    p = fma32(a2, p, -17.0f / 315.0f);
    p = fma32(a2, p, 2.0f / 15.0f);
    p = fma32(a2, p, -1.0f / 3.0f);
    r = fma32(a * a2, p, a);
  } else {
    const float d = exp32(a + a) + 1.0f;
    r = 1.0f - 2.0f / d;
  }
  return __builtin_copysignf(r, x);
}

// tanh32_plain bit for bit, without its branch and with fewer instructions.
// Nearly every wave holds both kinds of lanes, so both sides are evaluated and
// one is selected: two chains side by side instead of one after the other.
//   * small side on x itself, every step being odd or even in x (the sign of
//     a zero is put back with the others');
//   * e^{2a}: with h = min(a, 44), the doubling goes into the constants (a
//     power of two commutes with every rounding here): k = rint(h 2 log2 e),
//     r/2 = h - k ln 2 / 2, and the Horner coefficient of r^i times 2^i.  The
//     integer k is the low mantissa bits of h 2 log2 e + 1.5 2^23, rounded
//     once (at 62 inputs k is exp32's neighbour, with the same tanh), so 2^k
//     goes into p's exponent by one shift-and-add (k <= 127, p in [0.7, 1.42));
//   * 2 / d as the corrected reciprocal of d / 2;
//   * a NaN takes the small side, which returns it.
__device__ __forceinline__ float tanh32(float x) {
  const float x2 = x * x;
  float q = fma32(x2, -1382.0f / 155925.0f, 62.0f / 2835.0f);
  q = fma32(x2, q, -17.0f / 315.0f);
  q = fma32(x2, q, 2.0f / 15.0f);
  q = fma32(x2, q, -1.0f / 3.0f);
  const float low = fma32(x * x2, q, x);
  const float a = __builtin_fabsf(x);
  const float h = __builtin_fminf(a, 44.0f);
  constexpr float kMagic = 0x1.8p+23f;
  const float t = fma32(h, 2.0f * kLog2e, kMagic);
  const float k = t - kMagic;
  float r = fma32(k, -0.5f * kLn2Hi, h);
  r = fma32(k, -0.5f * kLn2Lo, r);
  float p = fma32(r, 128.0f * (1.0f / 5040.0f), 64.0f * (1.0f / 720.0f));
  p = fma32(r, p, 32.0f * (1.0f / 120.0f));
  p = fma32(r, p, 16.0f * (1.0f / 24.0f));
  p = fma32(r, p, 8.0f * (1.0f / 6.0f));
  p = fma32(r, p, 4.0f * 0.5f);
  p = fma32(r, p, 2.0f);
  p = fma32(r, p, 1.0f);
  const float e = __uint_as_float(__float_as_uint(p) + (__float_as_uint(t) << 23));
  const float half_d = fma32(e, 0.5f, 0.5f);
  const float y = __builtin_amdgcn_rcpf(half_d);
  const float high = 1.0f - fma32(fma32(-y, half_d, 1.0f), y, y);
  return __builtin_copysignf(a >= 0.3f ? high : low, x);
}

// 1 / (1 + e^{-x}).  FAST takes the quotient from div_rcp (same bits for
// |x| <= 1, the range of the tanh states it is applied to).
template <bool FAST = true>
__device__ __forceinline__ float sigmoid32(float x) {
  const float d = 1.0f + exp32(-x);
  return FAST ? div_rcp(1.0f, d) : 1.0f / d;
}

// ---------------------------------------------------------------------------
// Wave64 helpers.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Orders the LDS accesses of one wave's lanes around this point.  A wave's LDS
// instructions execute in program order, so the compiler's order is all it
// takes: no wait for a write before the reads that follow it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Pairwise fold of one value per lane in the fixed tree h = 32, 16, ..., 1
// (the partial of lane l is added to that of lane l + h), without LDS: the
// steps h = 32 and 16 exchange halves and rows with the lane-swap
// instructions, h = 8 .. 1 rotate within rows of 16 lanes (DPP).  Every step
// leaves each lane holding its pair's sum (addition commutes, so both members
// of a pair hold the same bits), and the total ends in every lane.
// DPP within rows of 16 lanes: row_ror<N> gives lane l the value of lane
// (l - N) mod 16.
template <int N>
__device__ __forceinline__ float row_ror(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x120 + N, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ int row_ror(int v) {
  return (int)__builtin_amdgcn_update_dpp(0u, (uint32_t)v, 0x120 + N, 0xf, 0xf, true);
}

// Lanes 0 .. 7 of each row of 16 lanes, in every lane of the row.  One block:
// between separate broadcasts the compiler places waits that these do not need
// (no VGPR that a DPP instruction reads may be written by either of the two
// instructions before it, which the s_nop sees to).
#define QD_ROW_BCAST(K) "v_mov_b32_dpp %" #K ", %8 row_newbcast:" #K " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void row_bcast8(float v, float (&out)[8]) {
  __asm__("s_nop 1\n\t" QD_ROW_BCAST(0) QD_ROW_BCAST(1) QD_ROW_BCAST(2) QD_ROW_BCAST(3)
              QD_ROW_BCAST(4) QD_ROW_BCAST(5) QD_ROW_BCAST(6) QD_ROW_BCAST(7)
          : "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3]), "=&v"(out[4]),
            "=&v"(out[5]), "=&v"(out[6]), "=&v"(out[7])
          : "v"(v));
}

// Keeps a value in a register of its own (an empty asm that claims to change
// it): the optimiser no longer derives other registers from how it was made.
template <class T>
__device__ __forceinline__ void hold(T& v) { __asm__ volatile("" : "+v"(v)); }

// Makes a scalar opaque to the optimiser (an empty asm that claims to change
// it), so that what follows from it is worked out where it is used.
__device__ __forceinline__ void hold_scalar(int& v) { __asm__ volatile("" : "+s"(v)); }

// A lane's value, in a scalar register.
template <class T>
__device__ __forceinline__ T from_lane(T v, int lane) {
  return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// Lane 0 of each row of 16 lanes, in all its lanes.
__device__ __forceinline__ float row_first(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x150, 0xf, 0xf, true));
}

// From a value per part (64 / OPW lanes) to one per half: of four parts out[0]
// gets parts 0 and 2 in its halves, out[1] parts 1 and 3.
template <int OPW, class T>
__device__ __forceinline__ void halves_of_parts(T v, T (&out)[(OPW + 1) / 2]) {
  if constexpr (OPW != 4) {
    out[0] = v;
  } else {
    const uint32_t b = __builtin_bit_cast(uint32_t, v);
    const auto s = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    const uint32_t even = s[0], odd = s[1];   // (a bit_cast of an element takes the vector's first)
    out[0] = __builtin_bit_cast(T, even);
    out[1] = __builtin_bit_cast(T, odd);
  }
}

// Rows 0 .. 3: the first rows of a's and b's halves, a's lower, b's lower, a's
// upper, b's upper.
__device__ __forceinline__ float rows_from_halves(float a, float b) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]);
}

// One rotation step of a row-wide minimum of (value, index) pairs, smaller
// index first among equal values.
template <int N>
__device__ __forceinline__ void min_pair_row(float& v, int& idx) {
  const float ov = row_ror<N>(v);
  const int oi = row_ror<N>(idx);
  const bool take = ov < v || (ov == v && oi < idx);
  v = take ? ov : v;
  idx = take ? oi : idx;
}

// Folds of OPW offspring's partials at once, offspring i's total in every lane
// of the i-th 64 / OPW lanes.  The first steps pack values into halves and rows
// of one register (a half-swap of a with b leaves lane l of the sum holding
// a_l + a_{l+32} below lane 32 and b's pair sums above; the row swap then does
// the same for rows of 16 lanes), after which the rotations finish all of them.
// Each value goes through exactly the pairs of wave_fold_sum.
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float row_fold_sum(float v) {
  v = v + row_ror<8>(v);
  v = v + row_ror<4>(v);
  v = v + row_ror<2>(v);
  return v + row_ror<1>(v);
}
__device__ __forceinline__ float wave_fold_sum(float v) {
  v = swap32_add(v, v);
  return row_fold_sum(swap16_add(v, v));
}
template <int OPW>
__device__ __forceinline__ float fold_offspring(const float (&v)[OPW]) {
  if constexpr (OPW == 4) {
    return row_fold_sum(swap16_add(swap32_add(v[0], v[2]), swap32_add(v[1], v[3])));
  } else if constexpr (OPW == 2) {
    const float h = swap32_add(v[0], v[1]);
    return row_fold_sum(swap16_add(h, h));
  } else {
    return wave_fold_sum(v[0]);
  }
}

// The same for partials that are zero in lanes 32 .. 63 of the wave the R64
// order describes (at most 128 genes: its h = 32 step adds +0 and changes
// nothing), with two offspring's lanes packed into one register's halves: v[0]
// holds offspring 0 and OPW / 2, v[1] offspring 1 and 3.
template <int OPW>
__device__ __forceinline__ float fold_halves(const float (&v)[(OPW + 1) / 2]) {
  if constexpr (OPW == 4) return row_fold_sum(swap16_add(v[0], v[1]));
  else return row_fold_sum(swap16_add(v[0], v[0]));
}

// Fold of 8 slices, lane l holding slice l / 8 of sum l mod 8: pairs of slices
// four, two and one apart, the total in every lane.
__device__ __forceinline__ float slice_fold_sum(float v) {
  v = swap32_add(v, v);
  v = swap16_add(v, v);
  return v + row_ror<8>(v);
}

// Order-preserving map of an fp32 objective to u32 (-0 folded onto +0).
__device__ __forceinline__ uint32_t order_bits(float f) {
  const uint32_t u = __float_as_uint(f == 0.0f ? 0.0f : f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

}  // namespace qd
