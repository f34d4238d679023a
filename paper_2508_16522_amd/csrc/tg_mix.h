// The mix of the task bodies on the device, shared by the executors and by
// the probe that measures its rate:
//   x ^= x << 13;  x ^= x >> 17;  x ^= x << 5;  x = x * kMul + kAdd  (mod 2^32)
// repeated R times on every word.
//
// What bounds it: instruction issue.  Each of these vector instructions takes
// about four cycles of its SIMD (16 lanes per cycle), the 32-bit multiply and the
// 64-bit shifts included; so the rate is set by
// the instructions per word.  Written out, a round is eight (three shifts,
// three xors, a multiply, an add).  Here it is six:
//   * kAdd = kMul * kPre (kMul is odd), so the add moves before the multiply,
//     where one v_xad_u32 does it together with the last xor;
//   * two words share the first two shifts: a 64-bit shift moves both, and the
//     bits that cross from one word into the other are masked in the xor that
//     follows (v_bitop3_b32: a ^ (b & mask)), at no cost.  The third shift
//     gains nothing from this: its xor is a v_xad_u32, which cannot mask.
// Measured (32 waves per SIMD in turn, 4 words per lane): 4.94e12 word-rounds/s
// with eight instructions, 5.43e12 with the add folded, 6.25e12 with the
// shared shifts; 6.67e12 with eight rounds a turn of the loop besides (8 waves per
// SIMD: 1.02 instructions per CU and cycle at 2.39 GHz, 3.9 cycles each; 4 waves
// 0.99, 2 waves 0.94, a lone wave 0.76).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tg {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kMul = 0x9E3779B1u, kAdd = 0x7F4A7C15u;

// Inverse of an odd number mod 2^32 (Newton's iteration doubles the correct
// low bits each time, from the three that m itself has).
constexpr uint32_t odd_inverse(uint32_t m) {
  uint32_t v = m;
  for (int i = 0; i < 4; ++i) v *= 2u - m * v;
  return v;
}
constexpr uint32_t kPre = kAdd * odd_inverse(kMul);
static_assert(kMul * odd_inverse(kMul) == 1u && kMul * kPre == kAdd, "the add moved before the multiply");

// The instructions by name: left to itself the compiler splits the 64-bit
// shifts into their halves, moves the add back behind the multiply and makes
// two instructions of a masked xor.  (The host compilation pass sees plain
// expressions.)
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ uint64_t shl13_pair(uint64_t v) {
  uint64_t d;
  asm("v_lshlrev_b64 %0, 13, %1" : "=v"(d) : "v"(v));
  return d;
}
__device__ __forceinline__ uint64_t shr17_pair(uint64_t v) {
  uint64_t d;
  asm("v_lshrrev_b64 %0, 17, %1" : "=v"(d) : "v"(v));
  return d;
}
// a ^ (b & mask): truth table 0x78 over (a, b, mask)
__device__ __forceinline__ uint32_t xor_masked(uint32_t a, uint32_t b, uint32_t mask) {
  uint32_t d;
  asm("v_bitop3_b32 %0, %1, %2, %3 bitop3:0x78" : "=v"(d) : "v"(a), "v"(b), "s"(mask));
  return d;
}
__device__ __forceinline__ uint32_t xor_add(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_xad_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}
#else
__device__ inline uint64_t shl13_pair(uint64_t v) { return v << 13; }
__device__ inline uint64_t shr17_pair(uint64_t v) { return v >> 17; }
__device__ inline uint32_t xor_masked(uint32_t a, uint32_t b, uint32_t mask) { return a ^ (b & mask); }
__device__ inline uint32_t xor_add(uint32_t a, uint32_t b, uint32_t c) { return (a ^ b) + c; }
#endif

__device__ __forceinline__ void mix_pair(uint32_t& x0, uint32_t& x1) {
  // x1:x0 << 13 carries the top 13 bits of x0 into x1's low ones
  const uint64_t s = shl13_pair(((uint64_t)x1 << 32) | x0);
  const uint32_t a0 = x0 ^ (uint32_t)s, a1 = xor_masked(x1, (uint32_t)(s >> 32), 0xFFFFE000u);
  // a1:a0 >> 17 carries the low 17 bits of a1 into a0's high ones
  const uint64_t t = shr17_pair(((uint64_t)a1 << 32) | a0);
  const uint32_t b0 = xor_masked(a0, (uint32_t)t, 0x7FFFu), b1 = a1 ^ (uint32_t)(t >> 32);
  x0 = xor_add(b0, b0 << 5, kPre) * kMul;
  x1 = xor_add(b1, b1 << 5, kPre) * kMul;
}

// A lone wavefront of a SIMD, as in a graph of wide tasks or on a chain that
// everything waits for, pays for every taken branch: eight rounds a turn took
// 1024 rounds of 4 words a lane from 58 to 48 us (the pure instruction time is
// 41; four a turn: 50), and change nothing where the SIMD has other wavefronts to
// issue from.  Tasks without rounds, which are a chain of memory round trips, fall
// through one test (100 levels of butterfly 166 -> 162 us).
template <class Round, class Around>
__device__ __forceinline__ void repeat_round(uint32_t R, Round&& round, Around&& around) {
  if (__builtin_expect(R == 0, 1)) return;
  constexpr uint32_t kTurn = 8;
  around(true);
  for (; R >= kTurn; R -= kTurn) {
#pragma unroll
    for (uint32_t i = 0; i < kTurn; ++i) round();
  }
  for (; R; --R) round();
  around(false);
}

// R rounds on every word of x.  around(true) runs before the first round,
// around(false) after the last, neither if there are none.
template <class Around>
__device__ __forceinline__ uint32_t mix_rounds(uint32_t x, uint32_t R, Around&& around) {
  repeat_round(R, [&] {
    x ^= x << 13;
    x ^= x >> 17;
    x = xor_add(x, x << 5, kPre) * kMul;
  }, around);
  return x;
}
template <class Around>
__device__ __forceinline__ u32x2 mix_rounds(u32x2 v, uint32_t R, Around&& around) {
  uint32_t x0 = v[0], x1 = v[1];
  repeat_round(R, [&] { mix_pair(x0, x1); }, around);
  return u32x2{x0, x1};
}
template <class Around>
__device__ __forceinline__ u32x4 mix_rounds(u32x4 v, uint32_t R, Around&& around) {
  uint32_t x0 = v[0], x1 = v[1], x2 = v[2], x3 = v[3];
  repeat_round(R, [&] {
    mix_pair(x0, x1);
    mix_pair(x2, x3);
  }, around);
  return u32x4{x0, x1, x2, x3};
}
template <class V>
__device__ __forceinline__ V mix_rounds(V v, uint32_t R) {
  return mix_rounds(v, R, [](bool) {});
}

}  // namespace tg
