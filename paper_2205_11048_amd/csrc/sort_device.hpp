// Device pieces shared by the ID sort's kernels.
#pragma once

#include "gba_device.hpp"

namespace gba {

constexpr int kXcds = 8;   // MI355X: 8 accelerator dies, each with its own L2

// Mask of the active lanes whose digit equals this lane's digit.  Per bit,
// the lanes that differ from this one are the ballot of the bit, flipped
// where this lane's bit is 1: ballot ^ (0 or all ones), OR-ed into a mask of
// mismatches (one sign-extending bit extract, a compare for the ballot and
// one three-input bit operation per 32-lane half).
__device__ __forceinline__ uint64_t match_digit(uint32_t digit, int bits, bool active) {
  uint32_t diff_lo, diff_hi;
  {
    const uint64_t on = __ballot(active);
    diff_lo = ~(uint32_t)on;
    diff_hi = ~(uint32_t)(on >> 32);
  }
  for (int b = 0; b < bits; ++b) {
    const uint32_t x = (uint32_t)((int32_t)(digit << (31 - b)) >> 31);   // 0 or all ones: the lane's bit b
    const uint64_t bal = __ballot(x != 0u);
    // diff | (ballot ^ x) in one gfx950 three-input bit operation (table: S0 | (S1 ^ S2))
    diff_lo = __builtin_amdgcn_bitop3_b32(diff_lo, (uint32_t)bal, x, 0xF6);
    diff_hi = __builtin_amdgcn_bitop3_b32(diff_hi, (uint32_t)(bal >> 32), x, 0xF6);
  }
  const uint64_t m = ~(((uint64_t)diff_hi << 32) | diff_lo);
  return active ? m : 0ull;
}

// The same match for a digit width known at compile time (the loop unrolled).
template <int BITS>
__device__ __forceinline__ uint64_t match_digit_n(uint32_t digit, bool active) {
  uint32_t diff_lo, diff_hi;
  {
    const uint64_t on = __ballot(active);
    diff_lo = ~(uint32_t)on;
    diff_hi = ~(uint32_t)(on >> 32);
  }
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const uint32_t x = (uint32_t)((int32_t)(digit << (31 - b)) >> 31);
    const uint64_t bal = __ballot(x != 0u);
    diff_lo = __builtin_amdgcn_bitop3_b32(diff_lo, (uint32_t)bal, x, 0xF6);
    diff_hi = __builtin_amdgcn_bitop3_b32(diff_hi, (uint32_t)(bal >> 32), x, 0xF6);
  }
  const uint64_t m = ~(((uint64_t)diff_hi << 32) | diff_lo);
  return active ? m : 0ull;
}

// A copy of x that the compiler cannot tie to earlier uses of x, so values
// derived from it (LDS addresses) are recomputed where needed instead of
// being held in registers across a phase.
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Tile of scatter block b.  Blocks are dispatched round-robin over the 8 XCDs
// (block b on XCD b % 8); giving XCD x the x-th eighth of the tiles, in order,
// puts neighbouring tiles on one L2, which then merges their partial-line
// writes into the same digit bucket before they reach HBM.
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t tiles) {
  const int64_t x = b % kXcds, i = b / kXcds, q = tiles / kXcds, r = tiles % kXcds;
  return x * q + (x < r ? x : r) + i;
}

}  // namespace gba
