// Device-side arithmetic shared by the kernels: the forms of ceil(a/d) of the cost
// model (section 2: execution time c/s, transfer time t/B, each rounded up to whole ticks)
// and lane permutations inside a row of 16 lanes.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "cpeval_internal.hpp"

namespace cpeval {

// ceil(a/d) through the multiply-shift constants of the cost tables; {0, 0} (a free transfer)
// yields 0.  Exact for every a the table was built for.
__device__ __forceinline__ uint32_t magic_div(uint32_t a, Magic mg) {
    uint32_t nn = a + mg.dm1;
    return (uint32_t)(((uint64_t)nn * mg.mul + nn) >> 32);
}

// The same through a 4-byte table entry (d - 1 in the low byte, the upper 24 bits of the
// multiplier above it; the multiplier's low byte is taken as all ones); 0 (a free transfer)
// yields 0 for every a < 2^24.  Exact for every a the entry was built for.
__device__ __forceinline__ uint32_t magic_div(uint32_t a, uint32_t entry) {
    uint32_t nn = a + (entry & 0xffu);
    return (uint32_t)(((uint64_t)nn * (entry | 0xffu) + nn) >> 32);
}

// ceil(a/d) as one multiply-add rounded up: the tables hold a number just below 1/d (build_inverse_table), so that a times it
// lies above the whole number below a/d and not above the one at or above it; adding `base` makes the rounding one to whole
// numbers, which end up in the low bits.  Exact while a times the inverse's relative error is below 1: doubles for every 32-bit a, floats for
// a < 2^23 (kFloatMost), whatever the divisor.  An inverse of 0 (a free transfer) yields 0.  One instruction of four cycles where
// the multiply-shift forms take three or more, one of them a 64-bit product at a quarter of that rate.
// `base` comes from round_up, which sets the wavefront's rounding: whatever uses it comes after.  (Set behind the compiler's
// back, which would set it back in front of every operation on doubles.  A division of whole numbers that are not constants
// is done in floats: none behind round_up(float).)
__device__ __forceinline__ double round_up(double) {
    double base = 4503599627370496.0;        // 2^52
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 1" : "+v"(base));
    return base;
}
__device__ __forceinline__ uint32_t inverse_div(uint32_t a, double inverse, double base) {
    return (uint32_t)(uint64_t)__double_as_longlong(__builtin_fma((double)a, inverse, base));
}
// Floats count in units of 2^-6 (kFloatUnit): base is 2^17, and its bits, 0x48000000, leave a 32-bit word that the
// quotient is shifted into by kLaneIdBits.
__device__ __forceinline__ float round_up(float) {
    float base = kFloatUnit * 8388608.0f;
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 1" : "+v"(base));
    return base;
}
// A dividend out of one half of a 64-bit load, made a word of its own for a division by floats: the compiler would convert all 64
// bits, five instructions in place of one, as it did in the lane-window kernel (1,578 levels of 34 vertices, 118 partitions: 885
// -> 809 us a call).  Not for others, since it keeps conversions from being moved or folded: by doubles 467 levels of 8 vertices with
// 64-bit words took 174 us with it, 148 without, and 200,000 vertices in 20 levels with hubs 2.92 and 2.88 ms.
template <typename Tab>
__device__ __forceinline__ uint32_t word_for(uint32_t a) {
    if constexpr (sizeof(Tab) == sizeof(float)) asm("" : "+v"(a));
    return a;
}
__device__ __forceinline__ uint32_t inverse_bits(uint32_t a, float inverse, float base) {
    return __float_as_uint(__builtin_fmaf((float)a, inverse, base));
}
__device__ __forceinline__ uint32_t inverse_div(uint32_t a, float inverse, float base) {
    return inverse_bits(a, inverse, base) & 0x7fffffu;
}

// ceil(a/d) by division; d = 0 marks a free transfer.
__device__ __forceinline__ uint64_t plain_div(uint64_t a, uint64_t d) {
    return d ? (a + d - 1) / d : 0;
}

// x of the lane a DPP control word names (a permutation inside each row of 16 lanes):
// 0xB1 swaps neighbours, 0x4E swaps pairs, 0x141 mirrors halves of 8, 0x140 mirrors the row.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);
}

// (the same where every lane is named: no register holds a value for the others)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_row(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}

template <int CTRL>
__device__ __forceinline__ long long dpp_i64(long long x) {
    const uint32_t lo = dpp_u32<CTRL>((uint32_t)x);
    const uint32_t hi = dpp_u32<CTRL>((uint32_t)((unsigned long long)x >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// The smallest x of the wavefront, the same in every lane: rows of 16 by register permutations, the four rows'
// minima through scalar registers.
__device__ __forceinline__ uint32_t min_over_wave(uint32_t x) {
    x = min(x, dpp_u32<0xB1>(x));
    x = min(x, dpp_u32<0x4E>(x));
    x = min(x, dpp_u32<0x141>(x));
    x = min(x, dpp_u32<0x140>(x));
    return min(min((uint32_t)__builtin_amdgcn_readlane((int)x, 0), (uint32_t)__builtin_amdgcn_readlane((int)x, 16)),
               min((uint32_t)__builtin_amdgcn_readlane((int)x, 32), (uint32_t)__builtin_amdgcn_readlane((int)x, 48)));
}

// value + (ceil(a/d) << kLaneIdBits), the division by one multiply-add, the rest as one shift-and-add: the compiler would
// otherwise take the two apart.
template <typename Word>
__device__ __forceinline__ Word add_shifted(Word value, uint32_t x) {
    asm("" : "+v"(x));
    return value + ((Word)x << kLaneIdBits);
}
template <typename Word>
__device__ __forceinline__ Word add_quotient(Word value, uint32_t a, double inverse, double base) {
    return add_shifted(value, inverse_div(a, inverse, base));
}
template <typename Word>
__device__ __forceinline__ Word add_quotient(Word value, uint32_t a, float inverse, float base) {
    static_assert(kFloatUnit * 8388608.0f == 131072.0f && kLaneIdBits == 6, "0x48000000 << 6 leaves 32 bits");
    a = word_for<float>(a);
    return add_shifted(value, sizeof(Word) == 4 ? inverse_bits(a, inverse, base) : inverse_div(a, inverse, base));
}

}  // namespace cpeval
