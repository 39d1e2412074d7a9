// Device-side arithmetic shared by the kernels: the two forms of ceil(a/d) of the cost
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

// The same through the rounded form (CostTables::round): exact whatever the product, at the price of
// the remainder.
__device__ __forceinline__ uint32_t round_div(uint32_t a, Magic mg) {
    const uint32_t nn = a + mg.dm1;
    const uint32_t q = __umulhi(nn, mg.mul);
    return q + (nn - q * (mg.dm1 + 1u) > mg.dm1 ? 1u : 0u);
}

// ceil(a/d) as one multiply-add of doubles rounded up: a - 1/2 lies between two multiples of 1/d next to a/d, adding 1.5 * 2^52
// makes the rounding one to whole numbers (also below 0: a = 0, d = 1), and they end up in the low word.  Exact for every 32-bit a and every divisor:
// 1/d and the product are off by 2^-52 of a/d at most, the margin is 1/(2d).  inverse = 0 (a free transfer) yields 0.  One
// instruction of four cycles where the multiply-shift forms take three, one of them a 64-bit product at a quarter of that
// rate.  `base` is 1.5 * 2^52 from round_up_doubles, which sets the wavefront's rounding of doubles: whatever uses it comes after.
// (Set behind the compiler's back, which would set it back in front of every operation on doubles.)
__device__ __forceinline__ double round_up_doubles() {
    double base = 6755399441055744.0;
    asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 1" : "+v"(base));
    return base;
}
__device__ __forceinline__ double less_half(uint32_t a) { return (double)a - 0.5; }      // (exact)
__device__ __forceinline__ uint32_t inverse_div(double a_less_half, double inverse, double base) {
    return (uint32_t)(uint64_t)__double_as_longlong(__builtin_fma(a_less_half, inverse, base));
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

// The cost tables' three forms: 8-byte multiply-shift entries, the same with the remainder looked at, and
// 4-byte entries.  A table read by 64 lanes is the lane kernels' most expensive LDS access (random rows): 4-byte
// entries are taken where they are exact, and the remainder form where nothing else is, with 64-bit words.
enum Form { kMagic8, kRound8, kMagic4 };
template <int FORM> struct TabOf { typedef Magic type; };
template <> struct TabOf<kMagic4> { typedef uint32_t type; };

template <int FORM>
__device__ __forceinline__ uint32_t div_by(uint32_t x, typename TabOf<FORM>::type m) {
    if constexpr (FORM == kRound8) return round_div(x, m);
    else return magic_div(x, m);
}

// value + (x << 6) as one shift-and-add: the compiler would otherwise fold the shift into the product's
// upper half, which takes three instructions
template <typename Word>
__device__ __forceinline__ Word add_shifted(Word value, uint32_t x) {
    asm("" : "+v"(x));
    return value + ((Word)x << kLaneIdBits);
}

}  // namespace cpeval
