// Cost model of one cp_eval call: the divisors of every vertex cost (device
// speeds) and of every transfer cost (bandwidth matrix), as plain divisors and,
// where it is provably exact, as 32-bit multiply-shift constants.
#include <algorithm>
#include <cstring>

#include "cpeval_internal.hpp"

namespace cpeval {
namespace {

// ceil(a/d) for all 0 <= a <= amax through ((N*mul + N) >> 32) with N = a + d - 1,
// mul = M - 1, M = ceil(2^32/d).  Writing M*d = 2^32 + r (0 <= r < d) and
// N = q*d + rem:  N*M/2^32 = q + rem/d + N*r/(d*2^32), whose floor is q as long as
// N*r < 2^32.  N itself must fit 32 bits.
bool magic_for(int64_t d, int64_t amax, Magic &out) {
    if (d < 1 || d >= (int64_t)1 << 32) return false;
    uint64_t nmax = (uint64_t)amax + (uint64_t)d - 1;
    if (nmax >= (1ull << 32)) return false;
    uint64_t M = ((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d;
    uint64_t r = M * (uint64_t)d - (1ull << 32);
    if (r != 0 && nmax >= ((1ull << 32) + r - 1) / r) return false;  // nmax * r >= 2^32
    out.mul = (uint32_t)(M - 1);
    out.dm1 = (uint32_t)(d - 1);
    return true;
}

// The 4-byte form: ceil(a/d) = (N * M' - N * 0 + ...) >> 32 with N = a + d - 1 and
// M' = 256 * ceil(2^24 / d), a multiple of 256 (the kernels take the entry's low byte, which
// holds d - 1, as all ones: multiplier M' - 1, plus N).  With M' * d = 2^32 + r the floor is
// exact as long as N * r < 2^32, as above.
bool magic4_for(int64_t d, int64_t amax, uint32_t &out) {
    if (d < 1 || d > 256) return false;
    const uint64_t nmax = (uint64_t)amax + (uint64_t)d - 1;
    if (nmax >= (1ull << 32)) return false;
    const uint64_t m24 = ((1ull << 24) + (uint64_t)d - 1) / (uint64_t)d;     // <= 2^24
    const uint64_t r = 256 * m24 * (uint64_t)d - (1ull << 32);
    if (r != 0 && nmax >= ((1ull << 32) + r - 1) / r) return false;          // nmax * r >= 2^32
    out = (uint32_t)((m24 - 1) << 8) | (uint32_t)(d - 1);
    return true;
}

}  // namespace

int build_cost_tables(int32_t k, const int64_t *speeds, const int64_t *bandwidth,
                      bool narrow, int64_t max_c, int64_t max_t, CostTables &out) {
    for (int i = 0; i < k; ++i)
        if (speeds[i] < 1) return CP_ERR_SPEED;
    for (int i = 0; i < k; ++i)
        for (int j = 0; j < k; ++j)
            if (i != j && bandwidth[(size_t)i * k + j] < 1) return CP_ERR_BANDWIDTH;

    const size_t kk = (size_t)k * k;
    out.k = k;
    out.divisor.assign(table_entries(k), 0);
    out.magic.assign(table_entries(k), Magic{0, 0});
    out.tab4.assign(table_entries(k), 0u);
    bool ok = narrow && k <= kMagicMaxK;
    // a free transfer's entry 0 multiplies by 255: 0 ticks only while the volume is below 2^24
    bool ok4 = ok && max_t < ((int64_t)1 << 24) && max_c < ((int64_t)1 << 24);

    // (an entry is worked out once: the division in it takes longer than all the rest)
    for (size_t i = 0; i < (size_t)k; ++i)
        for (size_t j = 0; j < (size_t)k; ++j) {
            if (i == j) continue;  // same device: free, stays {0,0} / divisor 0
            // b sweep: row = device of the edge's source vertex, column = device of its target; t sweep: the other way round
            const int64_t d = bandwidth[i * k + j];
            const size_t at_b = i * k + j, at_t = kk + j * k + i;
            out.divisor[at_b] = out.divisor[at_t] = d;
            if (ok) {
                ok = magic_for(d, max_t, out.magic[at_b]);
                out.magic[at_t] = out.magic[at_b];
            }
            if (ok4) {
                ok4 = magic4_for(d, max_t, out.tab4[at_b]);
                out.tab4[at_t] = out.tab4[at_b];
            }
        }
    for (int i = 0; i < k; ++i) {
        out.divisor[2 * kk + i] = speeds[i];
        if (ok) ok = magic_for(speeds[i], max_c, out.magic[2 * kk + i]);
        if (ok4) ok4 = magic4_for(speeds[i], max_c, out.tab4[2 * kk + i]);
    }
    out.magic_ok = ok;
    out.tab4_ok = ok && ok4;
    return CP_OK;
}

bool wide_words_fit(int32_t k, const int64_t *speeds, const int64_t *bandwidth, int64_t max_c, int64_t max_t) {
    auto fits = [](int64_t d, int64_t amax) { return d < (int64_t)1 << 32 && (uint64_t)amax + (uint64_t)d - 1 < (1ull << 32); };
    for (int i = 0; i < k; ++i) {
        if (!fits(speeds[i], max_c)) return false;
        for (int j = 0; j < k; ++j)
            if (i != j && !fits(bandwidth[(size_t)i * k + j], max_t)) return false;
    }
    return true;
}

// The next number below 1.0 / d, which is at most half a unit above 1 / d, is a unit and a half below it at most, and no branch
// tells (past 2^53 the divisor is rounded, and only has to be larger than every dividend).
static double inverse_below(int64_t d) {
    const double x = 1.0 / (double)d;
    uint64_t bits;
    std::memcpy(&bits, &x, 8);
    --bits;
    double out;
    std::memcpy(&out, &bits, 8);
    return out;
}

// Rounded to the nearest float, and to the next one below where that is above.
static float float_below(double x) {
    const float f = (float)x;
    uint32_t bits;
    std::memcpy(&bits, &f, 4);
    bits -= (double)f > x ? 1u : 0u;
    float out;
    std::memcpy(&out, &bits, 4);
    return out;
}

template <typename T, typename Entry>
static void fill_inverses(int32_t k, const int64_t *speeds, const int64_t *bandwidth, T *out, Entry entry) {
    const size_t kk = (size_t)k * k;
    for (size_t i = 0; i < (size_t)k; ++i) {
        for (size_t j = 0; j < (size_t)k; ++j)
            out[i * k + j] = out[kk + j * k + i] = i == j ? T(0) : entry(bandwidth[i * k + j]);
        out[2 * kk + i] = entry(speeds[i]);
    }
}

void build_inverse_table(int32_t k, const int64_t *speeds, const int64_t *bandwidth, double *out) {
    fill_inverses(k, speeds, bandwidth, out, inverse_below);
}

void build_float_table(int32_t k, const int64_t *speeds, const int64_t *bandwidth, float *out) {
    fill_inverses(k, speeds, bandwidth, out, [](int64_t d) { return float_below(inverse_below(d) * kFloatUnit); });
}

}  // namespace cpeval
