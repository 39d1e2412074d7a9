// PCT priority lists (paper, section 4.1): per partition, the vertices grouped by
// device and, inside a device, ordered by descending PCT = b, equal values by
// ascending vertex number.  That is a segmented sort under the key
// (device, -b, vertex), done here as a least-significant-digit radix sort with one
// segment per partition:
//
//   key(v) = device(v) << bb | (max_b - b(v))        bb = bit length of max_b
//
// Sorting keys ascending with a stable sort whose input is in vertex order yields the
// list; the vertex number never enters the key.  Each digit (8 bits, or 9 where that
// saves a pass) takes three launches: per-tile digit counts, an exclusive scan of the counts per partition in
// (digit, tile) order, and a stable scatter.
//
// Ranking inside a wavefront is done by ballots (one per key bit): lanes with equal digits
// find each other, every lane reads its digit's counter, the last lane of a group moves it on.
//
// Partitions of at most 20,480 vertices with 32-bit keys are sorted by one workgroup each, entirely
// inside LDS (as a bucket is, the whole partition its bucket).
//
// Long partitions of 32-bit keys take a shorter way where they can: a pass on the LEADING 9
// bits cuts a partition into 512 buckets, and a bucket of at most 4,096 or 8,192 items is then
// sorted on the remaining bits entirely inside LDS by one workgroup (LDS to
// LDS, by bins where its keys are spread) and leaves as the finished list: an item crosses HBM three times (keys
// written, the leading digit's scatter, the bucket sort) whatever the key length.  Whether every bucket fits
// is only known on the device, after the scan of the leading digit's counts.  So both
// continuations are launched -- the leading digit's scatter and the bucket sort, or the
// ordinary passes from the low digit up -- and a flag the bucket check sets lets the kernels of
// one of them return at once.  With rows of b per partition, one kernel writes the keys and
// counts their leading digit.
// The leading scatter keeps vertices in order only where a bucket may have to be ranked by digits; bins have the vertex
// number in their key.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "cpeval_internal.hpp"
#include "launch.hpp"

namespace cpeval {

namespace {

constexpr int kMaxRadix = 512;
constexpr int kSortRounds = 16;                           // items per thread
// Items per workgroup = threads x 16.  Long partitions take 1024 threads: 16384 items, so a
// digit's run in a tile averages 64 items and leaves as full lines; short ones take 256
// threads (4096 items) so that several workgroups share a partition.
constexpr int kSortThreadsLong = 1024, kSortThreadsShort = 256;
constexpr int kSortLongFrom = 65536;                      // vertices from which the long tile is used
inline int sort_threads(int32_t n) { return n >= kSortLongFrom ? kSortThreadsLong : kSortThreadsShort; }
// Passes over a key of `bits` bits: digits of 8 bits, of up to 9 where allowed.
inline int pct_passes(int bits, bool wide) { return (bits + (wide ? 9 : 8) - 1) / (wide ? 9 : 8); }

// the bucket path cuts a partition by its leading kBucketBits bits, in tiles of kLeadThreads x 16
// items: half the long tile, so that two workgroups of the leading scatter share a compute unit
// and one's ranking overlaps the other's loads and stores
constexpr int kBucketBits = 9, kBuckets = 1 << kBucketBits;
constexpr int kLeadThreads = 512;

inline int hip_status(hipError_t e) { return e == hipSuccess ? CP_OK : CP_ERR_HIP; }

// ---------------------------------------------------------------- keys

struct KeyArgs {
    const void *b;            // ticks [n][P]
    const uint8_t *assign;
    int64_t a_stride_p, a_stride_v;
    void *keys;               // Key [P][n]
    int32_t *status;
    uint32_t *flag;           // of the bucket path, cleared here (a launch less), or null
    int64_t max_b;
    int32_t n, P, k, bb;
};

__device__ __forceinline__ void clear_flag(const KeyArgs &a) {
    if (a.flag != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *a.flag = 0;
}

// A kernel launched for one of two continuations returns at once when the device-side flag
// says the other one runs (flag == nullptr: always runs).  Uniform for the whole grid.
struct Gate {
    const uint32_t *flag;
    uint32_t want;
    __device__ __forceinline__ bool closed() const { return flag != nullptr && *flag != want; }
};

// b is vertex-major, the sort wants one contiguous key array per partition: 64 x 64
// tiles through LDS.  The device id is read in whichever phase reads it coalesced.
template <typename Tick, typename Key>
__global__ __launch_bounds__(256) void pct_keys_kernel(KeyArgs a) {
    __shared__ Key tile[64][65];
    clear_flag(a);
    const int lane = threadIdx.x & 63, row0 = threadIdx.x >> 6;
    const int64_t v0 = (int64_t)blockIdx.x * 64, q0 = (int64_t)blockIdx.y * 64;
    const Tick *b = (const Tick *)a.b;
    Key *keys = (Key *)a.keys;
    const bool ids_by_partition = a.a_stride_p == 1;      // vertex-major assignments
    bool bad_id = false, bad_b = false;
    for (int r = row0; r < 64; r += 4) {
        const int64_t v = v0 + r, q = q0 + lane;
        if (v < a.n && q < a.P) {
            long long bv = (long long)b[v * a.P + q];
            if (bv < 0 || bv > a.max_b) { bad_b = true; bv = bv < 0 ? 0 : a.max_b; }
            Key key = (Key)(a.max_b - bv);
            if (ids_by_partition) {
                uint32_t dev = a.assign[q * a.a_stride_p + v * a.a_stride_v];
                if (dev >= (uint32_t)a.k) { bad_id = true; dev = (uint32_t)a.k - 1; }
                key |= (Key)dev << a.bb;
            }
            tile[r][lane] = key;
        }
    }
    __syncthreads();
    for (int r = row0; r < 64; r += 4) {
        const int64_t q = q0 + r, v = v0 + lane;
        if (v < a.n && q < a.P) {
            Key key = tile[lane][r];
            if (!ids_by_partition) {
                uint32_t dev = a.assign[q * a.a_stride_p + v * a.a_stride_v];
                if (dev >= (uint32_t)a.k) { bad_id = true; dev = (uint32_t)a.k - 1; }
                key |= (Key)dev << a.bb;
            }
            keys[q * a.n + v] = key;
        }
    }
    if (bad_id) atomicOr(a.status, CP_STATUS_BAD_DEVICE_ID);
    if (bad_b) atomicOr(a.status, CP_STATUS_B_OUT_OF_RANGE);
}

// The same from b laid out [P][n]: no transpose, one key per thread.
template <typename Tick, typename Key>
__global__ __launch_bounds__(256) void pct_keys_rows_kernel(KeyArgs a) {
    clear_flag(a);
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= a.n) return;
    bool bad_b = false, bad_id = false;
    for (int64_t q = blockIdx.y; q < a.P; q += gridDim.y) {
        long long bv = (long long)((const Tick *)a.b)[q * a.n + v];
        if (bv < 0 || bv > a.max_b) { bad_b = true; bv = bv < 0 ? 0 : a.max_b; }
        uint32_t dev = a.assign[q * a.a_stride_p + v * a.a_stride_v];
        if (dev >= (uint32_t)a.k) { bad_id = true; dev = (uint32_t)a.k - 1; }
        ((Key *)a.keys)[q * a.n + v] = (Key)(a.max_b - bv) | (Key)dev << a.bb;
    }
    if (bad_id) atomicOr(a.status, CP_STATUS_BAD_DEVICE_ID);
    if (bad_b) atomicOr(a.status, CP_STATUS_B_OUT_OF_RANGE);
}

// ---------------------------------------------------------------- one digit pass


template <int RB, typename Key>
__device__ __forceinline__ uint32_t digit_of(Key key, int shift) {
    return (uint32_t)(key >> shift) & ((1u << RB) - 1);
}

// The counting kernels keep several copies of the histogram in LDS, a lane adding to copy
// (lane mod copies): the vertices of a wavefront often share a handful of leading digits, and
// adds to one counter queue up behind each other.  A copy's row is one word longer than the
// radix, so that equal digits in different copies fall into different banks.
template <int kThreads, int kRadix>
struct Histogram {
    static constexpr int kCopies = kThreads >= 1024 ? 8192 / kRadix : 8;      // 16 or 32; 8 for the short tile
    uint32_t h[kCopies][kRadix + 1];
    __device__ __forceinline__ void clear(int tid) {
        for (int i = tid; i < kCopies * (kRadix + 1); i += kThreads) (&h[0][0])[i] = 0;
    }
    __device__ __forceinline__ void add(int tid, uint32_t d) { atomicAdd(&h[tid & (kCopies - 1)][d], 1u); }
    __device__ __forceinline__ uint32_t total(uint32_t d) const {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kCopies; ++w) c += h[w][d];
        return c;
    }
};

// counts[q][digit][tile] = items of the tile with that digit
template <typename Key, int kSortThreads, int RB>
__global__ __launch_bounds__(kSortThreads) void pct_count_kernel(const Key *__restrict__ keys, int32_t n,
                                                                 int32_t tiles, int shift,
                                                                 uint32_t *__restrict__ counts, Gate gate) {
    constexpr int kSortTile = kSortThreads * kSortRounds, kRadix = 1 << RB;
    static_assert(kSortThreads >= kRadix, "one thread per digit writes the counts");
    if (gate.closed()) return;
    __shared__ Histogram<kSortThreads, kRadix> hist;
    const int tid = threadIdx.x;
    const int32_t tile = (int32_t)(blockIdx.x % (uint32_t)tiles), q = (int32_t)(blockIdx.x / (uint32_t)tiles);
    hist.clear(tid);
    __syncthreads();
    const Key *src = keys + (int64_t)q * n;
    const int64_t base = (int64_t)tile * kSortTile;
    Key key[kSortRounds];
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {               // all loads first, then the LDS updates
        const int64_t i = base + r * kSortThreads + tid;
        key[r] = i < n ? src[i] : (Key)0;
    }
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int64_t i = base + r * kSortThreads + tid;
        if (i < n) hist.add(tid, digit_of<RB>(key[r], shift));
    }
    __syncthreads();
    if (tid < kRadix) counts[((int64_t)q * kRadix + tid) * tiles + tile] = hist.total(tid);
}

// Keys from rows of b ([P][n]) and, in the same pass, the counts of their leading digit: what
// pct_keys_rows_kernel and the first pct_count_kernel do, with one read of b.  A thread takes four
// consecutive vertices per round (VEC: as one 16-byte load of b, one 4-byte load of device ids, one
// 16-byte store of keys; needs n % 4 == 0, unit stride between a partition's ids and aligned rows).
struct alignas(16) Keys4 { uint32_t x[4]; };
template <typename Tick> struct alignas(16) Ticks4 { Tick x[4]; };
template <typename Tick, bool VEC>
__global__ __launch_bounds__(kLeadThreads) void pct_keys_count_kernel(KeyArgs a, int32_t tiles, int shift,
                                                                          uint32_t *__restrict__ counts) {
    constexpr int kRadix = 1 << kBucketBits, kTile = kLeadThreads * kSortRounds;
    constexpr int kQuadRounds = kSortRounds / 4;
    __shared__ Histogram<kLeadThreads, kRadix> hist;
    clear_flag(a);
    const int tid = threadIdx.x;
    const int32_t tile = (int32_t)(blockIdx.x % (uint32_t)tiles), q = (int32_t)(blockIdx.x / (uint32_t)tiles);
    hist.clear(tid);
    __syncthreads();
    const Tick *b = (const Tick *)a.b + (int64_t)q * a.n;
    const uint8_t *ids = a.assign + q * a.a_stride_p;
    uint32_t *keys = (uint32_t *)a.keys + (int64_t)q * a.n;
    const int32_t base = tile * kTile;
    uint32_t key[kQuadRounds][4];
    bool bad_b = false, bad_id = false;
#pragma unroll
    for (int r = 0; r < kQuadRounds; ++r) {
        const int32_t i0 = base + (r * kLeadThreads + tid) * 4;
        Ticks4<Tick> bv{};
        uint32_t dv = 0;
        if (VEC) {
            if (i0 < a.n) {
                bv = *(const Ticks4<Tick> *)(b + i0);
                dv = *(const uint32_t *)(ids + i0);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i0 + j < a.n) {
                    bv.x[j] = b[i0 + j];
                    dv |= (uint32_t)ids[(int64_t)(i0 + j) * a.a_stride_v] << (8 * j);
                }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            long long t = (long long)bv.x[j];
            if (t < 0 || t > a.max_b) { bad_b = true; t = t < 0 ? 0 : a.max_b; }
            uint32_t dev = (dv >> (8 * j)) & 0xffu;
            if (dev >= (uint32_t)a.k) { bad_id = true; dev = (uint32_t)a.k - 1; }
            key[r][j] = (uint32_t)(a.max_b - t) | dev << a.bb;
        }
        if (VEC) {
            if (i0 < a.n) *(Keys4 *)(keys + i0) = Keys4{{key[r][0], key[r][1], key[r][2], key[r][3]}};
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i0 + j < a.n) keys[i0 + j] = key[r][j];
        }
    }
    if (bad_id) atomicOr(a.status, CP_STATUS_BAD_DEVICE_ID);
    if (bad_b) atomicOr(a.status, CP_STATUS_B_OUT_OF_RANGE);
#pragma unroll
    for (int r = 0; r < kQuadRounds; ++r) {
        const int32_t i0 = base + (r * kLeadThreads + tid) * 4;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i0 + j < a.n) hist.add(tid, digit_of<kBucketBits>(key[r][j], shift));
    }
    __syncthreads();
    if (tid < kRadix) counts[((int64_t)q * kRadix + tid) * tiles + tile] = hist.total(tid);
}

// In place: counts[q][*] becomes its exclusive prefix sum in (digit, tile) order, i.e.
// where the tile's run of that digit starts in the partition's output.  One workgroup per
// partition walks the entries 4,096 at a time, four neighbours per thread (entries is a
// multiple of the radix, so of four, and every partition's row is 16-byte aligned).
struct alignas(16) Counts4 { uint32_t x[4]; };
__global__ __launch_bounds__(1024) void pct_scan_kernel(uint32_t *__restrict__ counts, int32_t entries, Gate gate) {
    __shared__ uint32_t wave_sum[2][16];                  // (two sets: one barrier per step)
    if (gate.closed()) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t *c = counts + (int64_t)blockIdx.x * entries;
    uint32_t carry = 0;
    int set = 0;
    for (int32_t base = 0; base < entries; base += 4096, set ^= 1) {
        const int32_t i = base + tid * 4;
        Counts4 v{};
        if (i < entries) v = *(const Counts4 *)(c + i);
        const uint32_t sum = v.x[0] + v.x[1] + v.x[2] + v.x[3];
        uint32_t inc = sum;                               // inclusive scan over the wavefront
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t up = __shfl_up(inc, off);
            if (lane >= off) inc += up;
        }
        if (lane == 63) wave_sum[set][wave] = inc;
        __syncthreads();
        uint32_t before = carry;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const uint32_t ws = wave_sum[set][w];
            if (w < wave) before += ws;
            carry += ws;
        }
        uint32_t run = before + inc - sum;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t x = v.x[j];
            v.x[j] = run;
            run += x;
        }
        if (i < entries) *(Counts4 *)(c + i) = v;
    }
}

// The lanes of the wavefront whose item is valid and has the same RB-bit digit as this lane's
// (for a lane with a valid item).  One ballot per bit; a lane collects, per half of the
// wavefront, the lanes whose bit differs from its own.
template <int RB>
__device__ __forceinline__ unsigned long long lanes_with_same_digit(uint32_t d, bool valid) {
    uint32_t diff_lo = 0, diff_hi = 0;
#pragma unroll
    for (int bit = 0; bit < RB; ++bit) {
        const uint32_t mine = (uint32_t)((int32_t)(d << (31 - bit)) >> 31);      // all ones where the bit is set
        const unsigned long long bal = __ballot(mine != 0);
        diff_lo |= (uint32_t)bal ^ mine;
        diff_hi |= (uint32_t)(bal >> 32) ^ mine;
    }
    const unsigned long long live = __ballot(valid);
    return live & ~((unsigned long long)diff_hi << 32 | diff_lo);
}

// Rank of a valid lane's item among the wavefront's earlier items with its digit: the digit's
// counter (one row of counters per wavefront) plus the lane's place among the lanes of this
// round that share the digit; the last of them moves the counter on.  LDS reads and writes of
// one wavefront keep their order, so every lane has read before one writes.
template <int RB>
__device__ __forceinline__ uint32_t rank_in_wavefront(uint32_t *counters, uint32_t d, bool valid) {
    const unsigned long long same = lanes_with_same_digit<RB>(d, valid);
    const uint32_t place = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
    const uint32_t together = (uint32_t)__popcll(same);
    uint32_t before = 0;
    if (valid) {
        before = counters[d];
        if (place + 1 == together) counters[d] = before + together;
    }
    return before + place;
}

// Where the scatter kernel keeps what belongs to digit d in its LDS tables: a permutation of
// the digits that moves digits 32, 64, ... apart into different banks (the device id sits in
// the upper bits of the leading digit, so the digits of one wavefront often differ by that).
__device__ __forceinline__ uint32_t cell_of(uint32_t d) { return d ^ (d >> 5); }

// Stable scatter of one tile.  Wavefront w owns items [w*1024, (w+1)*1024) of the tile
// and takes them 64 at a time, so item order is (wavefront, round, lane).  Inside a
// round, lanes with equal digits find each other by ballots; the last of them
// advances the wavefront's counter for that digit.  The tile is then put in digit order
// in LDS and written out in runs: first the keys, then, through the same LDS buffer,
// the vertex numbers.
// Where nothing was found against a partition (found[q] == 0, the leading scatter only: see pct_bucket_check_kernel), its
// buckets are sorted with the vertex number as part of the key, and an item takes its place among equal digits by one
// returning LDS add in place of nine ballots (130 vector instructions an item): 211,000 vertices, 512 partitions, the call
// 982 -> 895 us on 16 devices, 979 -> 918 on 2; 17 partitions 99 -> 92.  Keys that repeat keep the ballots and their time.
template <typename Key, int kSortThreads, int RB, bool FIRST, bool LAST>
__global__ __launch_bounds__(kSortThreads) void pct_scatter_kernel(const Key *__restrict__ keys_in,
                                                                   const int32_t *__restrict__ vals_in,
                                                                   Key *__restrict__ keys_out,
                                                                   int32_t *__restrict__ vals_out, int32_t n,
                                                                   int32_t tiles, int shift,
                                                                   const uint32_t *__restrict__ starts, Gate gate,
                                                                   const int32_t *__restrict__ found, int32_t found_stride) {
    constexpr int kSortWaves = kSortThreads / 64, kSortTile = kSortThreads * kSortRounds, kRadix = 1 << RB;
    static_assert(kSortThreads >= kRadix, "one thread per digit when the tile's digit starts are computed");
    if (gate.closed()) return;
    extern __shared__ __align__(16) uint8_t sort_lds[];      // kSortTile keys, later kSortTile vertex numbers
    __shared__ uint32_t cnt[kSortWaves][kRadix];
    __shared__ int32_t out_base[kRadix];
    __shared__ uint32_t wave_sum[kRadix / 64];
    Key *skey = (Key *)sort_lds;
    int32_t *sval = (int32_t *)sort_lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t tile = (int32_t)(blockIdx.x % (uint32_t)tiles), q = (int32_t)(blockIdx.x / (uint32_t)tiles);
    const int64_t seg = (int64_t)q * n;
    const int64_t base = (int64_t)tile * kSortTile;
    const int32_t tile_items = (int32_t)min((int64_t)kSortTile, (int64_t)n - base);
    for (int i = tid; i < kSortWaves * kRadix; i += kSortThreads) (&cnt[0][0])[i] = 0;
    __syncthreads();

    const bool any_order = FIRST && !LAST && found != nullptr && found[(int64_t)q * found_stride] == 0;
    Key key[kSortRounds];
    int32_t val[kSortRounds];
    uint32_t loc[kSortRounds];       // rank among equal digits, then position in the sorted tile
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int32_t t = wave * (kSortRounds * 64) + r * 64 + lane;      // index inside the tile
        const bool valid = t < tile_items;
        key[r] = valid ? keys_in[seg + base + t] : (Key)0;
        val[r] = FIRST ? (int32_t)(base + t) : (valid ? vals_in[seg + base + t] : 0);
    }
    if (any_order) {
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r)
            if (wave * (kSortRounds * 64) + r * 64 + lane < tile_items)
                loc[r] = atomicAdd(&cnt[wave][cell_of(digit_of<RB>(key[r], shift))], 1u);
    } else {
#pragma unroll
        for (int r = 0; r < kSortRounds; ++r) {
            const int32_t t = wave * (kSortRounds * 64) + r * 64 + lane;
            const bool valid = t < tile_items;
            loc[r] = rank_in_wavefront<RB>(cnt[wave], cell_of(digit_of<RB>(key[r], shift)), valid);
        }
    }
    __syncthreads();
    uint32_t run = 0, inc = 0;
    if (tid < kRadix) {   // thread d: wavefront bases, then the tile's digit starts
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
            const uint32_t c = cnt[w][cell_of(tid)];
            cnt[w][cell_of(tid)] = run;
            run += c;
        }
        inc = run;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t up = __shfl_up(inc, off);
            if (lane >= off) inc += up;
        }
        if (lane == 63) wave_sum[wave] = inc;
    }
    __syncthreads();
    if (tid < kRadix) {
        uint32_t before = 0;
        for (int w = 0; w < wave; ++w) before += wave_sum[w];
        const uint32_t start = before + inc - run;
        out_base[cell_of(tid)] = (int32_t)starts[((int64_t)q * kRadix + tid) * tiles + tile] - (int32_t)start;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) cnt[w][cell_of(tid)] += start;   // now positions in the sorted tile
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int32_t t = wave * (kSortRounds * 64) + r * 64 + lane;
        if (t < tile_items) {
            const uint32_t d = cell_of(digit_of<RB>(key[r], shift));
            loc[r] = cnt[wave][d] + loc[r];
            skey[loc[r]] = key[r];
        }
    }
    __syncthreads();
    int32_t dst[kSortRounds];        // where item i of the sorted tile goes in the partition's output
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int32_t i = r * kSortThreads + tid;
        dst[r] = 0;
        if (i < tile_items) {
            const Key kk = skey[i];
            dst[r] = out_base[cell_of(digit_of<RB>(kk, shift))] + i;
            if (!LAST) keys_out[seg + dst[r]] = kk;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int32_t t = wave * (kSortRounds * 64) + r * 64 + lane;
        if (t < tile_items) sval[loc[r]] = val[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int32_t i = r * kSortThreads + tid;
        if (i < tile_items) vals_out[seg + dst[r]] = sval[i];
    }
}

// ---------------------------------------------------------------- buckets of the leading digit

// a bucket is sorted by a workgroup of 256 or 512 threads, 16 items per thread at most
constexpr int kBucketCapSmall = 256 * kSortRounds, kBucketCapLarge = 512 * kSortRounds;     // 4,096 / 8,192 items

// After the scan of the leading digit's counts, bucket d of partition q starts where tile 0's
// run of digit d starts.  flag |= 1 if some bucket holds more than `cap` items.
// found[q]: kLeftOver where some bucket holds more than `bins_cap` items, which the bins leave to the ranking by digits;
// kCrowded where 512 * kEach of the partition's keys, spread over its vertices, fall into common bins of
// pct_bucket_bins_kernel (keys without their low `shift` bits) as they would with more than kBinAverage items in an average
// item's bin: then ranking by digits is the faster way, and the bins would be tried in vain.  Few partitions are sampled
// more finely, because the call then takes as long as the one that was misjudged (a million vertices on 16 devices in 66
// items a bin, of 512 samples one partition in 14 passed for spread; 8 partitions: 231 us, 203 with 2,048).
constexpr int kBinMost = 96, kBinAverage = 32, kFineSamples = 128;
constexpr int32_t kCrowded = 1, kLeftOver = 2;
template <int kEach>
__global__ __launch_bounds__(kBuckets) void pct_bucket_check_kernel(const uint32_t *__restrict__ starts,
                                                                    const uint32_t *__restrict__ keys, int32_t n,
                                                                    int32_t tiles, int32_t cap, int32_t bins_cap, int shift,
                                                                    uint32_t *flag, int32_t *found, int32_t found_stride) {
    constexpr int kTableBits = kEach > 1 ? 13 : 12, kSamples = kBuckets * kEach;
    __shared__ uint32_t table[1 << kTableBits], wave_pairs[kBuckets / 64];
    const int32_t q = blockIdx.x, d = threadIdx.x;
    const uint32_t lo = starts[((int64_t)q * kBuckets + d) * tiles];
    const uint32_t hi = d + 1 < kBuckets ? starts[((int64_t)q * kBuckets + d + 1) * tiles] : (uint32_t)n;
    uint32_t x[kEach];
#pragma unroll
    for (int j = 0; j < kEach; ++j) x[j] = keys[(int64_t)q * n + (int64_t)(j * kBuckets + d) * n / kSamples] >> shift;
    for (int i = d; i < 1 << kTableBits; i += kBuckets) table[i] = 0xffffffffu;
    // (one atomic per partition at most, none once the flag is up: they queue up on the one word)
    const int any = __syncthreads_or(hi - lo > (uint32_t)cap);
    const int left_over = __syncthreads_or(hi - lo > (uint32_t)bins_cap);
    if (any && threadIdx.x == 0 && *(volatile const uint32_t *)flag == 0) atomicOr(flag, 1u);
    uint32_t before[kEach];
#pragma unroll
    for (int j = 0; j < kEach; ++j) before[j] = atomicExch(&table[x[j] * 0x9e3779b1u >> (32 - kTableBits)], x[j]);
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kEach; ++j) mine += (uint32_t)__popcll(__ballot(before[j] == x[j]));
    if (d % 64 == 0) wave_pairs[d / 64] = mine;
    __syncthreads();
    int pairs = 0;
#pragma unroll
    for (int w = 0; w < kBuckets / 64; ++w) pairs += (int)wave_pairs[w];
    if (d == 0)
        found[(int64_t)q * found_stride] =
            ((int64_t)pairs * n > (int64_t)kSamples * kSamples / 2 * kBinAverage ? kCrowded : 0) | (left_over ? kLeftOver : 0);
}

// Inclusive sum over the lanes of a wavefront: inside rows of 16 by shifts, then a row's last lane
// handed to the rows behind it.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);     // row_shr 1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);     // row_shr 2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);     // row_shr 4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);     // row_shr 8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);    // row_bcast 15 into rows 1, 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);    // row_bcast 31 into rows 2, 3
    return x;
}

// Items whose key bits spread them, sorted without ranking digit by digit: they are dealt to eight bins per
// thread, in any order, by one returning LDS add each; then every item compares itself with the others of
// its bin, the key's bits below the bin's and the vertex number as one word, which gives its place in the list.
// An item costs some 50 instructions plus five for each other item that the fullest bin of its wavefront holds,
// instead of the 130 per digit that ranking by ballots takes.  (val_bits: of a vertex number; both parts of the word
// fit 32 bits.)  False, with nothing written, where a bin holds more than kBinMost items or (WHOLE: the items are a
// partition's vertices in their order, their keys loaded as sort_bucket wants them) one item per thread, out of all parts
// of the list, shares its bin as it would with more than kBinAverage items in an average item's bin: keys that repeat, or
// that differ in their low bits only.
constexpr int bin_bits(int threads) { return threads == 128 ? 10 : threads == 256 ? 11 : threads == 512 ? 12 : 13; }
// 211,000 vertices, 512 partitions, 16 devices, ranked and by bins: 1,325 -> 315 us, bound by vector issue (83 %; the LDS pipe
// is busy 64 % of the time, half of that with bank conflicts).  Whole partitions, the call:
// 19,000 vertices, 512 partitions 154 -> 83 us; 5,000 vertices, 3,000 partitions 186 -> 96.  Keys that repeat are found out
// by the sample and pay for it: whole partitions 2 - 3 us, 3 to 8 % of the call; longer ones 0 - 2 us in one launch
// (bins_and_ranking_in_one), in two 3 to 8 % of a call of up to 128 partitions and nothing beyond; most where buckets want
// 512 threads (480,000 vertices, 9 devices, 300 values of b: 8 partitions 120 -> 136 us, 32 303 -> 324, 64 539 -> 509).
template <int kThreads, int kRounds, bool WHOLE>
__device__ __forceinline__ bool sort_by_bins(const uint32_t *__restrict__ keys_in, const int32_t *__restrict__ vals_in,
                                             int32_t *__restrict__ vals_out, int32_t items, int bits, int val_bits,
                                             uint32_t *sorted, uint32_t *bins, uint32_t *wave_sum,
                                             uint32_t (&key)[kRounds]) {
    constexpr int kWaves = kThreads / 64;
    static_assert(kThreads * 8 == 1 << bin_bits(kThreads), "eight bins per thread");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int shift = max(0, bits - bin_bits(kThreads));
    const uint32_t below = (1u << shift) - 1, bin_of = (1u << (bits - shift)) - 1;
    const int nr = WHOLE ? (items + kThreads - 1) / kThreads : kRounds;
    auto at = [&](int r) -> int32_t { return WHOLE ? wave * (nr * 64) + r * 64 + lane : r * kThreads + tid; };
    auto valid = [&](int r) { return (!WHOLE || r < nr) && at(r) < items; };
    uint32_t rank[kRounds], bin[kRounds];
    int32_t val[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        if (WHOLE) {
            val[r] = at(r);
        } else if (valid(r)) {
            key[r] = keys_in[at(r)];
            val[r] = vals_in[at(r)];
        }
    }
    Counts4 *mine = (Counts4 *)(bins + tid * 8);
    mine[0] = mine[1] = Counts4{};
    __syncthreads();
    int early = -1;                                       // the round whose item has been dealt already
    if (WHOLE && items > kThreads) {
        // (a thread of the last wavefronts may have no such item)
        const int r0 = tid % nr;
        uint32_t sample = 0, got = 0;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) sample = r == r0 ? key[r] : sample;
        if (at(r0) < items) {
            got = atomicAdd(&bins[sample >> shift & bin_of], 1u);
            early = r0;
        }
#pragma unroll
        for (int r = 0; r < kRounds; ++r) rank[r] = got;
        // pairs in one bin: the sum of the places
        const uint32_t pairs = wave_inclusive_sum(got), some = (uint32_t)__popcll(__ballot(early >= 0));
        if (lane == 63) {
            wave_sum[wave] = pairs;
            wave_sum[kWaves + wave] = some;
        }
        __syncthreads();
        uint64_t all_pairs = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            all_pairs += wave_sum[w];
            all += wave_sum[kWaves + w];
        }
        if (all_pairs * (uint32_t)items > all * all / 2 * kBinAverage) return false;
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (valid(r) && r != early) rank[r] = atomicAdd(&bins[key[r] >> shift & bin_of], 1u);
    __syncthreads();
    Counts4 c[2] = {mine[0], mine[1]};
    uint32_t most = 0, sum = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        most = max(most, c[j / 4].x[j % 4]);
        sum += c[j / 4].x[j % 4];
    }
    const uint32_t inc = wave_inclusive_sum(sum);
    const bool crowded = __ballot(most > (uint32_t)kBinMost) != 0;
    if (lane == 63) wave_sum[wave] = crowded ? inc | 1u << 31 : inc;
    __syncthreads();
    uint32_t run = inc - sum, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        run += w < wave ? wave_sum[w] : 0u;
        all |= wave_sum[w];
    }
    if (all >> 31) {
        __syncthreads();                                  // (the caller goes on with the same LDS)
        return false;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t x = c[j / 4].x[j % 4];
        c[j / 4].x[j % 4] = run | x << 16;                // start and length
        run += x;
    }
    mine[0] = c[0];
    mine[1] = c[1];
    __syncthreads();
    auto word_of = [&](uint32_t k, int32_t v) { return (k & below) << val_bits | (uint32_t)v; };
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (valid(r)) {
            bin[r] = bins[key[r] >> shift & bin_of];
            sorted[(bin[r] & 0xffffu) + rank[r]] = word_of(key[r], val[r]);
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (valid(r)) {
            const uint32_t first = bin[r] & 0xffffu, end = first + (bin[r] >> 16);
            const uint32_t x = word_of(key[r], val[r]);
            uint32_t place = first, j = first;
            if (end - first > 1) {
                for (; j + 4 <= end; j += 4) {
                    const uint32_t a = sorted[j], b = sorted[j + 1], c = sorted[j + 2], d = sorted[j + 3];
                    place += (a < x ? 1u : 0u) + (b < x ? 1u : 0u) + (c < x ? 1u : 0u) + (d < x ? 1u : 0u);
                }
                for (; j < end; ++j) place += sorted[j] < x ? 1u : 0u;
            }
            rank[r] = place;
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (valid(r)) sorted[rank[r]] = (uint32_t)val[r];
    __syncthreads();
    for (int32_t t = tid; t < items; t += kThreads) vals_out[t] = (int32_t)sorted[t];
    return true;
}

// What the ranking needs of a bucket whose items the scatter dealt by LDS adds, 64 vertices an add in whatever order it takes its
// lanes (a bin that is crowded after all, in a partition that nothing was found against).  They are neighbours here, in runs of
// vertex numbers that differ in their low six bits only, and mostly in order, which is looked at; if not, the first thread of a
// run puts it in order.  (Sorting by the vertex numbers' digits instead took three passes more, and spilled registers in all
// buckets: 142,000 vertices in 53 levels, 4 devices, 8 partitions, whose last level's keys repeat, 82 us a call before there was
// the scatter by adds, 146 and more with those passes, 78 with this.  A call, because inlined it cost
// registers: 66 instead of 60 in the bins of 128 threads, the call of 211,000 vertices and 512 partitions 888 -> 932 us.)
template <int kThreads>
__device__ __noinline__ void order_runs(uint32_t *keys, int32_t *vals, int32_t items, int tid) {
    bool apart = false;
    for (int32_t t = tid + 1; t < items; t += kThreads) apart |= vals[t - 1] > vals[t];
    if (!__syncthreads_or(apart)) return;
    for (int32_t t = tid; t < items; t += kThreads) {
        const int32_t run = vals[t] >> 6;
        if (t > 0 && vals[t - 1] >> 6 == run) continue;
        for (int32_t i = t + 1; i < items && vals[i] >> 6 == run; ++i) {
            const int32_t v = vals[i];
            const uint32_t k = keys[i];
            int32_t at = i;
            for (; at > t && vals[at - 1] > v; --at) {
                vals[at] = vals[at - 1];
                keys[at] = keys[at - 1];
            }
            vals[at] = v;
            keys[at] = k;
        }
    }
    __syncthreads();
}

// The buckets of the leading digit, by bins, `each` neighbours per workgroup.  left[i] = 1 for those that
// pct_bucket_sort_kernel has to sort: of more than eight items per thread, of a partition whose keys the sample of
// pct_bucket_check_kernel found in common bins, or with a crowded bin after all.
constexpr int kBinRounds = 8;
template <int kThreads>
__global__ __launch_bounds__(kThreads) void pct_bucket_bins_kernel(const uint32_t *__restrict__ keys_in,
                                                                   const int32_t *__restrict__ vals_in,
                                                                   int32_t *__restrict__ vals_out, int32_t n, int32_t each,
                                                                   int32_t tiles, int bits, int val_bits,
                                                                   const uint32_t *__restrict__ starts, Gate gate,
                                                                   const int32_t *__restrict__ found, int32_t found_stride,
                                                                   uint32_t *left) {
    __shared__ uint32_t sorted[kThreads * kBinRounds];
    __shared__ __align__(16) uint32_t bins[kThreads * 8];
    __shared__ uint32_t wave_sum[kThreads / 64];
    uint32_t key[kBinRounds];
    // (turned by one neighbourhood from partition to partition: workgroups go round the eight XCDs, and the digits in use
    // are the same in all partitions; of 9 devices, 19 in every 32: 884 us one by one, so 568)
    const uint32_t per = (uint32_t)(kBuckets / each), q = blockIdx.x / per, d0 = (blockIdx.x + q) % per * (uint32_t)each;
    const int lane = threadIdx.x & 63;
    uint32_t bound = (uint32_t)n;                         // where bucket d0 + lane starts
    if (lane <= each && d0 + lane < kBuckets) bound = starts[((int64_t)q * kBuckets + d0 + lane) * tiles];
    if (gate.closed()) return;
    left += (int64_t)q * kBuckets + d0;
    if ((found[(int64_t)q * found_stride] & kCrowded) != 0) {
        const uint32_t next = __shfl_down(bound, 1);
        if ((int)threadIdx.x < each) left[threadIdx.x] = next != bound ? 1u : 0u;
        return;
    }
    for (int i = 0; i < each; ++i) {
        const uint32_t lo = __builtin_amdgcn_readlane(bound, i), hi = __builtin_amdgcn_readlane(bound, i + 1);
        const int32_t items = (int32_t)(hi - lo);
        const int64_t at = (int64_t)q * n + lo;
        bool done = items <= 0;
        if (!done && items <= kThreads * kBinRounds)
            done = sort_by_bins<kThreads, kBinRounds, false>(keys_in + at, vals_in + at, vals_out + at, items, bits,
                                                                   val_bits, sorted, bins, wave_sum, key);
        if (threadIdx.x == 0) left[i] = done ? 0u : 1u;
    }
}

// One bucket, sorted on the low `bits` bits inside LDS: stable passes of 8 bits, each ranking
// the items as the scatter kernel does (wavefront w owns items [w*1024, (w+1)*1024) of the
// bucket in (round, lane) order) and moving keys and vertex numbers through one LDS buffer;
// the vertex numbers of the last pass go straight out.
// WHOLE: the "bucket" is a whole partition (at most kBucketThreads * kRounds vertices), its keys
// in vertex order and already in `key`, sorted on all `bits` key bits: short partitions need no pass over
// HBM at all.
// slot: kBucketThreads * kRounds words; cnt: 256 per wavefront
template <int kBucketThreads, int kRounds, bool WHOLE>
__device__ __forceinline__ void sort_bucket(const uint32_t *__restrict__ keys_in, const int32_t *__restrict__ vals_in,
                                            int32_t *__restrict__ vals_out, int32_t items, int bits, uint32_t *slot,
                                            uint32_t (*cnt)[256], int tid, uint32_t (&key)[kRounds]) {
    constexpr int kWaves = kBucketThreads / 64, kRadix = 256;
    __shared__ uint32_t wave_sum[kRadix / 64];
    const int lane = tid & 63, wave = tid >> 6;
    // rounds this bucket needs (the same for every wavefront: wavefront w owns items
    // [w * nr * 64, (w + 1) * nr * 64) of the bucket)
    const int nr = (items + kBucketThreads - 1) / kBucketThreads;

    uint32_t loc[kRounds];
    int32_t val[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int32_t t = wave * (nr * 64) + r * 64 + lane;
        const bool valid = r < nr && t < items;
        if (!WHOLE) key[r] = valid ? keys_in[t] : 0u;
        val[r] = WHOLE ? t : (valid ? vals_in[t] : 0);
    }
    for (int shift = 0; shift < bits; shift += 8) {
        const bool last = shift + 8 >= bits;
        for (int i = tid; i < kWaves * kRadix; i += kBucketThreads) (&cnt[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            if (r >= nr) continue;           // (uniform)
            const int32_t t = wave * (nr * 64) + r * 64 + lane;
            const bool valid = t < items;
            loc[r] = rank_in_wavefront<8>(cnt[wave], digit_of<8>(key[r], shift), valid);
        }
        __syncthreads();
        // thread dg: the digit's items per wavefront, the bucket's digit starts, then every
        // wavefront's first position for the digit
        uint32_t per_wave[kWaves], run = 0, inc = 0;
        if (tid < kRadix) {
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                per_wave[w] = cnt[w][tid];
                run += per_wave[w];
            }
            inc = run;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t up = __shfl_up(inc, off);
                if (lane >= off) inc += up;
            }
            if (lane == 63) wave_sum[wave] = inc;
        }
        __syncthreads();
        if (tid < kRadix) {
            uint32_t first = inc - run;
            for (int w = 0; w < wave; ++w) first += wave_sum[w];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                cnt[w][tid] = first;
                first += per_wave[w];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int32_t t = wave * (nr * 64) + r * 64 + lane;
            if (r < nr && t < items) {
                const uint32_t dg = digit_of<8>(key[r], shift);
                loc[r] = cnt[wave][dg] + loc[r];
                if (!last) slot[loc[r]] = key[r];
            }
        }
        if (!last) {          // the keys come back in sorted order, then the vertex numbers the same way
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int32_t t = wave * (nr * 64) + r * 64 + lane;
                if (r < nr && t < items) key[r] = slot[t];
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int32_t t = wave * (nr * 64) + r * 64 + lane;
            if (r < nr && t < items) slot[loc[r]] = (uint32_t)val[r];
        }
        __syncthreads();
        if (last) {
            for (int32_t i = tid; i < items; i += kBucketThreads) vals_out[i] = (int32_t)slot[i];
        } else {
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int32_t t = wave * (nr * 64) + r * 64 + lane;
                if (r < nr && t < items) val[r] = (int32_t)slot[t];
            }
            __syncthreads();
        }
    }
}

// A whole partition per workgroup: by bins (BINS: the words fit 32 bits), else by digits.  (80 registers are six
// wavefronts a SIMD: with 89 a unit had two workgroups of 512 threads instead of three.)
template <int kThreads, int kRounds, bool BINS>
__global__ __launch_bounds__(kThreads, kThreads == 1024 ? 4 : 6) void pct_whole_sort_kernel(const uint32_t *__restrict__ keys_in,
                                                                  int32_t *__restrict__ vals_out, int32_t n, int bits,
                                                                  int val_bits) {
    extern __shared__ __align__(16) uint32_t slot[];
    __shared__ __align__(16) uint32_t counters[kThreads * (BINS ? 8 : 4)];
    __shared__ uint32_t wave_sum[2 * (kThreads / 64)];
    const int64_t at = (int64_t)blockIdx.x * n;
    const int nr = (n + kThreads - 1) / kThreads;
    uint32_t key[kRounds];
    const uint32_t *mine = keys_in + at;
    int tid = threadIdx.x;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {                   // (as sort_bucket deals them out)
        const int32_t t = (threadIdx.x >> 6) * (nr * 64) + r * 64 + (threadIdx.x & 63);
        key[r] = r < nr && t < n ? mine[t] : 0u;
    }
    if constexpr (BINS) {
        if (sort_by_bins<kThreads, kRounds, true>(nullptr, nullptr, vals_out + at, n, bits, val_bits, slot, counters,
                                                   wave_sum, key))
            return;
        if (kThreads == 512) {   // (again: kept through the bins they would cost spills, or a workgroup per compute unit)
            asm("" : "+v"(tid), "+s"(mine));
            __builtin_assume(tid >= 0 && tid < kThreads);
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int32_t t = (tid >> 6) * (nr * 64) + r * 64 + (tid & 63);
                key[r] = r < nr && t < n ? mine[t] : 0u;
            }
        }
    }
    sort_bucket<kThreads, kRounds, true>(nullptr, nullptr, vals_out + at, n, bits, slot, (uint32_t (*)[256])counters, tid,
                                         key);
}

// Both in one launch, a bucket per workgroup, for few partitions: their calls are a row of launches of a few microseconds,
// and a second one for what the bins leave would cost them as much as the bins save.  Up to 24 partitions, up to 48
// where the bins want the ranking's workgroup of 256 anyway (smaller ones want more of them on a compute unit than the
// ranking has registers and LDS for), and up to 16 where they want the larger one, in which the ranking is slower.  Ranked as
// before there were bins / in two launches / in one, us; spread keys, then 300 values of b:
//   211,000 vertices,  3 devices, 17, 48, 64 partitions: 104 / 96 / 90, 188 / 156 / 150, 246 / 200 / 198;
//                                                        104 / 115 / 105, 189 / 204 / 191, 246 / 258 / 250
//                      9 devices: 122 / 98 / 92, 236 / 154 / 155, 310 / 194 / 205; 124 / 134 / 125, 240 / 252 / 240, 315 / 296 / 314
//                     16 devices, 17, 24, 32: 139 / 100 / 97, 175 / 116 / 115, 216 / 126 / 138;
//                                             139 / 150 / 143, 175 / 188 / 180, 216 / 216 / 223
//   900,000 vertices,  3 devices, 8 (workgroups of 512): 142 / 133 / 129; 206 / 213 / 210
inline bool bins_and_ranking_in_one(int32_t P, int for_bins, int threads) {
    return P <= (threads == 512 ? 16 : for_bins > 128 ? 48 : 24);
}
template <int kThreads>
__global__ __launch_bounds__(kThreads, 6) void pct_bucket_kernel(uint32_t *keys_in, int32_t *vals_in,
                                                              int32_t *__restrict__ vals_out, int32_t n, int32_t tiles, int bits,
                                                              int val_bits, const uint32_t *__restrict__ starts, Gate gate,
                                                              const int32_t *__restrict__ found, int32_t found_stride) {
    // sorted words and bins, or the ranking's slots
    __shared__ __align__(16) uint32_t slot[kThreads * kSortRounds], counters[kThreads / 64][256], wave_sum[kThreads / 64];
    static_assert(kSortRounds == kBinRounds + 8, "eight bins per thread behind the sorted words");
    const uint32_t q = blockIdx.x / kBuckets, d = (blockIdx.x + q) % kBuckets;    // (turned, as in pct_bucket_bins_kernel)
    const uint32_t *at_bucket = starts + ((int64_t)q * kBuckets + d) * tiles;
    const uint32_t lo = at_bucket[0], hi = d + 1 == kBuckets ? (uint32_t)n : at_bucket[tiles];
    const int32_t what = found[(int64_t)q * found_stride];
    const bool bins = (what & kCrowded) == 0;
    if (gate.closed()) return;
    uint32_t few[kBinRounds], key[kSortRounds];
    const int32_t items = (int32_t)(hi - lo);
    if (items <= 0 || items > kThreads * kSortRounds) return;                      // (more: the flag is up)
    const int64_t at = (int64_t)q * n + lo;
    if (bins && items <= kThreads * kBinRounds &&
        sort_by_bins<kThreads, kBinRounds, false>(keys_in + at, vals_in + at, vals_out + at, items, bits, val_bits, slot,
                                                   slot + kThreads * kBinRounds, wave_sum, few))
        return;
    if (what == 0) order_runs<kThreads>(keys_in + at, vals_in + at, items, threadIdx.x);
    sort_bucket<kThreads, kSortRounds, false>(keys_in + at, vals_in + at, vals_out + at, items, bits, slot, counters,
                                              threadIdx.x, key);
}

// The buckets that pct_bucket_bins_kernel left, out of the `each` that a workgroup looks at (left_over_bucket).
// (Six wavefronts a SIMD, and the thread's number new in every round: else the loop keeps every address that follows from
// it, 110 registers, or spills some; so 77 and no scratch.)
template <int kThreads>
__global__ __launch_bounds__(kThreads, 6) void pct_bucket_sort_kernel(uint32_t *keys_in, int32_t *vals_in,
                                                                   int32_t *__restrict__ vals_out, int32_t n, int32_t each,
                                                                   int32_t tiles, int bits,
                                                                   const uint32_t *__restrict__ starts, Gate gate,
                                                                   const int32_t *__restrict__ found, int32_t found_stride,
                                                                   const uint32_t *__restrict__ left) {
    __shared__ uint32_t slot[kThreads * kSortRounds], counters[kThreads / 64][256];
    if (gate.closed()) return;
    const uint32_t q = blockIdx.x / (uint32_t)(kBuckets / each);
    const bool any_order = found[(int64_t)q * found_stride] == 0;
    uint32_t lo = 0, hi = 0;
    if ((int)(threadIdx.x & 63) < each) {
        const uint32_t d = left_over_bucket<kBuckets>(blockIdx.x, threadIdx.x & 63, each);
        const int64_t i = (int64_t)q * kBuckets + d;
        if (left[i] != 0) {
            lo = starts[i * tiles];
            hi = d + 1 == kBuckets ? (uint32_t)n : starts[(i + 1) * tiles];
        }
    }
    if (hi - lo > kThreads * kSortRounds) hi = lo;        // (more: the flag is up)
    unsigned long long some = __ballot(hi > lo);          // the same in every wavefront
    for (; some != 0; some &= some - 1) {
        int tid = threadIdx.x;
        asm("" : "+v"(tid));
        __builtin_assume(tid >= 0 && tid < kThreads);
        const int which = __ffsll((long long)some) - 1;
        const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)lo, which);
        const int32_t items = (int32_t)((uint32_t)__builtin_amdgcn_readlane((int)hi, which) - first);
        const int64_t at = (int64_t)q * n + first;
        uint32_t key[kSortRounds];
        if (any_order) order_runs<kThreads>(keys_in + at, vals_in + at, items, tid);
        sort_bucket<kThreads, kSortRounds, false>(keys_in + at, vals_in + at, vals_out + at, items, bits, slot, counters, tid,
                                                  key);
        __syncthreads();
    }
}

// seg[q][d] = first position of the sorted list whose vertex sits on a device >= d
__global__ void pct_segments_kernel(const int32_t *__restrict__ order, const uint8_t *__restrict__ assign,
                                    int64_t a_stride_p, int64_t a_stride_v, int32_t n, int32_t P, int32_t k,
                                    int32_t *__restrict__ seg) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)P * (k + 1)) return;
    const int32_t q = (int32_t)(i / (k + 1)), d = (int32_t)(i % (k + 1));
    const int32_t *ord = order + (int64_t)q * n;
    int32_t lo = 0, hi = n;
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        const int32_t dev = min((int32_t)assign[q * a_stride_p + (int64_t)ord[mid] * a_stride_v], k - 1);
        if (dev < d) lo = mid + 1; else hi = mid;
    }
    seg[i] = lo;
}

// The launches of one digit pass of RB bits starting at bit `shift`: counts, scan, scatter.
template <typename Key, int THREADS, int RB>
struct DigitPass {
    static constexpr int kTile = THREADS * kSortRounds;
    const PctOrderLaunch &s;
    hipStream_t st;
    int shift;
    Gate gate;
    int32_t tiles() const { return (s.n + kTile - 1) / kTile; }
    dim3 grid() const { return dim3((unsigned)((int64_t)tiles() * s.P)); }     // one workgroup per (partition, tile)
    void count(const Key *kin) const {
        hipLaunchKernelGGL((pct_count_kernel<Key, THREADS, RB>), grid(), dim3(THREADS), 0, st, kin, s.n, tiles(), shift,
                           s.counts, gate);
    }
    void scan() const {
        hipLaunchKernelGGL(pct_scan_kernel, dim3((unsigned)s.P), dim3(1024), 0, st, s.counts, (1 << RB) * tiles(), gate);
    }
    int scatter(bool first, bool last, const Key *kin, Key *kout, const int32_t *vin, int32_t *vout,
                const int32_t *found = nullptr) const {
        const size_t lds = (size_t)kTile * sizeof(Key);
#define CP_SCATTER(F, L)                                                                                   \
    do {                                                                                                   \
        auto kern = pct_scatter_kernel<Key, THREADS, RB, F, L>;                                            \
        /* more than 64 KB of dynamic LDS has to be asked for */                                           \
        if (lds > 64 * 1024 && hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                                   (int)lds) != hipSuccess)                                \
            return CP_ERR_HIP;                                                                             \
        hipLaunchKernelGGL(kern, grid(), dim3(THREADS), lds, st, kin, vin, kout, vout, s.n, tiles(), shift, s.counts, \
                           gate, found, s.k + 1);                                                                          \
    } while (0)
        if (first && last) CP_SCATTER(true, true);
        else if (first) CP_SCATTER(true, false);
        else if (last) CP_SCATTER(false, true);
        else CP_SCATTER(false, false);
#undef CP_SCATTER
        return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_HIP;
    }
};

template <typename Key, int THREADS, int RB>
int run_pass(const PctOrderLaunch &s, hipStream_t st, int shift, bool first, bool last, const Key *kin, Key *kout,
             const int32_t *vin, int32_t *vout, Gate gate) {
    const DigitPass<Key, THREADS, RB> pass{s, st, shift, gate};
    pass.count(kin);
    pass.scan();
    return pass.scatter(first, last, kin, kout, vin, vout);
}

// WIDE: 9-bit digits may be used (long tiles of 32-bit keys: the counters of a 64-bit
// tile's 512 digits would not fit LDS beside the tile).
template <typename Key, int THREADS, bool WIDE>
int run_sort(const PctOrderLaunch &s, hipStream_t st, Gate gate = Gate{nullptr, 0}) {
    Key *ka = (Key *)s.keys_a, *kb = (Key *)s.keys_b;
    const int passes = pct_passes(s.key_bits, WIDE);
    // 8 bits per pass; where that leaves bits over, the leading passes take 9
    const int wide_passes = std::max(0, s.key_bits - 8 * passes);
    int shift = 0;
    // vertex lists alternate between the scratch list and the output so that the last
    // pass writes the output
    for (int p = 0; p < passes; ++p) {
        const bool first = p == 0, last = p == passes - 1;
        const Key *kin = (p & 1) ? kb : ka;
        Key *kout = (p & 1) ? ka : kb;
        const bool to_out = ((passes - 1 - p) & 1) == 0;
        int32_t *vout = to_out ? s.order_out : s.vals_tmp;
        const int32_t *vin = to_out ? s.vals_tmp : s.order_out;
        int rc;
        if (WIDE && p < wide_passes) {
            rc = run_pass<Key, THREADS, WIDE ? 9 : 8>(s, st, shift, first, last, kin, kout, vin, vout, gate);
            shift += 9;
        } else {
            rc = run_pass<Key, THREADS, 8>(s, st, shift, first, last, kin, kout, vin, vout, gate);
            shift += 8;
        }
        if (rc) return rc;
    }
    return CP_OK;
}

// The key kernels, for all four (tick, key) widths.
void launch_keys(const PctOrderLaunch &s, const KeyArgs &a, hipStream_t st) {
#define CP_KEYS(KERNEL, GRID)                                                                         \
    do {                                                                                              \
        if (s.key_bytes == 4) {                                                                       \
            if (s.tick_bytes == 4) hipLaunchKernelGGL((KERNEL<int32_t, uint32_t>), GRID, dim3(256), 0, st, a); \
            else hipLaunchKernelGGL((KERNEL<int64_t, uint32_t>), GRID, dim3(256), 0, st, a);          \
        } else {                                                                                      \
            if (s.tick_bytes == 4) hipLaunchKernelGGL((KERNEL<int32_t, uint64_t>), GRID, dim3(256), 0, st, a); \
            else hipLaunchKernelGGL((KERNEL<int64_t, uint64_t>), GRID, dim3(256), 0, st, a);          \
        }                                                                                             \
    } while (0)
    if (s.b_by_partition) {
        const dim3 kgrid((unsigned)((s.n + 255) / 256), (unsigned)std::min(s.P, 65535));
        CP_KEYS(pct_keys_rows_kernel, kgrid);
    } else {
        const dim3 kgrid((unsigned)((s.n + 63) / 64), (unsigned)((s.P + 63) / 64));
        CP_KEYS(pct_keys_kernel, kgrid);
    }
#undef CP_KEYS
}

// The leading digit's counts, the bucket check on their scan, and both continuations: the
// leading digit's scatter and the buckets sorted inside LDS (flag 0), or the ordinary passes
// from the untouched keys (flag 1).  With rows of b per partition one kernel writes the keys
// and counts their leading digit.
int run_bucket_sort(const PctOrderLaunch &s, KeyArgs a, hipStream_t st) {
    constexpr int kTile = kLeadThreads * kSortRounds;
    const int32_t tiles = (s.n + kTile - 1) / kTile;
    uint32_t *flag = s.counts + (size_t)s.P * kMaxRadix * (size_t)tiles;     // behind the counts
    a.flag = flag;
    const int rem = s.key_bits - kBucketBits;
    if (s.b_by_partition) {
        const dim3 grid((unsigned)((int64_t)tiles * s.P)), block(kLeadThreads);
        const bool vec = s.n % 4 == 0 && s.a_stride_v == 1 && s.a_stride_p % 4 == 0 && (uintptr_t)s.assign % 4 == 0 &&
                         (uintptr_t)s.b % 16 == 0 && (uintptr_t)s.keys_a % 16 == 0;
        if (s.tick_bytes == 4) {
            if (vec) hipLaunchKernelGGL((pct_keys_count_kernel<int32_t, true>), grid, block, 0, st, a, tiles, rem, s.counts);
            else hipLaunchKernelGGL((pct_keys_count_kernel<int32_t, false>), grid, block, 0, st, a, tiles, rem, s.counts);
        } else {
            if (vec) hipLaunchKernelGGL((pct_keys_count_kernel<int64_t, true>), grid, block, 0, st, a, tiles, rem, s.counts);
            else hipLaunchKernelGGL((pct_keys_count_kernel<int64_t, false>), grid, block, 0, st, a, tiles, rem, s.counts);
        }
    } else {
        launch_keys(s, a, st);
    }
    const DigitPass<uint32_t, kLeadThreads, kBucketBits> lead{s, st, rem, Gate{nullptr, 0u}};
    if (!s.b_by_partition) lead.count((const uint32_t *)s.keys_a);
    lead.scan();
    // the smaller workgroup (more of them per compute unit) where buckets of twice the average size fit it
    const bool small = 2 * ((int64_t)s.n / kBuckets + 1) <= kBucketCapSmall;
    const int for_bins = bucket_threads(s.n, s.k, s.b_bits, rem, s.max_b);
    // (a bucket that the bins do not hold after all is ranked by the same workgroup: an eighth to spare will do)
    const int64_t average = bucket_average(s.n, s.k, s.b_bits, rem, s.max_b);
    const int in_one = small && average * 8 / 7 <= 256 * kBinRounds ? 256 : 512;
    const bool both = bins_and_ranking_in_one(s.P, for_bins, in_one);
    const int threads = both ? in_one : for_bins;
    const int shift = std::max(0, rem - bin_bits(threads));
    // (noted where the partition's list bounds will stand)
    int32_t *found = s.seg_out;
    auto check = s.P <= kFineSamples ? pct_bucket_check_kernel<4> : pct_bucket_check_kernel<1>;
    hipLaunchKernelGGL(check, dim3((unsigned)s.P), dim3(kBuckets), 0, st, s.counts, (const uint32_t *)s.keys_a, s.n, tiles,
                       small ? kBucketCapSmall : kBucketCapLarge, threads * kBinRounds, shift, flag, found, s.k + 1);
    if (hipGetLastError() != hipSuccess) return CP_ERR_HIP;
    const Gate fit{flag, 0u};
    const DigitPass<uint32_t, kLeadThreads, kBucketBits> lead_if_fit{s, st, rem, fit};
    const int rc = lead_if_fit.scatter(/*first=*/true, /*last=*/false, (const uint32_t *)s.keys_a, (uint32_t *)s.keys_b,
                                       nullptr, s.vals_tmp, found);
    if (rc) return rc;
    // (what the bins leave is noted in keys_a, which nothing reads any more on this way)
    uint32_t *left = (uint32_t *)s.keys_a;
    uint32_t *keys = (uint32_t *)s.keys_b;
    const uint32_t *starts = s.counts;
    int32_t *vals = s.vals_tmp;
    const int32_t all = s.P * kBuckets;
    const int val_bits = 32 - __builtin_clz((unsigned)s.n - 1);
    // (keys of 32 bits: shift is 13, 12 or 11 at most for up to 2^18, 2^19 or 2^20 vertices, less for larger workgroups)
    if (shift + val_bits > 32) return CP_ERR_ARG;
    const int32_t dealt = bins_each(all);
    if (both) {
#define CP_BOTH(T)                                                                                                    \
    hipLaunchKernelGGL(pct_bucket_kernel<T>, dim3((unsigned)all), dim3(T), 0, st, keys, vals, s.order_out, s.n, tiles, rem, \
                       val_bits, starts, fit, (const int32_t *)found, s.k + 1)
        if (threads == 256) CP_BOTH(256);
        else CP_BOTH(512);
#undef CP_BOTH
        if (hipGetLastError() != hipSuccess) return CP_ERR_HIP;
        return run_sort<uint32_t, kSortThreadsLong, true>(s, st, Gate{flag, 1u});
    }
#define CP_BINS(T)                                                                                                    \
    hipLaunchKernelGGL(pct_bucket_bins_kernel<T>, dim3((unsigned)(all / dealt)), dim3(T), 0, st, keys, vals, s.order_out, s.n, dealt, tiles, \
                       rem, val_bits, starts, fit, (const int32_t *)found, s.k + 1, left)
    if (threads == 128) CP_BINS(128);
    else if (threads == 256) CP_BINS(256);
    else CP_BINS(512);
#undef CP_BINS
    const int32_t each = left_over_each(all);
#define CP_LEFT(T)                                                                                                    \
    hipLaunchKernelGGL(pct_bucket_sort_kernel<T>, dim3((unsigned)(all / each)), dim3(T), 0, st, keys, vals, s.order_out, \
                       s.n, each, tiles, rem, starts, fit, (const int32_t *)found, s.k + 1, (const uint32_t *)left)
    if (small) CP_LEFT(256);
    else CP_LEFT(512);
#undef CP_LEFT
    if (hipGetLastError() != hipSuccess) return CP_ERR_HIP;
    return run_sort<uint32_t, kSortThreadsLong, true>(s, st, Gate{flag, 1u});
}

// Partitions of at most 20,480 vertices with 32-bit keys: one workgroup sorts a whole partition
// inside LDS.
constexpr int kWholeRoundsMax = 20, kWholeMax = kSortThreadsLong * kWholeRoundsMax;
template <int THREADS, int ROUNDS, bool BINS>
int launch_whole_as(const PctOrderLaunch &s, hipStream_t st, int val_bits) {
    auto kern = pct_whole_sort_kernel<THREADS, ROUNDS, BINS>;
    const size_t lds = (size_t)THREADS * ROUNDS * 4;
    // more than 64 KB of LDS has to be asked for
    if (lds + THREADS * 32 > 64 * 1024 &&
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return CP_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)s.P), dim3(THREADS), lds, st, (const uint32_t *)s.keys_a, s.order_out, s.n,
                       s.key_bits, val_bits);
    return hip_status(hipGetLastError());
}
template <int THREADS, int ROUNDS>
int launch_whole(const PctOrderLaunch &s, hipStream_t st) {
    const int val_bits = 32 - __builtin_clz((unsigned)s.n);
    return std::max(0, s.key_bits - bin_bits(THREADS)) + val_bits <= 32
               ? launch_whole_as<THREADS, ROUNDS, true>(s, st, val_bits)
               : launch_whole_as<THREADS, ROUNDS, false>(s, st, val_bits);
}
int run_whole_sort(const PctOrderLaunch &s, hipStream_t st) {
    if (s.n <= 256 * kSortRounds) return launch_whole<256, kSortRounds>(s, st);
    if (s.n <= 512 * kSortRounds) return launch_whole<512, kSortRounds>(s, st);
    if (s.n <= 1024 * kSortRounds) return launch_whole<1024, kSortRounds>(s, st);
    return launch_whole<1024, kWholeRoundsMax>(s, st);
}

}  // namespace

int32_t pct_sort_tiles(int32_t n) {
    // (long partitions: the leading pass of the bucket path has the most tiles)
    const int tile = (n >= kSortLongFrom ? kLeadThreads : kSortThreadsShort) * kSortRounds;
    return (n + tile - 1) / tile;
}
size_t pct_counts_bytes(int32_t n, int32_t P) {
    // (and the flag of the bucket path behind them)
    return align_up((size_t)P * kMaxRadix * (size_t)pct_sort_tiles(n) * sizeof(uint32_t) + 256);
}

int launch_pct_order(const PctOrderLaunch &s, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    KeyArgs a{};
    a.b = s.b;
    a.assign = s.assign;
    a.a_stride_p = s.a_stride_p;
    a.a_stride_v = s.a_stride_v;
    a.keys = s.keys_a;
    a.status = s.status;
    a.max_b = s.max_b;
    a.n = s.n; a.P = s.P; a.k = s.k; a.bb = s.b_bits;
    int rc;
    // the bucket path: long partitions of 32-bit keys whose buckets hold a quarter of their
    // capacity on average (so that an uneven spread still fits), at least two passes to save
    const bool buckets = sort_threads(s.n) == kSortThreadsLong && s.key_bytes == 4 && s.key_bits > kBucketBits + 8 &&
                         (int64_t)s.n <= (int64_t)kBuckets * kBucketCapLarge / 4 && (int64_t)s.P * kBuckets < (1ll << 31);
    const bool whole = s.key_bytes == 4 && s.n <= kWholeMax;
    if (!buckets) {
        launch_keys(s, a, st);
        if (hipGetLastError() != hipSuccess) return CP_ERR_HIP;
    }
    if (whole)
        rc = run_whole_sort(s, st);
    else if (buckets)
        rc = run_bucket_sort(s, a, st);
    else if (sort_threads(s.n) == kSortThreadsLong)
        rc = s.key_bytes == 4 ? run_sort<uint32_t, kSortThreadsLong, true>(s, st)
                              : run_sort<uint64_t, kSortThreadsLong, false>(s, st);
    else
        rc = s.key_bytes == 4 ? run_sort<uint32_t, kSortThreadsShort, false>(s, st)
                              : run_sort<uint64_t, kSortThreadsShort, false>(s, st);
    if (rc) return rc;
    const int64_t cells = (int64_t)s.P * (s.k + 1);
    hipLaunchKernelGGL(pct_segments_kernel, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, st,
                       (const int32_t *)s.order_out, s.assign, s.a_stride_p, s.a_stride_v, s.n, s.P, s.k,
                       s.seg_out);
    return hip_status(hipGetLastError());
}

}  // namespace cpeval
