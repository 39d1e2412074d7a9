// Host-callable launchers implemented in kernels.hip.
#pragma once

#include <algorithm>

#include "cpeval_internal.hpp"

namespace cpeval {

struct SweepLaunch {
    const uint8_t *blob = nullptr;      // device blob base
    const ColumnDir *dir = nullptr;     // wave-column plan
    const WindowDir *win = nullptr;     // resident-window plan
    size_t c_off = 0;
    bool tsweep = false;
    bool magic = false;                 // multiply-shift tables (else plain divisors)
    bool narrow = false;                // 32-bit weights in the blob
    int tick_bytes = 4;
    int32_t n = 0, P = 0, k = 0, L = 0, max_width = 0;
    int64_t m = 0;                      // critical-path walk only, and Packed::hops
    int32_t hops = 0, reach = 0;
    const uint8_t *pT = nullptr;        // [n][P] device ids (wave-column)
    const uint8_t *assign = nullptr;    // caller's assignments (resident-window: input of the gather)
    const uint8_t *pperm = nullptr;     // [P][ticks*wpad] device ids in sweep order (resident-window)
    bool direct_ids = false;            // resident-window: stage ids straight from `assign`
    int64_t a_stride_p = 0, a_stride_v = 0;
    void *val = nullptr;                // ticks of (v, q) at v * out_sv + q * out_sq (resident-window sweep,
                                        // critical-path walk); the wave-column sweep writes [n][P]
    int64_t out_sv = 0, out_sq = 1;
    int64_t *cp_out = nullptr;          // resident-window b sweep only
    const void *edge_tab = nullptr;
    const void *vert_tab = nullptr;
    const uint32_t *edge_tab4 = nullptr;   // the same tables as 4-byte entries (compact, or inverses as floats), or null
    const uint32_t *vert_tab4 = nullptr;
    int32_t *status = nullptr;
    // resident-window t sweep that also writes the mask rows (partition-major): b, CP and the
    // zeroed mask; all null otherwise
    const void *mask_b = nullptr;
    const int64_t *mask_cp = nullptr;
    uint64_t *mask_out = nullptr;
};

// Launch shape of the resident-window kernel for one sweep direction.
struct WindowCfg {
    int nl = 0;        // 16-byte loads per loader lane per level
    int nlw = 0;       // loader wavefronts
    int nc = 0;        // compute wavefronts
    int nfw = 0;       // far wavefronts
    int dr = 0;        // levels a loader runs ahead in registers
    bool packed = false;   // ring holds {value, device} pairs (one LDS read per relaxation)
    int groups = 1;        // partitions per workgroup (they share the cost tables)
    size_t sub_bytes = 0;  // LDS of one partition: ring, far pairs, two stage slots
    size_t lds_bytes = 0;  // of the workgroup: groups * sub_bytes + tables
};

// Launch shape of the shared-window kernel (several partitions per workgroup behind one
// loader set and one pair of stage slots) for one sweep direction.
struct SharedCfg {
    int groups = 0;    // partitions per workgroup: 2 or 4
    int nl = 0;        // 16-byte loads per loader lane per tick
    int nlw = 0;       // loader wavefronts
    int nc = 0;        // compute wavefronts
    int nfw = 0;       // far wavefronts
    size_t vals_off = 0, stage_off = 0, tab_off = 0;   // LDS byte offsets: ring values, stage slots, cost tables
    size_t lds_bytes = 0;
    int tab_rs = -1;   // >= 0: 4-byte cost-table entries, each 2^tab_rs times in LDS
};
// False if the direction cannot run that way under `lds_limit` bytes of dynamic LDS.
// tab4: the call's cost tables exist as 4-byte entries.
bool shared_config(const WindowDir &d, int32_t k, int groups, size_t lds_limit, SharedCfg &out, bool tab4 = false);
// Bytes of the cost tables in LDS as 4-byte entries, every transfer entry 2^rs times.
inline size_t tab4_lds_bytes(int32_t k, int rs) {
    return ((((size_t)k * k * 4) << rs) + (size_t)k * 4 + 15) & ~(size_t)15;
}
int launch_window_shared(const SweepLaunch &s, const SharedCfg &cfg, void *stream);

// Launch shape of the streamed resident-window kernel (compute wavefronts fetch their own
// slices; only the per-partition bytes are staged) for one sweep direction.
struct StreamCfg {
    bool wide = false; // some slice has more than 8 entries per lane: 16 entry registers instead of 8
    int nl = 0;        // 16-byte loads per loader lane per tick
    int nlw = 0;       // loader wavefronts
    int nc = 0;        // compute wavefronts = slices of the widest tick
    size_t stage_off = 0, tab_off = 0;   // LDS byte offsets of the stage slots and the cost tables
    size_t lds_bytes = 0;
};
// False if the direction cannot run that way under `lds_limit` bytes of dynamic LDS.
// with_mask: the t sweep also stages the tick's b values and writes the mask.
bool stream_config(const WindowDir &d, int32_t k, size_t lds_limit, bool with_mask, StreamCfg &out);
int launch_window_stream(const SweepLaunch &s, const StreamCfg &cfg, void *stream);

// Workgroups of 256 threads of the launch that writes `words` table entries and clears `cells` CP values:
// a thread per cell, up to kPrepareBlocks workgroups.
constexpr int kPrepareBlocks = 2048;
inline unsigned prepare_blocks(int32_t words, int32_t cells) {
    return (unsigned)std::max<int64_t>({1, ((int64_t)words + 255) / 256,
                                        std::min<int64_t>(kPrepareBlocks, ((int64_t)cells + 255) / 256)});
}

// Which row of a level and which 64 partitions (a slice) a wavefront of the wave-column kernel takes.  Rows are sorted by
// length, and blocks go round the 8 XCDs.
//   by rows   (parts = 0) all slices of a row before the next one: the longest rows start first, and all XCDs share them
//   by runs   slice after slice, a slice's blocks cut into `parts` runs that are dealt to the XCDs: an XCD's L2 keeps a
//             slice's values while its rows read them, and the edges of its rows from slice to slice
// By runs go launches of hub rows (all long, so that runs are even), and rows of up to kHubDegree edges with long ones
// among them where the slices are few or one per XCD: those of a slice then share an L2.  With more slices, one
// XCD would get all long rows.  Everything else goes by rows: t sweeps of the graphs below 1.05 to 1.3 times as fast as by runs.
// Levels with one row in a hundred of a tenth of a level's edges, by rows -> by runs, b sweeps: 10,000 rows, 17 slices
// 1,766 -> 1,347 us (hubs by runs), 6,500 rows, 5 slices 269 -> 257; 2,446 rows (244 edges, no hub rows) 1 slice 294 ->
// 260, 4 slices 312 -> 256, 8 slices 308 -> 247, but 10 slices 328 -> 378, 17 slices 342 -> 507.
#if defined(__HIPCC__)
#define CP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define CP_HOST_DEVICE inline
#endif
constexpr int kColumnRunRow = 64;         // edges of a long row
struct ColumnDeal { int32_t parts, part_blocks; };
inline bool column_by_runs(int32_t longest_row, int32_t slices) {
    return longest_row >= kHubDegree || (longest_row >= kColumnRunRow && (slices <= 4 || slices == 8));
}
inline ColumnDeal column_deal(int32_t rows, int32_t slices, int rows_per_block, bool by_runs) {
    if (!by_runs) return ColumnDeal{0, 0};
    const int32_t row_blocks = (rows + rows_per_block - 1) / rows_per_block;
    const int32_t even = slices % 8 == 0 ? 1 : (slices % 4 == 0 ? 2 : (slices % 2 == 0 ? 4 : 8));
    const int32_t parts = std::max(1, std::min(even, row_blocks));
    return ColumnDeal{parts, (row_blocks + parts - 1) / parts};
}
inline int64_t column_blocks(const ColumnDeal &d, int32_t rows, int32_t slices, int rows_per_block) {
    if (!d.parts) return ((int64_t)rows * slices + rows_per_block - 1) / rows_per_block;
    return ((int64_t)slices * d.parts + 7) / 8 * 8 * d.part_blocks;
}
// Row and slice of a wavefront; either may lie past the end.  (A grid holds fewer than 2^24 blocks of 256 threads.)
CP_HOST_DEVICE void column_place(uint32_t block, uint32_t wave, const ColumnDeal &d, uint32_t slices,
                                 uint32_t rows_per_block, int32_t &row, int32_t &slice) {
    if (!d.parts) {
        const uint32_t task = block * rows_per_block + wave;
        row = (int32_t)(task / slices);
        slice = (int32_t)(task % slices);
        return;
    }
    const uint32_t parts = (uint32_t)d.parts, part_blocks = (uint32_t)d.part_blocks, i = block / 8;
    const uint32_t unit = i / part_blocks * 8 + block % 8;
    row = (int32_t)((unit % parts * part_blocks + i % part_blocks) * rows_per_block + wave);
    slice = (int32_t)(unit / parts);
}

// Launch shape of the lane-window kernel, the same for both sweeps.
struct LaneCfg {
    int groups = 0;    // partitions per workgroup: 4 or 8
    int nl = 0;        // 16-byte loads per loader lane per tick
    int width = 0, word = 0;           // entries of a sub-row, bytes of a ring word
    bool floats = false;               // cost tables of floats, else doubles
    int nc = 0, nlw = 0, nsw = 0, nfw = 0;     // compute, loader, store and far wavefronts
    size_t stage_off = 0, stage_bytes = 0, tab_off = 0, ticks_off = 0, lds_bytes = 0;
};
// False if the graph cannot run that way under `lds_limit` bytes of LDS.
bool lane_config(const LaneDir &db, const LaneDir &dt, int32_t n, int32_t k, int groups, int word_bytes, bool with_out,
                 int64_t workgroups, size_t lds_limit, LaneCfg &out);
// Workspace of the sweeps a call asks for (null: not that one): the device ids regrouped for that many
// partitions per workgroup, and the far reads' copies.
size_t lane_work_bytes(const LaneDir *db, const LaneDir *dt, int32_t n, int32_t P, int groups, int word_bytes);
int launch_window_lanes(const SweepLaunch &sb, const SweepLaunch &st, const LaneDir &db, const LaneDir &dt,
                        const LaneCfg &cfg, bool want_b, bool want_t, uint8_t *ids, void *stream);

// The chain sweep of a few partitions (null: not that sweep): what the costs of P of them take, LDS of a workgroup, the
// launches, two for every `at_once` partitions, whose costs `work` has room for.
// cost16: no edge's cost and its vertex's w together reach 2^16.
size_t chain_work_bytes(const ChainDir *db, const ChainDir *dt, int32_t width, int32_t P, bool cost16);
size_t chain_lds_bytes(const ChainDir &d, int word_bytes);
int launch_chain(const SweepLaunch &sb, const SweepLaunch &st, const ChainDir &db, const ChainDir &dt, int32_t width,
                 int word_bytes, bool cost16, bool want_b, bool want_t, uint8_t *work, int32_t at_once, void *stream);

// The whole-graph sweep.
constexpr int kWholeTableWords = 880;        // 3.4 KB of cost tables among a kernel's arguments
struct WholeCfg {
    int groups = 0, word = 0, threads = 0;   // partitions per workgroup, bytes of a ring word, lanes of a workgroup
    bool floats = false;                     // tables of floats, else doubles
    size_t lds_bytes = 0, table_bytes = 0;   // ... of edge and vertex entries
};
// False if a workgroup of `groups` partitions and that many sweeps does not fit `lds_limit` bytes of LDS or 1,024 lanes.
bool whole_config(const WholeDir &d, int32_t n, int32_t k, int groups, int word_bytes, bool floats, int sweeps,
                  size_t lds_limit, WholeCfg &out);
// table: cfg.table_bytes of edge and vertex entries that go with the launch, or null: they are in device memory.
// check_all: the launch writes the status itself; else it has been cleared, and cp_out as well.
int launch_whole(const SweepLaunch &sb, const SweepLaunch &st, const WholeDir &d, const WholeCfg &cfg, bool want_b,
                 bool want_t, bool by_partition, const void *table, bool check_all, void *stream);

// False if the direction cannot run under `lds_limit` bytes of LDS.
// with_mask: the t sweep also stages the tick's b values and writes the mask.
bool window_config(const WindowDir &d, int32_t k, size_t tick_bytes, size_t lds_limit, WindowCfg &out,
                   bool with_mask = false);
// The two sweeps side by side in one launch (window_pair_kernel): shapes for both, or false
// where that form does not apply.
bool window_pair_config(const WindowDir &db, const WindowDir &dt, int32_t k, size_t lds_limit, WindowCfg &out_b,
                        WindowCfg &out_t);
int launch_window_pair(const SweepLaunch &sb, const SweepLaunch &st, const WindowCfg &cfg_b, const WindowCfg &cfg_t,
                       void *stream);
int32_t window_mask_bpad(const WindowDir &d);
int launch_gather_assign(const SweepLaunch &s, uint8_t *out, void *stream);

int launch_clear(int64_t *cp_out, int32_t batch, int32_t *status, void *stream);
int launch_transpose(const uint8_t *in, uint8_t *out, int32_t n, int32_t P, void *stream);
int launch_column_sweep(const SweepLaunch &s, void *stream, int32_t *launches);
// The same with four partitions a lane; the tables hold inverses (build_inverse_table), 16 bytes a pair of devices in the t
// sweep, which is 16 KB of a workgroup's LDS at 32.  Only where a level makes two and a half wavefronts for each of the 1,024
// SIMDs, or two with several slices and tables of up to 8 devices: below, a launch is a chain of round trips, and this kernel's is the longer one.  Without and with: 10,000 vertices a
// level, 4 and 16 slices 1,277 and 982 us, 4,226 and 2,916; 1,500 a level, 16 slices 395 and 319; 3,000 a level, one slice 164
// and 204.  Over 285 calls from two wavefronts on 0.89 times as long, 9 of them by 3 to 12 % longer (9,700 vertices a level, 40
// partitions, t sweep alone 250 and 280), but none with several slices and up to 8 devices (1,057 a level, 532 partitions, b
// alone 201 and 175); none of those left by more than 2.8 %.
constexpr int32_t kColumn4Devices = 32;
inline bool column4_fits(int32_t n, int32_t L, int32_t P, int32_t k, bool narrow, int tick_bytes) {
    return narrow && tick_bytes == 4 && P % 4 == 0 && k <= kColumn4Devices && n < 1 << 24 && P < 1 << 24 &&
           (uint64_t)n * (uint64_t)P < 1ull << 30 &&
           (int64_t)(n / L) * ((P + 63) / 64) >= (P > 64 && k <= 8 ? 4 * 2 * 1024 : 4 * 5 * 512);
}
int launch_column4(const SweepLaunch &s, void *stream, int32_t *launches);
int launch_window_sweep(const SweepLaunch &s, const WindowCfg &cfg, void *stream, int32_t *launches);
int launch_column_slice(const SweepLaunch &s, void *stream);   // CP_ERR_ARG without 32-bit multiply-shift tables
int launch_cp_sources(const int32_t *sources, int32_t nsrc, const void *b, int32_t P,
                      int tick_bytes, int64_t *cp_out, void *stream);
// One segmented radix sort per call: the PCT priority lists of section 4.1.
struct PctOrderLaunch {
    int32_t n = 0, P = 0, k = 0;
    const void *b = nullptr;          // ticks [n][P], or [P][n] with b_by_partition
    bool b_by_partition = false;
    int tick_bytes = 4;
    const uint8_t *assign = nullptr;
    int64_t a_stride_p = 0, a_stride_v = 0;
    int64_t max_b = 0;                // every b lies in [0, max_b]
    int b_bits = 1, key_bits = 1, key_bytes = 4;
    void *keys_a = nullptr, *keys_b = nullptr;   // key [P][n] each
    int32_t *vals_tmp = nullptr;      // [P][n]
    uint32_t *counts = nullptr;       // pct_counts_bytes
    int32_t *order_out = nullptr, *seg_out = nullptr, *status = nullptr;
};
size_t pct_counts_bytes(int32_t n, int32_t P);
// Buckets of the leading digit that one workgroup looks through for those that are left to the ranking by ballots, which it
// sorts one after the other: one while they are few, up to sixteen where 8,192 workgroups remain, because one that finds
// none costs as much as a whole one (262,144 buckets, none left: 65 us one by one, 14 by sixteens).  All in use left, ranked
// one by one / so: 211,000 vertices on 3 devices, 32 partitions 63 / 69 us, 128 partitions 234 / 233; on 16 devices, 512
// partitions 1,900 / 1,385.  (Fixed workgroups, 1,792 that share all buckets out in turn: 93, 278 and 1,603.)
constexpr int32_t kLeftOverMost = 16;
inline int32_t left_over_each(int32_t buckets) {
    int32_t each = 1;
    while (each < kLeftOverMost && buckets / (2 * each) >= 8192) each *= 2;
    return each;
}
// The bucket of its partition that a workgroup looks at as its t-th: far apart, and turned from partition to partition and
// from one to the next, because left buckets lie beside each other, the digits in use are the same in all partitions
// (of 9 devices, 19 in every 32) and workgroups go round the eight XCDs.
template <int kAll>
CP_HOST_DEVICE uint32_t left_over_bucket(uint32_t workgroup, uint32_t t, int32_t each) {
    const uint32_t per = (uint32_t)(kAll / each), q = workgroup / per;
    return t * per + (workgroup + q + t * 79) % per;
}
// Neighbouring buckets that one workgroup deals to bins: four where 8,192 workgroups remain, because one whose partition is
// crowded costs as much as a whole one.  262,144 buckets, all crowded: 65 us one by one, 41, 22 and 12 by twos, fours and
// eights; with work, 16 devices: 477, 369, 361 and 357; with work for the odd partition only (300 values of b): 168, 132,
// 141 and 158.  16,384 buckets, all crowded: 11 one by one, 6.7 by twos.
constexpr int32_t kBinsMost = 4;
inline int32_t bins_each(int32_t buckets) {
    int32_t each = 1;
    while (each < kBinsMost && buckets / (2 * each) >= 8192) each *= 2;
    return each;
}
// Threads of the workgroup that deals a bucket to bins, eight items each: the smallest for 1.4 times the average of the
// buckets in use (layered graphs of 211,000 to 480,000 vertices: the fullest holds 1.14 to 1.38 of it).  In use are the
// leading digits (keys without their low `rem` bits) that a device number below k and a max_b - b of max_b at most can
// have: a quarter of the 512 where both lie just above a power of two, and sized by all 512 the bins left every bucket of
// 211,000 vertices on 9 or 33 devices to the ranking.  9 devices, 512 partitions: bins 150 us in vain and 1,080 of ranking,
// then bins of 256 threads for all, 570.  A size too large costs too (16 devices, 320 digits: 128 threads 500, 256 680).
inline int64_t bucket_average(int32_t n, int32_t k, int b_bits, int rem, int64_t max_b) {
    const int64_t used = rem >= b_bits ? ((int64_t)(k - 1) >> (rem - b_bits)) + 1 : k * ((max_b >> rem) + 1);
    return n / used + 1;
}
inline int bucket_threads(int32_t n, int32_t k, int b_bits, int rem, int64_t max_b) {
    const int64_t wanted = bucket_average(n, k, b_bits, rem, max_b) * 7 / 5;
    return wanted <= 8 * 128 ? 128 : wanted <= 8 * 256 ? 256 : 512;
}
int32_t pct_sort_tiles(int32_t n);
int launch_pct_order(const PctOrderLaunch &s, void *stream);

// List-scheduling simulation (sections 4, 4.1, 5.1), one wavefront per partition.
struct SimulateLaunch {
    const uint8_t *blob = nullptr;
    const ColumnDir *succ = nullptr;    // successor CSR
    const ColumnDir *pred = nullptr;    // predecessor CSR (row bounds only)
    size_t c_off = 0;
    bool magic = false, narrow = false, pct = false;
    int32_t n = 0, P = 0, k = 0, max_in_degree = 0;
    int64_t m = 0;
    uint32_t window = 0;                // shortest execution time + shortest transfer time - 1
    int32_t groups = 1;                 // partitions per wavefront (at most 64 / k)
    const uint8_t *assign = nullptr;
    int64_t a_stride_p = 0, a_stride_v = 0;
    const void *b = nullptr;
    int64_t b_sv = 0, b_sq = 0;
    int b_bytes = 4;
    const int32_t *tie = nullptr;
    int32_t *tie_inv = nullptr;         // [n] scratch when tie is given
    const void *edge_tab = nullptr, *vert_tab = nullptr;
    int32_t *ready = nullptr, *need = nullptr, *inbox = nullptr;   // [P][n] each
    uint64_t *pending = nullptr, *available = nullptr;             // [P][n] each (available: PCT only)
    int64_t *makespan = nullptr;
    int32_t *start = nullptr;
    int32_t *status = nullptr;
};
int launch_simulate(const SimulateLaunch &s, void *stream);

int launch_validate(const uint8_t *assign, int64_t a_stride_p, int64_t a_stride_v, int32_t n, int32_t P, int32_t k,
                    int64_t num_pairs, const int32_t *pairs, int64_t num_pins, const int32_t *pins,
                    uint8_t *valid, int32_t *violations, int32_t *status, void *stream);
int launch_zero_bytes(uint8_t *dst, int64_t bytes, void *stream);
int launch_zero_words(uint64_t *dst, int64_t words, void *stream);
int launch_ranks(const void *b, const void *tl, const void *c, bool narrow, int tick_bytes, int32_t n,
                 int64_t *up, int64_t *down, int64_t *total, void *stream);
// jumps: scratch of path_jump_words(n) words for one partition's path by jumps, or null.
// records: scratch of n records of kPathRecordWords words, on a 64-byte boundary, for the walk over records, or null.
constexpr size_t kPathRecordWords = 16;
int launch_critical_path(const SweepLaunch &s, const int32_t *sources, int32_t nsrc, const int64_t *cp,
                         int32_t max_len, int32_t *path, int32_t *len, int32_t *jumps, uint32_t *records,
                         void *stream);
inline size_t path_jump_words(int32_t n) { return 3 * ((size_t)n + 1); }
// Both rules ask for levels and for hops: a critical path has about as many vertices as L over the levels that its edges
// climb, and it takes the short ones (measured: 13 to 25 vertices for 5 to 29 hops, 323 for 288, 749 for 587).  A path of
// some 20 vertices through 300 levels is walked before the records are written.
// The jumps are four more launches and read the whole graph once (45 us a million vertices) where the walk pays
// its round trips, half a microsecond to one, per path vertex: many levels, and not too many vertices to one.  Walked and
// by jumps: 128 levels of 300 vertices 42 and 26 us, of 4,000 90 and 63, 300 of 3,000 190 and 93.
inline bool path_by_jumps(int32_t n, int32_t P, int32_t L, int32_t hops) {
    return P == 1 && L >= 128 && n / L < 4096 && hops >= 32;
}
// Records are one more launch, which reads the graph and writes 64 bytes a vertex (5 us at 60,000 vertices, 16 at 240,000),
// and save a tenth to a half of a microsecond per path vertex.  Without and with: 195 levels of 65 vertices 107 and
// 105 us, 256 of 900 163 and 114, 300 of 300 131 and 98, 1,000 of 60 406 and 304; edges of up to 299 levels, 300 of 1,000,
// 74 and 78.  Not where most rows are longer than a record: 400 levels of 300 vertices with 20 edges each, 24 partitions,
// 225 and 341 us.
inline bool path_by_records(int32_t n, int64_t m, int32_t L, int32_t hops) {
    return L >= 256 && n / L < 1024 && m / n <= 5 && hops >= 64;
}
// Fewer than 32 partitions have to share the launch: not with more than 500 or, from 8 on, 700 vertices to one of a path, nor with fewer edges than two
// for three vertices, whose paths end after a few, nor, unless the vertices are few, with rows near a record's seven edges, from
// four on under 8 partitions and five under 32.  Of 800 calls of up to 7 partitions without and with records 466 take
// them, 0.90 times as long, one of those more than 1.1 times, 1.24; of all 800 108 were more than 1.1 times, 2.1
// at most (365,000 vertices, 182,000 edges, one partition 53 and 114 us; 236,000 vertices with six edges each, two 83 and 123).
inline bool records_for(int32_t n, int64_t m, int32_t P, int32_t hops) {
    return P >= 32 || (3 * m >= 2 * (int64_t)n && n / (P < 8 ? 500 : 700) <= hops &&
                       (m < (P < 8 ? 4 : 5) * (int64_t)n ||
                        (n < std::min(2000 * P, 12000) && m < (P < 8 ? 5 : 6) * (int64_t)n)));
}
// Vertices of the LDS ring that b and the device ids are streamed through on a walk over records, or 0 where they are not.
// The whole rows are read for it, 5 bytes a vertex at 4.5 TB/s, which half a microsecond a path vertex has to outweigh.  With
// fewer than 64 partitions b comes from the caches, and past 1,024 the walks of a compute unit hide each other's round trips.
// Loaded as asked for and streamed: 121,000 vertices in 701 levels, 8, 100 and 777 partitions 196 and 274 us, 227 and 171,
// 326 and 292; 18,000 in 300 levels, 64, 777 and 3,000 partitions 136 and 128, 138 and 107, 196 and 237; 240,000 in 1,000
// levels, 200 partitions 684 and 469.  Not with rings of 16,384, one workgroup a compute unit (240,000 in 400 levels, 300
// partitions 178 both), nor where every XCD's records are more than the rows (950,000 in 1,900 levels, 80 partitions 673
// and 799), nor where fewer than 32 partitions would not take records for the number of vertices or edges (406,000 vertices
// in 1,127 levels, 404,800 edges, 123 partitions 199 and 338), nor where the ring and the tables leave the LDS of the
// compute units, in granules of 1,280 bytes, no room for all partitions at once (64 devices, whose tables are 33 KB, 599
// partitions 586 and 1,004).  Over 1,950 calls streamed took 0.90 times as long, none more than 1.09 times.
constexpr size_t kPathLdsBytes = 64 * 1024;
inline int32_t path_ring(int32_t n, int64_t m, int32_t P, int32_t hops, int32_t reach, size_t tables_bytes) {
    if (reach <= 0 || P < 64 || P > 1024 || n > 500000 || (double)n * P * 5 / 4.5e6 > 0.5 * hops || n / 700 > hops ||
        3 * m < 2 * (int64_t)n)
        return 0;
    for (int32_t ring : {4096, 8192}) {
        const size_t lds = tables_bytes + (size_t)ring * 5, taken = (lds + 64 + 1279) / 1280 * 1280;
        if (reach + 4 * 512 <= ring) return lds <= kPathLdsBytes && (size_t)P <= 256 * (kLdsBudget / taken) ? ring : 0;
    }
    return 0;
}
// cp_eval of one partition (CP_PLAN_AUTO) with scratch of its own for the chain sweep (eval_chain_bytes), or null;
// `workspace` as for a call that goes without it (eval_one_bytes).
size_t eval_chain_bytes(const cp_graph *g, bool both);
int eval_one_bytes(const cp_graph *g, int32_t k, int out_layout, int tick_dtype, size_t *out_bytes);
int eval_one(const cp_graph *g, int32_t k, const uint8_t *assignment, const int64_t *speeds, const int64_t *bandwidth,
             void *workspace, size_t workspace_bytes, void *stream, int64_t *cp_out, void *blevel_out, void *tlevel_out,
             int tick_dtype, int out_layout, int32_t *status_out, uint8_t *chain_scratch, size_t chain_scratch_bytes);
// cp_critical_path with scratch for the jumps or null; with it, what lies behind the path in path_out stays as it was.
int critical_path(const cp_graph *g, int32_t batch, int32_t k, const uint8_t *assignments, int assign_layout,
                  const int64_t *speeds, const int64_t *bandwidth, const void *blevel, const int64_t *cp,
                  int tick_dtype, int b_layout, void *workspace, size_t workspace_bytes, void *stream,
                  int32_t max_len, int32_t *path_out, int32_t *len_out, int32_t *status_out, int32_t *jumps);
int launch_mask(const void *b, const void *tl, const int64_t *cp, int32_t n, int32_t P,
                int tick_bytes, bool by_partition, uint64_t *mask, void *stream);
int launch_transpose_ticks(const void *in, void *out, int32_t rows, int32_t cols, int tick_bytes, void *stream);

}  // namespace cpeval
