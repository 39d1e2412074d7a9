// Internal declarations shared by the host-side graph packer, the cost-table
// builder and the kernel launchers.  Nothing here is part of the C ABI.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/cpeval.h"

namespace cpeval {

constexpr int kWave = 64;              // wavefront width on gfx950
constexpr int kHubDegree = 256;        // wave-column plan: rows this long get a whole workgroup
constexpr int kHubWaves = 16;          // ... of this many wavefronts
constexpr int kColumnSplit = 24;       // ... and, four partitions a lane, rows this long a wavefront
constexpr int kMagicMaxK = 64;         // multiply-shift tables are staged in LDS up to this many devices
constexpr size_t kAlign = 256;
constexpr size_t kLdsBudget = 160 * 1024;   // LDS per workgroup on gfx950
constexpr int kWindowMaxWaves = 16;      // wavefronts per workgroup (compute + loader)
constexpr int kWindowTickSlices = 8;     // slices (compute wavefronts) per tick
constexpr int kStreamSlackChunks = 256;  // 16-byte chunks behind the packet stream that a fixed-count entry fetch may touch
constexpr int kStreamTailTicks = 16;     // empty ticks behind the last one in the slice table (the streaming loop runs on
                                         // to a multiple of 8 ticks and fetches four ticks ahead)
constexpr uint64_t kWindowTickBytes = 15 * 1024;   // packet bytes per tick, unless one slice alone is larger
constexpr int kWindowFarTicks = 12;      // a neighbour this many ticks back (or more) is read from the output array
constexpr int kWindowFarLead = 4;        // ticks a far wavefront runs ahead (twice: read list, then gather)
constexpr int kWindowMaxFarWaves = 4;    // 64 far reads per tick each
constexpr int kWindowMaxGroups = 8;     // partitions one workgroup may hold
constexpr int kLaneUnit = 8;             // lane-window plan: sub-rows of a unit
constexpr int kLaneIdBits = 6;           // a ring word is value << 6 | device id
constexpr int kLaneTickVerts = 256;      // vertices of a tick
constexpr int kLaneTickBytes = 12 * 1024; // packet of a tick
constexpr int kLaneFarTicks = 16;        // a neighbour this many ticks back (or more) may be a far read
constexpr int kLaneMaxFar = 96;          // far reads of a tick
// Ring of a workgroup of 8 partitions, beside stage slots and tables.  Graphs whose ring only fits 4 at a
// time are slower than under the other window plans (211,000 vertices in 1,000 levels, 512 partitions:
// 1.8 against 1.5 ms for both sweeps): they are not packed for this one.
constexpr size_t kLaneRingBytes = 80 * 1024;
constexpr int kMaskWords = 72;           // 32-bit mask words one tick's id range may touch (fused mask)

inline size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }

// One sweep direction of the wave-column plan: a CSR over original vertex ids.
struct ColumnDir {
    size_t ptr_off = 0;     // int32 [n+1]
    size_t idx_off = 0;     // int32 [m]     neighbour vertex (head for the b sweep, tail for the t sweep)
    size_t wt_off = 0;      // uint32 or int64 [m]  t(e) in this CSR's order
    size_t order_off = 0;   // int32 [n]     vertices in sweep order, long rows first inside a level
    size_t rows_off = 0;    // int32 [n][4]  {vertex, first edge, end of its edges, step} in sweep order: what a
                            //               wavefront of the wave-column plan needs to start, in one load; step =
                            //               the vertex's level, counted in the direction of the sweep
    size_t lvl_off = 0;     // int32 [L][4]  {first position, hub rows, rows, 0} per level in sweep order
    // per level, in sweep order
    std::vector<int32_t> lvl_begin, lvl_hubs, lvl_count;
    std::vector<int32_t> lvl_longest;    // edges of the longest row that is no hub row
    std::vector<int32_t> lvl_split;      // rows of kColumnSplit edges or more that are no hub rows
};

// One sweep direction of the resident-window plan.  Vertices are renumbered by
// position in sweep order.  A level is cut into ticks (runs of at most
// kWindowTickSlices slices and about kWindowTickBytes of packet), and everything
// a tick needs is one contiguous "packet" of 16-byte chunks, so that loader
// wavefronts can stream it into LDS ahead of the compute wavefronts.  A slice is
// 64 rows (vertices), one per compute wavefront; a slice of at most 32 rows gives
// each row 2..64 lanes that share its edges and fold their maxima at the end.
//   descriptors  smax x {byte offset of the slice's entries in the packet,
//                        width | rows << 16 | log2(lanes per row) << 24,
//                        lowest vertex id of the tick, ring slot of row 0}
//                (rows = 0 for slices this tick does not have)
//   records      per slice 64 x {original vertex id, c}; rows past `rows` are padding
//                and carry the tick's lowest vertex id
//   entries      per slice width x 64 x {ring field of the neighbour, t(e)}: entry j
//                of lane l of a slice sits at base + j*64 + l.  The ring field is the
//                neighbour's slot (times 8 when the ring holds {value, device}
//                pairs: a byte offset); padding entries point at slot `slots`,
//                which holds the constant 0, with t = 0.  When the ring cannot hold
//                every neighbour (far_cap > 0), a neighbour computed far_ticks or more
//                ticks earlier is a far read: its entry points at a pair behind the ring
//                (byte offset ring bytes + (tick & 1) * 8 * far_cap + 8 * index) that a far
//                wavefront fills from the output array before the tick starts.  An entry is two uint32, or
//                one uint32 (field | t << 16) when both fit 16 bits (ent4).
struct WindowDir {
    size_t stream_off = 0;   // uint4 [total_chunks]
    size_t tick_off = 0;     // uint32 [ticks+1][4] {first chunk, chunks, lowest id, id span}
    size_t gmap_off = 0;     // int32 [ticks*wpad] original id per padded position, -1 = padding
    size_t far_off = 0;      // uint32 [ticks][far_cap][2] {vertex, c} of the tick's far reads (padding: vertex 0)
    size_t stab_off = 0;     // uint32 [ticks][smax][8] per slice {record chunk, entry chunk, width | rows << 16 | log2 lanes
                             // per row << 24, lowest id of the tick, ring slot of row 0, 0, 0, 0}: where a compute wavefront
                             // that streams its own slices finds them (chunks of 16 bytes from the start of the stream;
                             // slices a tick does not have point at its packet with rows = 0).  0 = not built (only
                             // for 4-byte entries, a packed ring and no far reads)
    int32_t max_width = 0;   // entries per lane of the widest slice
    int32_t far_cap = 0;     // far reads per tick, a multiple of 64; 0 = every neighbour is in the ring
    int64_t total_chunks = 0;
    int32_t ticks = 0;
    int32_t max_chunks = 0;  // largest packet
    int32_t wpad = 0;        // tick width rounded up to whole slices of 64
    int32_t smax = 0;        // slices of the widest tick
    int32_t slots = 0;       // ring capacity R: slot of position i is i mod R
    int32_t idpad = 0;       // bytes a stage slot reserves for device ids
    bool direct_ok = false;  // every tick's vertices lie in a short id range
    bool packed = false;     // ring of {value, device} pairs (32-bit ticks only)
    bool ent4 = false;       // 4-byte entries
};

// One sweep direction of the lane-window plan (window_lanes.hip): several partitions per
// workgroup, side by side in the lanes.  A vertex's edges are cut into sub-rows of `width` entries
// (2 or 4, one for the whole graph); a unit is 8 sub-rows, and a tick has an even number of units (the
// last one may be all padding).  What a tick needs is one packet:
//   units     8 x {ring slot of the vertex, c}, then width x 8 x {ring slot of the neighbour, t}: entry j of
//             sub-row r at j * 8 + r.  Padding entries read slot `slots`, which holds 0, with t = 0;
//             padding sub-rows write to slot `slots + 1`, which nothing reads
//   vertices  {id, c} in ring order
//   far out   ring slots of the vertices that far reads of later ticks ask for
// rounded up to 16 bytes.  Where the ring cannot hold every neighbour, one computed far_ticks or more ticks
// earlier is a far read: its entry names a row behind the ring, slots + 2 + (tick & 1) * far_cap + number,
// which a far wavefront fills before the tick starts from a copy of the word kept in the workspace.
struct LaneDir {
    size_t stream_off = 0;   // the packets, tick after tick
    size_t tick_off = 0;     // uint32 [ticks] units | vertices << 14 | far out << 23
    size_t far_off = 0;      // int32 [ticks][far_cap] numbers of the vertices the tick's far reads ask for, counted in the
                             // order they are computed; padding: 0
    int32_t far_cap = 0;     // far reads per tick, a multiple of 16; 0 = none anywhere
    int32_t far_count = 0;   // vertices some far read asks for
    size_t pos_off = 0;      // int32 [n] position of a vertex: the positions of a tick follow those of the last
    int32_t ticks = 0, slots = 0, max_chunks = 0, max_verts = 0, width = 0;
    int64_t units = 0;       // of all ticks
};
inline uint32_t lane_unit_bytes(int width) { return 64u * (1u + (uint32_t)width); }

// One sweep direction of the chain sweep (chain_sweep.hip).  A row is a vertex with its edges, four a lane in a group of 1, 2,
// 4, 8 or 16 lanes; one of more than kChainRow edges is put together from rows with kChainRow of them each, in a stage of
// its level before its own.  Rows are numbered as they are computed; a stage is one or more ticks of `chain_width` lanes.
//   units     per lane {ring slots of the neighbours, 16 bits each, two words; ring slot written | log2 of the row's lanes
//             << 16 | the same of the widest row in the wavefront << 20; vertex for the first lane of its row, else
//             2^32 - 1}.  An edge that a lane does not have reads slot `slots`; lanes that are not the first of a
//             row write slots behind it, one a lane
//   edges     per lane {first edge in the CSR, the top bit set where the row is put together from others and its edges cost
//             nothing; vertex, the top bit set in the rows that one is put together from, which leave w out}, {0, 2^32 - 1}
//             for lanes without a row
// Behind the ticks come one or more empty ones that are run through, to a multiple of kChainAhead in all, and kChainAhead
// that are only read.
struct ChainDir {
    size_t unit_off = 0;     // uint32 [ticks][width][4]
    size_t edge_off = 0;     // uint32 [ticks][width][2]
    int32_t ticks = 0, slots = 0;
};
constexpr int kChainAhead = 8;           // ticks a lane's records are read ahead
constexpr int32_t kChainRow = 64;        // edges of a row
constexpr uint32_t kChainNobody = 0xffffffffu;
constexpr int32_t kChainLevels = 256;    // levels from which a graph is packed for it
constexpr size_t kChainLdsBytes = 152 * 1024;

// The whole-graph sweep (whole_sweep.hip).  A unit is up to four edges of a vertex, 32 bytes:
//   {neighbours, 16 bits each, two words; vertex; c} {t of the edges}
// An edge that a unit does not have names vertex n, with t = 0; units without a vertex are of vertex n + 1.  A tick is
// `units_a_tick` units of one level; both sweeps have as many ticks, a multiple of kWholeAhead, and kWholeAhead empty ones
// behind them that are only read.
struct WholeDir {
    size_t units_b = 0, units_t = 0;         // [ticks + kWholeAhead][units_a_tick]
    int32_t ticks = 0, units_a_tick = 0;
};
constexpr int kWholeAhead = 4;
// Both sweeps of 4 partitions take 40 bytes a vertex of 32-bit words, beside the tables: two such groups share a compute unit up
// to some 2,030 vertices on 4 devices and 1,980 on 16 (of 64-bit words half that, where the model's time decides).  Graphs
// that leave it to one are slower than under the lane-window plan: 3,600 vertices in 60 levels, 8 and 4,096 partitions 57 and
// 224 us against 45 and 168.
constexpr int32_t kWholeVertices = 2048;

struct Packed {
    int32_t n = 0, L = 0;
    int64_t m = 0;
    bool narrow = false;        // every c and t < 2^32: weights stored as uint32
    cp_graph_info info{};
    ColumnDir col_b, col_t;
    size_t c_off = 0;           // uint32 or int64 [n], original ids
    size_t sources_off = 0;     // int32 [num_sources]
    bool have_window = false;
    WindowDir win_b, win_t;
    bool have_lanes = false;
    int32_t lane_word = 4;      // bytes of a ring word of the lane-window plan
    LaneDir lane_b, lane_t;
    bool have_whole = false;
    WholeDir whole;
    bool have_chain = false;
    int32_t chain_width = 0;    // lanes of a workgroup of the chain sweep
    ChainDir chain_b, chain_t;
    int32_t max_width = 0;
    int32_t hops = 0;           // L times the mean of 1 / (levels an edge climbs)
    double scattered = 0;       // share of vertices that are 64 numbers or more from the one before them in level order
    int32_t reach = 0;          // every edge leads to a later vertex, this many further on at most; else 0
    std::vector<uint8_t> blob;  // host image of the device blob
};

// Room for a graph's blob, made at once: growing it piece by piece copied it more often than it was written (121,000
// vertices, 364,000 edges: 88 -> 60 ms, together with packets that are written in place).  A window packet takes up to
// 10 bytes an edge and 700 a level, a lane packet 20 an edge, as a rule; pages that stay untouched cost nothing.
inline size_t blob_room(int32_t n, int64_t m, int32_t L, bool narrow) {
    const size_t per_edge = 4 + (narrow ? 4 + 10 + 20 : 8), per_vertex = 24 + 8 + (narrow ? 16 + 40 : 0);
    // (a lane of the chain sweep takes 24 bytes: one a vertex and one for every four edges, or a few more)
    const size_t chain = narrow && L >= kChainLevels ? 2 * 24 * ((size_t)n + (size_t)m / 4 + 64 * (size_t)L) : 0;
    // (a unit of the whole-graph sweep 32, and up to 64 units a tick of a level)
    const size_t whole = narrow && n <= kWholeVertices ? 2 * 32 * ((size_t)n + (size_t)m / 4 + 64 * (size_t)L + 512) : 0;
    return 2 * ((size_t)m * per_edge + (size_t)n * per_vertex + (size_t)L * (narrow ? 700 : 32)) + (1 << 18) + chain + whole;
}

// Validate and pack.  Returns CP_OK or an error code.
int pack_graph(int32_t n, int64_t m, int32_t L,
               const int32_t *succ_ptr, const int32_t *succ_idx, const int64_t *succ_t,
               const int32_t *pred_ptr, const int32_t *pred_idx, const int32_t *pred_eid,
               const int64_t *c, const int32_t *level_ptr, const int32_t *level_vtx,
               Packed &out);

// ---- cost tables -----------------------------------------------------------

// Multiply-shift form of ceil(a/d) for a 32-bit dividend:
//   ceil(a/d) = ((a + dm1) * mul + (a + dm1)) >> 32     with dm1 = d-1, mul = ceil(2^32/d) - 1.
// A free transfer (same device) is the pair {0, 0}, which yields 0 for every a < 2^32.
struct alignas(8) Magic { uint32_t mul, dm1; };

struct CostTables {
    int32_t k = 0;
    bool magic_ok = false;              // every divisor admits the exact 32-bit form for this graph's weights
    std::vector<Magic> magic;           // [k*k edge (row = own device, col = neighbour), b sweep]
                                        // [k*k the same transposed, t sweep] [k vertex]
    std::vector<int64_t> divisor;       // same layout, plain divisors; 0 = free transfer
    // The compact form: every divisor <= 256 and exact as (d - 1) | (upper 24 bits of the multiplier) << 8
    // for this graph's weights, which must be below 2^24.  A 4-byte entry can sit in LDS once per
    // bank, which takes the bank conflicts out of the kernels' table reads.
    bool tab4_ok = false;
    std::vector<uint32_t> tab4;         // same layout; 0 = free transfer
};

// Returns CP_OK, CP_ERR_SPEED or CP_ERR_BANDWIDTH.
int build_cost_tables(int32_t k, const int64_t *speeds, const int64_t *bandwidth,
                      bool narrow, int64_t max_c, int64_t max_t, CostTables &out);

// Whether the lane-window and whole-graph sweeps take a call with 64-bit ring words: every divisor, and every volume and divisor
// together, below 2^32.  (Their divisions are exact without that; it keeps the calls that they take, and those that
// CP_PLAN_LANE_WINDOW refuses, as they were when it was needed.)
bool wide_words_fit(int32_t k, const int64_t *speeds, const int64_t *bandwidth, int64_t max_c, int64_t max_t);

// Numbers just below 1 / divisor, 0 for a free transfer; same layout.  For kernels that divide by one multiply-add rounded up
// (inverse_div), exact for every dividend a below 2^32: a / divisor less a times the entry is below 1 / divisor.
void build_inverse_table(int32_t k, const int64_t *speeds, const int64_t *bandwidth, double *out);
// The same as floats, in units of kFloatUnit: for dividends below kFloatMost.
void build_float_table(int32_t k, const int64_t *speeds, const int64_t *bandwidth, float *out);
constexpr float kFloatUnit = 0.015625f;      // 2^-6
constexpr int64_t kFloatMost = 1 << 23;

inline size_t table_entries(int32_t k) { return (size_t)2 * k * k + k; }
// 64-bit words of one call's tables in device memory: the 8-byte entries, then the 4-byte ones
inline size_t table_words(int32_t k) { return table_entries(k) + (table_entries(k) + 1) / 2; }

}  // namespace cpeval

struct cp_graph {
    cpeval::Packed packed;
    void *device_blob = nullptr;
};
