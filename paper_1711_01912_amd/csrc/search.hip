// Critical-path move search on top of cp_eval.  The paper's path-based strategies
// (section 3.2) place the critical path first because it decides the running time;
// this is the same idea as a descent over partitions: every single move of a vertex of
// the current critical path to another device is a candidate, and the best one that meets
// the placement constraints (section 2) is taken while it shortens the critical path.
//
// A candidate moves one vertex v and nothing else, so its critical path needs no sweep of
// its own.  Ranks that do not pass through v stay what they are in the current partition:
// tl of v's predecessors, b of its successors, and every path that avoids v.  Hence
//
//     CP(v -> d) = max( longest path that avoids v,  tl_d(v) + b_d(v) )
//
// with tl_d and b_d from v's own edges under device d.  A path visits a level at most once,
// so it avoids v exactly if, at v's level, it visits another vertex, jumps over the level
// with one edge, has ended, or has not begun: the first term is a maximum over the other
// vertices u of the level (tl + b), the edges (x, y) that span it (tl(x) + w(x) + x(e) + b(y)),
// the sinks before it (tl + w) and the sources after it (b).  Every edge, sink and source is a
// range of levels with a value, and the maxima of all levels come from one pass over the graph.
// A step is then both sweeps of ONE partition, the walk of its path, and that pass, whatever
// the number of candidates: 211,000 vertices in 1,000 levels on 16 devices, three moves of about
// 5,000 candidates each take 2.9 ms, 32.2 ms when every candidate was evaluated by a sweep of its
// own.  Per step: both sweeps 0.78 ms (chains of dependent steps of one partition), the path by jumps
// 0.045 ms, the pass over the graph 0.03 ms, the candidates 0.007 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <new>
#include <vector>

#include "cpeval_internal.hpp"
#include "device_math.hpp"
#include "launch.hpp"

namespace cpeval {

namespace {

constexpr long long kNoValue = LLONG_MAX;
constexpr int kLongRow = 32;         // edges from which a vertex's row is shared out over the wavefront
constexpr int kOneBlockLevels = 4096;     // range tables up to this many levels are folded by one workgroup
constexpr int32_t kAnyDevice = -1, kNoDevice = -2;

// One path vertex's best candidate; slots are numbered along the path.
struct SlotBest {
    long long value;     // smallest CP, kNoValue = no admissible move
    int32_t device;      // lowest-numbered device that reaches it
    int32_t pad;
};

// What a step leaves for the host, read back in one copy.
struct StepResult {
    int32_t len;
    int32_t status[2];
    int32_t moved;       // 1: the partition was changed
    int64_t cp;          // of the partition before the move
    int64_t best;        // ... and after it
    int32_t vertex, device;
};

struct StepArgs {
    const int4 *rows_t;           // {vertex, first in-edge, end, level}, levels first to last
    const int32_t *s_ptr, *s_idx; // successor CSR
    const void *s_wt;
    const int32_t *p_ptr, *p_idx; // predecessor CSR
    const void *p_wt;
    const void *c;
    const uint8_t *assign;
    const void *b, *tl;           // of the current partition
    const void *edge_tab;         // row = device of the edge's source vertex
    const void *vert_tab;
    int32_t *level;               // [n]
    int32_t *slot_at;             // [L] slot of the path vertex of a level, -1 = none
    const int32_t *path;
    unsigned long long *over;     // [log2][L] maxima of level ranges of 2^j levels, by first level; row 0 = per level
    int32_t *want;                // [L] per slot: the device its constraints ask for
    int32_t *mine;                // [L] per slot: broken constraints that name its vertex
    int32_t *broken;              // broken constraints in all
    SlotBest *slots;              // [L]
    StepResult *res;
    int32_t n, L, k, rows_over;
    bool constrained;
};

template <typename WT, bool MAGIC>
__device__ __forceinline__ long long cost_of(WT a, const void *tab, int32_t at) {
    return MAGIC ? (long long)magic_div((uint32_t)a, ((const Magic *)tab)[at])
                 : (long long)plain_div((uint64_t)a, (uint64_t)((const int64_t *)tab)[at]);
}

__device__ __forceinline__ uint32_t device_of(const StepArgs &a, int32_t v) {
    return min((uint32_t)a.assign[v], (uint32_t)(a.k - 1));      // an id >= k is reported by the sweeps
}

__global__ __launch_bounds__(256) void level_kernel(StepArgs a) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < a.n) {
        const int4 r = a.rows_t[i];
        a.level[r.x] = r.w;
    }
}

// Clears the step's tables: level ranges, slots of levels, constraint state.
__global__ __launch_bounds__(256) void step_clear_kernel(StepArgs a) {
    const int64_t cells = (int64_t)a.rows_over * a.L;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < cells; i += (int64_t)gridDim.x * 256) {
        a.over[i] = 0;
        if (i < a.L) {
            a.slot_at[i] = -1;
            a.want[i] = kAnyDevice;
            a.mine[i] = 0;
        }
        if (i == 0) *a.broken = 0;
    }
}

__global__ __launch_bounds__(256) void step_path_kernel(StepArgs a) {
    const int32_t len = a.res->len;
    for (int32_t i = blockIdx.x * 256 + threadIdx.x; i < len; i += gridDim.x * 256)
        a.slot_at[a.level[a.path[i]]] = i;
}

// over[row][at] = max(over[row][at], x).  The cells only grow, so a look at the cell first
// (past the L1, where the atomics do not go) keeps most values from queueing up at it.
__device__ __forceinline__ void raise_cell(unsigned long long *cell, unsigned long long x) {
    if (__hip_atomic_load(cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < x) atomicMax(cell, x);
}

// The cells of a workgroup's own levels are raised in LDS first and handed on once: where a level holds
// thousands of vertices, all of them meet in a handful of cells (10 levels of 3,000 vertices, 16 devices, three
// moves: 1.44 ms without, 0.70 with).  Cells of levels past these go to the table directly; there are many of them.
constexpr int kNearLevels = 32;
constexpr int kRangeRows = 32;             // at least rows_over: ranges of 1, 2, 4, ... levels

struct Cells {
    unsigned long long *near;              // LDS [kRangeRows][kNearLevels]
    int32_t base;                          // first level in LDS
};

__device__ __forceinline__ void raise_at(const StepArgs &a, const Cells &c, int j, int32_t s, unsigned long long x) {
    const uint32_t d = (uint32_t)(s - c.base);
    if (d < (uint32_t)kNearLevels) {
        unsigned long long *cell = c.near + j * kNearLevels + d;
        if (*(volatile unsigned long long *)cell < x) atomicMax(cell, x);
    } else {
        raise_cell(a.over + (int64_t)j * a.L + s, x);
    }
}

// A path of length x visits no vertex on the levels lo .. hi: two ranges of a power of two cover them.
__device__ __forceinline__ void raise_levels(const StepArgs &a, const Cells &c, int32_t lo, int32_t hi, long long x) {
    if (lo > hi) return;
    const int j = 31 - __clz(hi - lo + 1);
    raise_at(a, c, j, lo, (unsigned long long)x);
    if (hi - lo + 1 != 1 << j) raise_at(a, c, j, hi + 1 - (1 << j), (unsigned long long)x);
}

// One thread per vertex, in level order; long rows are left to the whole wavefront.
template <typename Tick, typename WT, bool MAGIC>
__global__ __launch_bounds__(256) void avoid_kernel(StepArgs a) {
    __shared__ unsigned long long near[kRangeRows * kNearLevels];
    const int lane = threadIdx.x & 63;
    const int32_t i = blockIdx.x * 256 + threadIdx.x;
    const Cells cells{near, a.rows_t[blockIdx.x * 256].w};
    for (int j = threadIdx.x; j < a.rows_over * kNearLevels; j += 256) near[j] = 0;
    const Tick *b = (const Tick *)a.b, *tl = (const Tick *)a.tl;
    const WT *wt = (const WT *)a.s_wt, *c = (const WT *)a.c;
    int32_t e0 = 0, e1 = 0, lv = 0, dv = 0;
    long long head = 0;                    // tl + w: when v's tensors leave
    auto edge = [&](int32_t e, int32_t from_level, int32_t from_dev, long long left) {
        const int32_t y = a.s_idx[e];
        const int32_t ly = a.level[y];
        if (ly - from_level > 1)
            raise_levels(a, cells, from_level + 1, ly - 1,
                         left + cost_of<WT, MAGIC>(wt[e], a.edge_tab, from_dev * a.k + (int32_t)device_of(a, y)) +
                             (long long)b[y]);
    };
    __syncthreads();
    if (i < a.n) {
        const int4 r = a.rows_t[i];
        const int32_t v = r.x;
        lv = r.w;
        dv = (int32_t)device_of(a, v);
        head = (long long)tl[v] + cost_of<WT, MAGIC>(c[v], a.vert_tab, dv);
        const long long through = (long long)tl[v] + (long long)b[v];
        const int32_t slot = a.slot_at[lv];
        if (slot < 0 || a.path[slot] != v) raise_at(a, cells, 0, lv, (unsigned long long)through);
        e0 = a.s_ptr[v];
        e1 = a.s_ptr[v + 1];
        if (r.y == r.z) raise_levels(a, cells, 0, lv - 1, through);        // a source: nothing before it
        if (e0 == e1) raise_levels(a, cells, lv + 1, a.L - 1, through);    // a sink: nothing after it
        if (e1 - e0 < kLongRow)
            for (int32_t e = e0; e < e1; ++e) edge(e, lv, dv, head);
    }
    for (unsigned long long wide = __ballot(e1 - e0 >= kLongRow); wide; wide &= wide - 1) {
        const int src = __ffsll((long long)wide) - 1;
        const int32_t f0 = __shfl(e0, src), f1 = __shfl(e1, src), fl = __shfl(lv, src), fd = __shfl(dv, src);
        const long long fh = __shfl(head, src);
        for (int32_t e = f0 + lane; e < f1; e += 64) edge(e, fl, fd, fh);
    }
    __syncthreads();
    for (int j = threadIdx.x; j < a.rows_over * kNearLevels; j += 256)
        if (near[j])                       // (cells past the last level are 0)
            raise_cell(a.over + (int64_t)(j / kNearLevels) * a.L + cells.base + j % kNearLevels, near[j]);
}

// Row j of the range tables handed down to row j - 1.
__device__ __forceinline__ void fold_cell(const StepArgs &a, int j, int32_t s) {
    const unsigned long long *up = a.over + (int64_t)j * a.L;
    const int32_t half = 1 << (j - 1);
    unsigned long long x = a.over[(int64_t)(j - 1) * a.L + s];
    x = max(x, up[s]);                         // cells that would reach past the last level stay 0
    if (s >= half) x = max(x, up[s - half]);
    a.over[(int64_t)(j - 1) * a.L + s] = x;
}

__global__ __launch_bounds__(1024) void fold_all_kernel(StepArgs a) {
    for (int j = a.rows_over - 1; j > 0; --j) {
        for (int32_t s = threadIdx.x; s < a.L; s += 1024) fold_cell(a, j, s);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void fold_row_kernel(StepArgs a, int j) {
    const int32_t s = blockIdx.x * 256 + threadIdx.x;
    if (s < a.L) fold_cell(a, j, s);
}

// Slot of v on the current path, -1 if it is not on it.
__device__ __forceinline__ int32_t slot_of(const StepArgs &a, int32_t v) {
    const int32_t s = a.slot_at[a.level[v]];
    return s >= 0 && a.path[s] == v ? s : -1;
}

// A constraint on the vertex of a slot: it has to go to device d, or, broken now, is mended or not by its move.
__device__ __forceinline__ void ask(const StepArgs &a, int32_t slot, int32_t d, bool is_broken) {
    if (slot < 0) return;
    const int32_t seen = atomicCAS(&a.want[slot], kAnyDevice, d);
    if (seen != kAnyDevice && seen != d) atomicExch(&a.want[slot], kNoDevice);
    if (is_broken) atomicAdd(&a.mine[slot], 1);
}

// The placement constraints, once per step: how many are broken, how many of them name each
// path vertex, and which device those that name it ask for.  A candidate is valid if no
// constraint is broken but those of its vertex, and they all ask for its device.  Constraints
// out of range are left out, as in cp_validate.
__global__ __launch_bounds__(256) void constraint_kernel(StepArgs a, int64_t num_pairs, const int32_t *pairs,
                                                         int64_t num_pins, const int32_t *pins) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    int32_t broken = 0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < num_pairs; i += stride) {
        const int32_t u = pairs[2 * i], v = pairs[2 * i + 1];
        if ((uint32_t)u >= (uint32_t)a.n || (uint32_t)v >= (uint32_t)a.n || u == v) continue;
        const int32_t du = a.assign[u], dv = a.assign[v];
        broken += du != dv;
        ask(a, slot_of(a, u), dv, du != dv);
        ask(a, slot_of(a, v), du, du != dv);
    }
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < num_pins; i += stride) {
        const int32_t v = pins[2 * i], d = pins[2 * i + 1];
        if ((uint32_t)v >= (uint32_t)a.n || (uint32_t)d >= (uint32_t)a.k) continue;
        const bool off = (int32_t)a.assign[v] != d;
        broken += off;
        ask(a, slot_of(a, v), d, off);
    }
    for (int off = 32; off > 0; off >>= 1) broken += __shfl_xor(broken, off);
    if ((threadIdx.x & 63) == 0 && broken) atomicAdd(a.broken, broken);
}

// One wavefront per path vertex, lane r its move to device r (past 64 devices, lanes go round
// again).  64 edges at a time are loaded by the lanes and handed round with readlane.
template <typename Tick, typename WT, bool MAGIC>
__global__ __launch_bounds__(64) void candidate_kernel(StepArgs a) {
    const int lane = threadIdx.x;
    const int32_t len = a.res->len, k = a.k;
    const Tick *b = (const Tick *)a.b, *tl = (const Tick *)a.tl;
    const WT *swt = (const WT *)a.s_wt, *pwt = (const WT *)a.p_wt, *c = (const WT *)a.c;
    auto spread = [&](long long x, int j) {
        return (long long)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, j) |
                           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), j) << 32);
    };
    for (int32_t slot = blockIdx.x; slot < len; slot += gridDim.x) {
        const int32_t v = a.path[slot];
        const int32_t own = (int32_t)device_of(a, v);
        const long long avoid = (long long)a.over[a.level[v]];
        const int32_t want = a.want[slot];
        const bool others_hold = !a.constrained || *a.broken == a.mine[slot];
        long long best = kNoValue;
        int32_t at = 0x7fffffff;
        for (int32_t d0 = 0; d0 < k; d0 += 64) {
            const int32_t d = d0 + lane, dc = min(d, k - 1);
            long long up = 0, down = 0;        // tl and b - w of v on device d
            const int32_t p1 = a.p_ptr[v + 1], s1 = a.s_ptr[v + 1];
            for (int32_t e0 = a.p_ptr[v]; e0 < p1; e0 += 64) {
                const int32_t e = min(e0 + lane, p1 - 1);
                const int32_t u = a.p_idx[e];
                const WT te = pwt[e];
                const int32_t du = (int32_t)device_of(a, u);
                const long long left = (long long)tl[u] + cost_of<WT, MAGIC>(c[u], a.vert_tab, du);
                const int cnt = min(64, p1 - e0);
                for (int j = 0; j < cnt; ++j) {
                    const WT tj = (WT)spread((long long)te, j);
                    up = max(up, spread(left, j) +
                                     cost_of<WT, MAGIC>(tj, a.edge_tab, __builtin_amdgcn_readlane(du, j) * k + dc));
                }
            }
            for (int32_t e0 = a.s_ptr[v]; e0 < s1; e0 += 64) {
                const int32_t e = min(e0 + lane, s1 - 1);
                const int32_t y = a.s_idx[e];
                const WT te = swt[e];
                const int32_t dy = (int32_t)device_of(a, y);
                const long long rest = (long long)b[y];
                const int cnt = min(64, s1 - e0);
                for (int j = 0; j < cnt; ++j) {
                    const WT tj = (WT)spread((long long)te, j);
                    down = max(down, spread(rest, j) +
                                         cost_of<WT, MAGIC>(tj, a.edge_tab, dc * k + __builtin_amdgcn_readlane(dy, j)));
                }
            }
            const long long cp = max(avoid, up + cost_of<WT, MAGIC>(c[v], a.vert_tab, dc) + down);
            const bool valid = d < k && d != own && others_hold && (want == kAnyDevice || want == d);
            if (valid && cp < best) {
                best = cp;
                at = d;
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            const long long ob = __shfl_xor(best, off);
            const int32_t oa = __shfl_xor(at, off);
            if (ob < best || (ob == best && oa < at)) { best = ob; at = oa; }
        }
        if (lane == 0) {
            a.slots[slot].value = best;
            a.slots[slot].device = at;
        }
    }
}

// The smallest CP over the slots, the earliest slot on ties; taken if it is smaller than the
// current one and the sweeps met no device id >= k.
__global__ __launch_bounds__(1024) void step_move_kernel(StepArgs a, uint8_t *assign) {
    __shared__ long long sv[16];
    __shared__ int32_t si[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t len = a.res->len;
    long long v = kNoValue;
    int32_t idx = 0x7fffffff;
    for (int32_t i = tid; i < len; i += 1024) {
        const long long x = a.slots[i].value;
        if (x < v) { v = x; idx = i; }          // i grows, so the first minimum stays
    }
    for (int off = 32; off > 0; off >>= 1) {
        const long long ov = __shfl_xor(v, off);
        const int32_t oi = __shfl_xor(idx, off);
        if (ov < v || (ov == v && oi < idx)) { v = ov; idx = oi; }
    }
    if (lane == 0) { sv[wave] = v; si[wave] = idx; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 16; ++w)
            if (sv[w] < v || (sv[w] == v && si[w] < idx)) { v = sv[w]; idx = si[w]; }
        StepResult &r = *a.res;
        const bool move = r.status[0] == CP_STATUS_OK && r.status[1] == CP_STATUS_OK && v < (long long)r.cp;
        r.moved = move;
        r.best = v;
        if (move) {
            r.vertex = a.path[idx];
            r.device = a.slots[idx].device;
            assign[r.vertex] = (uint8_t)r.device;
        }
    }
}

// ---------------------------------------------------------------- Critical Path strategy (section 3.2.2)

constexpr int kSeedMaxK = 64;        // one lane per device

struct SeedArgs {
    const void *c;            // uint32 or int64 [n]
    const int32_t *path;      // device-free critical path
    const int32_t *len;
    uint8_t *assign;          // [n]
    int32_t n, k, fastest;
    Magic mg[kSeedMaxK];         // where the graph and the speeds have them
    int64_t speed[kSeedMaxK];
};

__global__ void seed_mark_kernel(SeedArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < a.n) a.assign[i] = 0xff;          // not placed yet
}

__global__ void seed_path_kernel(SeedArgs a) {
    const int32_t len = *a.len;
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < len; i += gridDim.x * blockDim.x)
        a.assign[a.path[i]] = (uint8_t)a.fastest;
}

// Minimum over lanes 0 .. span-1 (span a power of two), valid in those lanes: inside a row
// of 16 by register permutations (swap neighbours, swap pairs, mirror 8, mirror 16), across
// rows by shuffles.
__device__ __forceinline__ long long min_over_lanes(long long x, int span) {
    x = min(x, dpp_i64<0xB1>(x));                     // quad_perm 1,0,3,2
    if (span > 2) x = min(x, dpp_i64<0x4E>(x));       // quad_perm 2,3,0,1
    if (span > 4) x = min(x, dpp_i64<0x141>(x));      // row_half_mirror
    if (span > 8) x = min(x, dpp_i64<0x140>(x));      // row_mirror
    if (span > 16) x = min(x, __shfl_xor(x, 16));
    if (span > 32) x = min(x, __shfl_xor(x, 32));
    return x;
}

// The same on 32-bit numbers over the first 16 lanes (WIDE: all 64), every step taken: lanes
// past the devices hold the largest number and never win.
template <bool WIDE>
__device__ __forceinline__ uint32_t min_over_lanes_u32(uint32_t x) {
    x = min(x, dpp_u32<0xB1>(x));
    x = min(x, dpp_u32<0x4E>(x));
    x = min(x, dpp_u32<0x141>(x));
    x = min(x, dpp_u32<0x140>(x));
    if (WIDE) {
        x = min(x, (uint32_t)__shfl_xor((int)x, 16));
        x = min(x, (uint32_t)__shfl_xor((int)x, 32));
    }
    return x;
}

// One batch of up to 64 vertices on relative 32-bit loads (see seed_greedy_kernel): lane j of
// `dev` holds vertex j's device (0xff: not placed yet), of `cv` its c.  No branch but the one
// that skips a placed vertex.
template <bool WIDE>
__device__ __forceinline__ void seed_batch_u32(uint32_t &rel, int32_t &dev, uint32_t cv, int cnt, bool mine,
                                               uint64_t sp, int lane) {
    for (int j = 0; j < cnt; ++j) {
        if (__builtin_amdgcn_readlane(dev, j) != 0xff) continue;            // on the critical path
        const uint32_t cj = (uint32_t)__builtin_amdgcn_readlane((int)cv, j);
        const uint32_t w = (uint32_t)plain_div((uint64_t)cj, sp);
        const uint32_t val = mine ? rel + w : 0xffffffffu;
        const uint32_t best = min_over_lanes_u32<WIDE>(val);
        const int chosen = __ffsll((long long)__ballot(val == best)) - 1;  // lowest device on ties
        rel = lane == chosen ? val : rel;
        dev = lane == j ? chosen : dev;
    }
}

// Barrier that orders LDS only: the global loads of the wavefronts stay in flight across it.
__device__ __forceinline__ void lds_only_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ long long lane0_i64(long long x) {
    return (long long)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)x >> 32)) << 32);
}

// The load rule is a chain: every choice changes the loads the next one sees.  One
// wavefront walks the vertices in order, lane d keeps load(d); 64 vertices are fetched
// at a time and handed round with readlane.  The chain is the wavefront's own instruction
// latency, so a batch of 64 vertices runs on 32-bit numbers where it can: loads relative
// to the smallest one, which stay below 2^32 - 1 through the batch when (largest - smallest
// load) + 64 * (largest c of the batch) does -- an execution time is at most c.  The choices
// are the same, a minimum and its ties do not move when every load loses the same amount.
// (For speeds and costs without multiply-shift constants: seed_keys_kernel places the others.)
template <typename WT>
__global__ __launch_bounds__(64) void seed_greedy_kernel(SeedArgs a) {
    const int lane = threadIdx.x;
    const WT *c = (const WT *)a.c;
    const bool mine = lane < a.k;
    const uint64_t sp = (uint64_t)a.speed[mine ? lane : 0];
    auto cost = [&](uint64_t cv) -> long long { return (long long)plain_div(cv, sp); };
    // the critical path is placed first: its execution times on the fastest device
    long long load = 0;
    {
        const uint64_t sf = (uint64_t)a.speed[a.fastest];
        const int32_t len = *a.len;
        long long part = 0;
        for (int32_t i = lane; i < len; i += 64) part += (long long)plain_div((uint64_t)c[a.path[i]], sf);
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
        if (lane == a.fastest) load = part;
    }
    int span = 1;
    while (span < a.k) span <<= 1;
    for (int32_t v0 = 0; v0 < a.n; v0 += 64) {
        const int32_t v = v0 + lane;
        const uint64_t cv = v < a.n ? (uint64_t)c[v] : 0;
        int32_t dev = v < a.n ? (int32_t)a.assign[v] : 0;      // (lanes past the last vertex: nothing to place)
        const int32_t cnt = min(64, a.n - v0);
        // smallest and largest load, largest c of the batch (the same in every lane)
        const long long low = lane0_i64(min_over_lanes(mine ? load : LLONG_MAX, span));
        const long long high = -lane0_i64(min_over_lanes(mine ? -load : LLONG_MAX, span));
        unsigned long long cmax = cv;
        for (int off = 32; off > 0; off >>= 1) cmax = max(cmax, (unsigned long long)__shfl_xor((long long)cmax, off));
        const bool narrow = cmax < (1ull << 32) && (unsigned long long)(high - low) + 64 * cmax < 0xffffffffull;
        if (narrow) {
            uint32_t rel = mine ? (uint32_t)(load - low) : 0xffffffffu;
            if (span <= 16) seed_batch_u32<false>(rel, dev, (uint32_t)cv, cnt, mine, sp, lane);
            else seed_batch_u32<true>(rel, dev, (uint32_t)cv, cnt, mine, sp, lane);
            if (mine) load = low + (long long)rel;
        } else {
            for (int j = 0; j < cnt; ++j) {
                if (__builtin_amdgcn_readlane(dev, j) != 0xff) continue;
                const uint64_t cj = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)cv, j) |
                                    (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(cv >> 32), j) << 32;
                const long long val = mine ? load + cost(cj) : LLONG_MAX;
                // the devices sit in lanes 0 .. k-1: a reduction over the next power of two covers them
                const long long best = min_over_lanes(val, span);
                const int chosen = __ffsll((long long)__ballot(val == best)) - 1;
                if (lane == chosen) load = val;
                if (lane == j) dev = chosen;
            }
        }
        if (v < a.n) a.assign[v] = (uint8_t)dev;
    }
}

// The same chain where execution times come from multiply-shift constants, with nothing but the chain on the wavefront
// that walks it.  Its numbers are keys, (load - low) << BITS | device, so that a minimum names its device and the
// lowest one wins a tie; every row of 16 lanes holds all devices, PER of them a lane (device r * 16 + lane).  A vertex
// is an addition, four minima over register permutations, a comparison and a selection.  Three wavefronts beside it read c and the
// vertices still to be placed 64 at a time, two batches ahead, put the execution times of every device into
// LDS and write the devices chosen a batch ago.  Where a batch might take a load past 32 - BITS bits above the lowest, its
// loads are 32 bits relative to that without a device number, and past 32 bits they are 64; ties are then told by ballots.
// Bound by that chain, 88 cycles a vertex (the unit's busy cycles over the vertices): 211,000 vertices on 16 devices 0.056 ->
// 0.037 us each, 32 devices 0.046, 50 0.067; c up to 2^26 (32-bit loads) 0.070, 0.094 and 0.15, up to 2^31 (64) 0.30, 0.35 and
// 0.38 (0.32, 0.37 and 0.39 with all of a call's work on one wavefront).  (A branch
// of any kind between two vertices costs as much as half a vertex.  Two vertices at a time, the second one's choice
// prepared for each outcome of the first, or both outcomes' keys added up ahead of the comparison: 4 % less and 4 % more.)
template <int PER, int BITS>
__global__ __launch_bounds__(256) void seed_keys_kernel(SeedArgs a) {
    static_assert(PER << 4 == 1 << BITS, "BITS bits name a device");
    constexpr int kBatch = 64, kCols = 16 * PER;
    constexpr uint32_t kLimit = 0xffffffffu >> BITS, kDevice = (1u << BITS) - 1;
    __shared__ __align__(16) uint32_t times[2 * kBatch + 8][kCols];              // (eight rows are read past the end)
    __shared__ unsigned long long open_of[4];                                    // vertices to be placed, of four batches
    __shared__ uint32_t cmax_of[4], chosen_of[2][16];                            // chosen: four devices a word
    __shared__ Magic mg[kCols];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t *c = (const uint32_t *)a.c;
    const int32_t batches = (a.n + kBatch - 1) / kBatch;
    for (int i = tid; i < (2 * kBatch + 8) * kCols; i += 256) (&times[0][0])[i] = 0;
    if (tid < kCols) mg[tid] = a.mg[tid];
    __syncthreads();
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        const int d = lane & 15;
        long long load[PER], base = 0;
        uint32_t key[PER], bound = 0;        // bound: no key's load is larger
        enum { kKeys, kLoads32, kLoads64 } form = kLoads64;
        {
            // the critical path is placed first: its execution times on the fastest device
            const Magic mf = a.mg[a.fastest];
            const int32_t len = *a.len;
            long long part = 0;
            for (int32_t i = lane; i < len; i += 64) part += (long long)magic_div(c[a.path[i]], mf);
            for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                load[r] = r * 16 + d == a.fastest ? part : 0;
                key[r] = 0xffffffffu;
            }
        }
        auto here = [&](int r) { return r * 16 + d < a.k; };
        auto id = [&](int r) { return (uint32_t)(r * 16 + d); };
        auto min_of_row = [&](uint32_t best) {
            best = min(best, dpp_row<0xB1>(best));
            best = min(best, dpp_row<0x4E>(best));
            best = min(best, dpp_row<0x141>(best));
            return min(best, dpp_row<0x140>(best));
        };
        // the lowest device for which `hit` is true (of one row: all rows are alike)
        auto lowest = [&](auto hit) {
            if constexpr (PER <= 2) {
                uint32_t hits = (uint32_t)__ballot(hit(0)) & 0xffffu;
                if (PER == 2) hits |= (uint32_t)__ballot(hit(PER - 1)) << 16;
                return (uint32_t)(__ffs((int)hits) - 1);
            } else {
                unsigned long long hits = 0;
#pragma unroll
                for (int r = 0; r < PER; ++r) hits |= (unsigned long long)((uint32_t)__ballot(hit(r)) & 0xffffu) << (16 * r);
                return (uint32_t)(__ffsll((long long)hits) - 1);
            }
        };
        // One vertex: its execution times to its device.  In keys: the winner's key.
        auto place_keys = [&](const uint32_t (&w)[PER]) {
            uint32_t val[PER], best = 0;
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                val[r] = (w[r] << BITS) + key[r];
                best = r ? min(best, val[r]) : val[r];
            }
            best = min_of_row(best);
#pragma unroll
            for (int r = 0; r < PER; ++r) key[r] = val[r] == best ? val[r] : key[r];
            return best;
        };
        auto place_32 = [&](const uint32_t (&w)[PER]) {
            uint32_t val[PER], best = 0;
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                val[r] = w[r] + key[r];
                best = r ? min(best, val[r]) : val[r];
            }
            best = min_of_row(best);
            const uint32_t got = lowest([&](int r) { return val[r] == best; });
#pragma unroll
            for (int r = 0; r < PER; ++r) key[r] = id(r) == got ? best : key[r];
            return got;
        };
        auto place_64 = [&](const uint32_t (&w)[PER]) {
            long long val[PER], best = LLONG_MAX;
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                val[r] = here(r) ? load[r] + (long long)w[r] : LLONG_MAX;
                best = val[r] < best ? val[r] : best;
            }
            best = lane0_i64(min_over_lanes(best, 16));
            const uint32_t got = lowest([&](int r) { return val[r] == best; });
#pragma unroll
            for (int r = 0; r < PER; ++r) load[r] = id(r) == got ? best : load[r];
            return got;
        };
        // loads of 64 bits, and from them the shortest form in which a load can grow by `room`
        auto choose_form = [&](unsigned long long room) {
#pragma unroll
            for (int r = 0; r < PER; ++r)
                load[r] = form == kKeys ? base + (long long)(key[r] >> BITS)
                                        : form == kLoads32 ? base + (long long)key[r] : load[r];
            form = kLoads64;
            if (room >= 0xffffffffull) return;
            long long low = LLONG_MAX, high = LLONG_MAX;
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                if (here(r) && load[r] < low) low = load[r];
                if (here(r) && -load[r] < high) high = -load[r];
            }
            low = lane0_i64(min_over_lanes(low, 16));
            high = -lane0_i64(min_over_lanes(high, 16));
            const unsigned long long most = (unsigned long long)(high - low) + room;
            if (most >= 0xffffffffull) return;
            form = most < kLimit ? kKeys : kLoads32;
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                const uint32_t rel = (uint32_t)(load[r] - low);
                key[r] = !here(r) ? 0xffffffffu : form == kKeys ? rel << BITS | id(r) : rel;
            }
            base = low;
            bound = (uint32_t)(high - low);
        };
        lds_only_barrier();                  // the first batch is there
        for (int32_t b = 0; b <= batches; ++b) {
            const uint32_t *row = &times[(b & 1) * kBatch][d * PER];
            uint32_t w[2][8][PER], chosen = 0;
            auto ask = [&](int at, uint32_t (&to)[8][PER]) {
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int r = 0; r < PER; ++r) to[i][r] = row[(at + i) * kCols + r];
            };
            ask(0, w[0]);
            const int cnt = b < batches ? __popcll(open_of[b & 3]) : 0;
            const unsigned long long room =
                (unsigned long long)kBatch * (uint32_t)__builtin_amdgcn_readfirstlane((int)cmax_of[b & 3]);
            // (a shorter form is looked for once a batch, where its numbers could hold the batch at all)
            const bool stays = form == kKeys ? bound + room < kLimit
                               : form == kLoads32 ? room >= kLimit && bound + room < 0xffffffffull : room >= 0xffffffffull;
            if (cnt > 0 && !stays) choose_form(room);
            if (form != kLoads64) bound += cnt > 0 ? (uint32_t)room : 0u;
            // eight vertices after the other without a test between them, all their reads at once (a wait for each would
            // be an instruction for each), then those that are left
            auto place_all = [&](auto place) {
                uint32_t packed[2] = {0, 0};
                int j = 0;
                auto note = [&]() {
                    chosen = lane == j / 4 ? packed[0] : chosen;
                    chosen = lane == j / 4 + 1 ? packed[1] : chosen;
                    j += 8;
                };
                auto eight = [&](const uint32_t (&w)[8][PER]) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) packed[i / 4] = __builtin_amdgcn_alignbit(place(w[i]), packed[i / 4], 8);
                    note();
                };
                while (j + 16 <= cnt) {
                    ask(j + 8, w[1]);
                    eight(w[0]);
                    ask(j + 8, w[0]);
                    eight(w[1]);
                }
                if (j + 8 <= cnt) {
                    ask(j + 8, w[1]);
                    eight(w[0]);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
#pragma unroll
                        for (int r = 0; r < PER; ++r) w[0][i][r] = w[1][i][r];
                }
                if (j < cnt) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        packed[i / 4] = __builtin_amdgcn_alignbit(j + i < cnt ? place(w[0][i]) : 0u, packed[i / 4], 8);
                    note();
                }
            };
            if (form == kKeys) place_all(place_keys);
            else if (form == kLoads32) place_all(place_32);
            else place_all(place_64);
            if (lane < 16) chosen_of[b & 1][lane] = chosen;
            lds_only_barrier();
        }
    } else {
        const int h = wave - 1;
        uint32_t cv[4], dev[4];              // of the batches on their way, two of them asked for but not there yet
        auto fetch = [&](int32_t b, uint32_t &cs, uint32_t &ds) {
            const int32_t v = min(b * kBatch + lane, a.n - 1);
            cs = c[v];
            ds = a.assign[v];
        };
        auto stage = [&](int32_t b, uint32_t cs, uint32_t ds) {
            const bool mine = ds == 0xff && b * kBatch + lane < a.n;
            const unsigned long long open = __ballot(mine);
            uint32_t *row = &times[(b & 1) * kBatch + __popcll(open & ((1ull << lane) - 1))][0];
#pragma unroll
            for (int i = 0; i < (kCols + 2) / 3; ++i) {
                const int d = min(h + 3 * i, a.k - 1);   // (past the last device: its times once more)
                const uint32_t w = magic_div(cs, mg[d]);
                if (mine) row[(d & 15) * PER + (d >> 4)] = w;
            }
            if (h == 0) {
                const uint32_t most = ~min_over_wave(~cs);
                if (lane == 0) {
                    open_of[b & 3] = open;
                    cmax_of[b & 3] = most;
                }
            }
        };
        fetch(0, cv[0], dev[0]);
        stage(0, cv[0], dev[0]);
        fetch(1, cv[1], dev[1]);
        fetch(2, cv[2], dev[2]);
        lds_only_barrier();
        for (int32_t b0 = 0; b0 <= batches; b0 += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int32_t b = b0 + i;
                if (b > batches) break;
                fetch(b + 3, cv[(i + 3) % 4], dev[(i + 3) % 4]);
                if (b + 1 < batches) stage(b + 1, cv[(i + 1) % 4], dev[(i + 1) % 4]);
                if (h == 0 && b >= 1) {
                    const unsigned long long open = open_of[(b - 1) & 3];
                    const uint32_t at = (uint32_t)__popcll(open & ((1ull << lane) - 1));
                    const uint32_t got = chosen_of[(b - 1) & 1][at / 4 & 15] >> (8 * (at % 4)) & kDevice;
                    if (open >> lane & 1) a.assign[(b - 1) * kBatch + lane] = (uint8_t)got;
                }
                lds_only_barrier();
            }
        }
    }
}

struct SearchLayout {
    size_t eval_ws = 0, b = 0, tl = 0, level = 0, over = 0, slot_at = 0, want = 0, mine = 0, slots = 0, path = 0,
           small = 0, total = 0, jumps = 0, chain = 0;
    size_t eval_bytes = 0;
    int rows_over = 1;       // rows of the level-range tables: ranges of 1, 2, 4, ... levels
    int tick = 4;
};

int search_layout(const cp_graph *g, int32_t k, SearchLayout &o) {
    cp_graph_info info;
    int rc = cp_graph_get_info(g, &info);
    if (rc) return rc;
    o.tick = info.min_tick_bytes;
    // one row of outputs is the same in either layout; room for whichever way the call goes
    for (int layout : {CP_OUT_VERTEX_MAJOR, CP_OUT_PARTITION_MAJOR}) {
        size_t ws = 0;
        rc = eval_one_bytes(g, k, layout, o.tick, &ws);
        if (rc) return rc;
        o.eval_bytes = std::max(o.eval_bytes, align_up(ws));
    }
    while ((2ll << (o.rows_over - 1)) <= info.L) ++o.rows_over;
    const size_t n = (size_t)info.n, L = (size_t)std::max(info.L, 1);
    size_t at = 0;
    o.eval_ws = at; at += o.eval_bytes;
    o.b = at;       at += align_up(n * (size_t)o.tick);
    o.tl = at;      at += align_up(n * (size_t)o.tick);
    o.level = at;   at += align_up(n * sizeof(int32_t));
    o.over = at;    at += align_up((size_t)o.rows_over * L * 8);
    o.slot_at = at; at += align_up(L * sizeof(int32_t));
    o.want = at;    at += align_up(L * sizeof(int32_t));
    o.mine = at;    at += align_up(L * sizeof(int32_t));
    o.slots = at;   at += align_up(L * sizeof(SlotBest));
    o.path = at;    at += align_up(L * sizeof(int32_t));
    o.small = at;   at += kAlign;        // StepResult, broken constraints
    o.total = at;           // (the path's jumps and the chain sweep's costs are optional: an array of this size still serves)
    o.jumps = path_by_jumps(info.n, 1, info.L, g->packed.hops) ? align_up(path_jump_words(info.n) * sizeof(int32_t)) : 0;
    o.chain = eval_chain_bytes(g, true);
    return CP_OK;
}

int copy_back(void *host, const void *dev, size_t bytes, hipStream_t st) {
    if (hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, st) != hipSuccess) return CP_ERR_HIP;
    return hipStreamSynchronize(st) == hipSuccess ? CP_OK : CP_ERR_HIP;
}

// Everything of a step behind the path: candidates of all path vertices, the best one applied.
template <typename Tick, typename WT, bool MAGIC>
int launch_step(const StepArgs &a, uint8_t *assign, int64_t num_pairs, const int32_t *pairs, int64_t num_pins,
                const int32_t *pins, hipStream_t st) {
    const dim3 per_vertex((unsigned)((a.n + 255) / 256)), block(256);
    const dim3 per_level((unsigned)std::min(1024, (a.L + 255) / 256));
    hipLaunchKernelGGL(step_path_kernel, per_level, block, 0, st, a);
    hipLaunchKernelGGL((avoid_kernel<Tick, WT, MAGIC>), per_vertex, block, 0, st, a);
    if (a.L <= kOneBlockLevels) {
        hipLaunchKernelGGL(fold_all_kernel, dim3(1), dim3(1024), 0, st, a);
    } else {
        for (int j = a.rows_over - 1; j > 0; --j)
            hipLaunchKernelGGL(fold_row_kernel, dim3((unsigned)((a.L + 255) / 256)), block, 0, st, a, j);
    }
    if (a.constrained) {
        const int64_t most = std::max(num_pairs, num_pins);
        hipLaunchKernelGGL(constraint_kernel, dim3((unsigned)std::min<int64_t>(1024, (most + 255) / 256)), block, 0, st,
                           a, num_pairs, pairs, num_pins, pins);
    }
    hipLaunchKernelGGL((candidate_kernel<Tick, WT, MAGIC>), dim3((unsigned)std::min(a.L, 4096)), dim3(64), 0, st, a);
    hipLaunchKernelGGL(step_move_kernel, dim3(1), dim3(1024), 0, st, a, assign);
    return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_HIP;
}

}  // namespace

}  // namespace cpeval

using namespace cpeval;

extern "C" {

int cp_search_workspace_bytes(const cp_graph *g, int32_t k, int32_t chunk, size_t *out_bytes) {
    if (!g || !out_bytes) return CP_ERR_NULL;
    if (k < 1 || k > 255 || chunk < 1) return CP_ERR_SIZE;
    SearchLayout lay;
    int rc = search_layout(g, k, lay);
    if (rc) return rc;
    *out_bytes = lay.total + lay.jumps + lay.chain;
    return CP_OK;
}

int cp_search(const cp_graph *g, int32_t k, const int64_t *speeds, const int64_t *bandwidth,
              uint8_t *assignment, int64_t num_pairs, const int32_t *pairs, int64_t num_pins,
              const int32_t *pins, int32_t max_moves, int32_t chunk, void *workspace, size_t workspace_bytes,
              void *stream, int64_t *cp_trace, int32_t *moves, int32_t *num_moves, int64_t *evaluated) {
    if (!g || !speeds || !bandwidth || !assignment || !workspace || !cp_trace || !num_moves) return CP_ERR_NULL;
    if (k < 1 || k > 255 || chunk < 1 || max_moves < 0 || num_pairs < 0 || num_pins < 0) return CP_ERR_SIZE;
    if ((num_pairs > 0 && !pairs) || (num_pins > 0 && !pins)) return CP_ERR_NULL;
    SearchLayout lay;
    int rc = search_layout(g, k, lay);
    if (rc) return rc;
    if (((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < lay.total) return CP_ERR_WORKSPACE;
    cp_graph_info info;
    rc = cp_graph_get_info(g, &info);
    if (rc) return rc;
    if (!info.uploaded) return CP_ERR_STATE;
    const Packed &p = g->packed;
    CostTables tabs;
    try {
        rc = build_cost_tables(k, speeds, bandwidth, p.narrow, p.info.max_c, p.info.max_t, tabs);
    } catch (const std::bad_alloc &) {
        rc = CP_ERR_ALLOC;
    }
    if (rc) return rc;
    int plan = CP_PLAN_AUTO;
    rc = cp_eval_choose_plan(g, 1, k, speeds, bandwidth, lay.tick, &plan);
    if (rc) return rc;
    // rows per partition is what the window plans write, rows per vertex what the wave-column plan does
    const int layout = plan == CP_PLAN_WAVE_COLUMN ? CP_OUT_VERTEX_MAJOR : CP_OUT_PARTITION_MAJOR;
    hipStream_t st = (hipStream_t)stream;
    uint8_t *ws = (uint8_t *)workspace;
    const uint8_t *blob = (const uint8_t *)g->device_blob;
    StepArgs a{};
    a.rows_t = (const int4 *)(blob + p.col_t.rows_off);
    a.s_ptr = (const int32_t *)(blob + p.col_b.ptr_off);
    a.s_idx = (const int32_t *)(blob + p.col_b.idx_off);
    a.s_wt = blob + p.col_b.wt_off;
    a.p_ptr = (const int32_t *)(blob + p.col_t.ptr_off);
    a.p_idx = (const int32_t *)(blob + p.col_t.idx_off);
    a.p_wt = blob + p.col_t.wt_off;
    a.c = blob + p.c_off;
    a.assign = assignment;
    a.b = ws + lay.b;
    a.tl = ws + lay.tl;
    a.edge_tab = ws + lay.eval_ws;               // cp_critical_path leaves the call's tables there
    a.vert_tab = ws + lay.eval_ws + 2 * (size_t)k * k * 8;
    a.level = (int32_t *)(ws + lay.level);
    a.slot_at = (int32_t *)(ws + lay.slot_at);
    a.path = (const int32_t *)(ws + lay.path);
    a.over = (unsigned long long *)(ws + lay.over);
    a.want = (int32_t *)(ws + lay.want);
    a.mine = (int32_t *)(ws + lay.mine);
    a.slots = (SlotBest *)(ws + lay.slots);
    a.res = (StepResult *)(ws + lay.small);
    a.broken = (int32_t *)(ws + lay.small + sizeof(StepResult));
    a.n = info.n; a.L = info.L; a.k = k;
    a.rows_over = lay.rows_over;
    a.constrained = num_pairs > 0 || num_pins > 0;
    int32_t *jumps = lay.jumps && workspace_bytes >= lay.total + lay.jumps ? (int32_t *)(ws + lay.total) : nullptr;
    uint8_t *chain = lay.chain && workspace_bytes >= lay.total + lay.jumps + lay.chain ? ws + lay.total + lay.jumps : nullptr;
    const bool stepping = max_moves > 0 && k > 1;
    int32_t done = 0;
    int64_t seen = 0;
    *num_moves = 0;
    if (stepping)
        hipLaunchKernelGGL(level_kernel, dim3((unsigned)((info.n + 255) / 256)), dim3(256), 0, st, a);
    for (;;) {
        // the current partition: CP, both levels, one critical path
        rc = eval_one(g, k, assignment, speeds, bandwidth, ws + lay.eval_ws, lay.eval_bytes, stream, &a.res->cp,
                      ws + lay.b, ws + lay.tl, lay.tick, layout, &a.res->status[0], chain, lay.chain);
        if (rc) return rc;
        rc = critical_path(g, 1, k, assignment, CP_ASSIGN_PARTITION_MAJOR, speeds, bandwidth, ws + lay.b,
                           &a.res->cp, lay.tick, layout, ws + lay.eval_ws, lay.eval_bytes, stream, info.L,
                           (int32_t *)(ws + lay.path), &a.res->len, &a.res->status[1], jumps);
        if (rc) return rc;
        if (stepping) {
            const int64_t cells = (int64_t)a.rows_over * a.L;
            hipLaunchKernelGGL(step_clear_kernel, dim3((unsigned)std::min<int64_t>(4096, (cells + 255) / 256)),
                               dim3(256), 0, st, a);
#define CP_STEP(TICK, WT, MAGIC) rc = launch_step<TICK, WT, MAGIC>(a, assignment, num_pairs, pairs, num_pins, pins, st)
            if (lay.tick == 4) {
                if (tabs.magic_ok) CP_STEP(int32_t, uint32_t, true);
                else if (p.narrow) CP_STEP(int32_t, uint32_t, false);
                else CP_STEP(int32_t, int64_t, false);
            } else {
                if (tabs.magic_ok) CP_STEP(int64_t, uint32_t, true);
                else if (p.narrow) CP_STEP(int64_t, uint32_t, false);
                else CP_STEP(int64_t, int64_t, false);
            }
#undef CP_STEP
            if (rc) return rc;
        }
        StepResult head;
        rc = copy_back(&head, a.res, sizeof(head), st);
        if (rc) return rc;
        if (head.status[0] != CP_STATUS_OK || head.status[1] != CP_STATUS_OK) return CP_ERR_ARG;   // bad device id
        cp_trace[done] = head.cp;
        if (!stepping) break;
        seen += (int64_t)head.len * (k - 1);
        if (!head.moved) break;
        if (moves) {
            moves[2 * done] = head.vertex;
            moves[2 * done + 1] = head.device;
        }
        cp_trace[++done] = head.best;
        if (done >= max_moves) break;
    }
    *num_moves = done;
    if (evaluated) *evaluated = seen;
    return CP_OK;
}

static int seed_bytes(const cp_graph *g, size_t *out_bytes, size_t *jump_bytes, size_t *chain_bytes) {
    if (!g || !out_bytes) return CP_ERR_NULL;
    cp_graph_info info;
    int rc = cp_graph_get_info(g, &info);
    if (rc) return rc;
    size_t eval = 0;
    rc = eval_one_bytes(g, 1, CP_OUT_VERTEX_MAJOR, info.min_tick_bytes, &eval);
    if (rc) return rc;
    *out_bytes = align_up(eval) + align_up((size_t)info.n) + align_up((size_t)info.n * (size_t)info.min_tick_bytes) +
                 align_up((size_t)info.L * sizeof(int32_t)) + kAlign;
    *jump_bytes = path_by_jumps(info.n, 1, info.L, g->packed.hops) ? align_up(path_jump_words(info.n) * sizeof(int32_t)) : 0;
    *chain_bytes = eval_chain_bytes(g, false);
    return CP_OK;
}

int cp_seed_workspace_bytes(const cp_graph *g, size_t *out_bytes) {
    size_t jump_bytes = 0, chain_bytes = 0;
    const int rc = seed_bytes(g, out_bytes, &jump_bytes, &chain_bytes);
    if (rc == CP_OK) *out_bytes += jump_bytes + chain_bytes;
    return rc;
}

int cp_seed_partition(const cp_graph *g, int32_t k, const int64_t *speeds, void *workspace, size_t workspace_bytes,
                      void *stream, uint8_t *assignment_out, int32_t *status_out) {
    if (!g || !speeds || !workspace || !assignment_out || !status_out) return CP_ERR_NULL;
    if (k < 1 || k > kSeedMaxK) return CP_ERR_SIZE;
    size_t need = 0, jump_bytes = 0, chain_bytes = 0;        // (only `need` bytes are asked for)
    int rc = seed_bytes(g, &need, &jump_bytes, &chain_bytes);
    if (rc) return rc;
    if (((uintptr_t)workspace % kAlign) != 0 || workspace_bytes < need) return CP_ERR_WORKSPACE;
    cp_graph_info info;
    rc = cp_graph_get_info(g, &info);
    if (rc) return rc;
    if (!info.uploaded) return CP_ERR_STATE;
    const Packed &p = g->packed;
    std::vector<int64_t> ones((size_t)k * k, 1);
    CostTables tabs;
    try {
        rc = build_cost_tables(k, speeds, ones.data(), p.narrow, p.info.max_c, p.info.max_t, tabs);
    } catch (const std::bad_alloc &) {
        rc = CP_ERR_ALLOC;
    }
    if (rc) return rc;
    size_t eval = 0;
    rc = eval_one_bytes(g, 1, CP_OUT_VERTEX_MAJOR, info.min_tick_bytes, &eval);
    if (rc) return rc;
    const size_t n = (size_t)info.n;
    const int T = info.min_tick_bytes;
    uint8_t *ws = (uint8_t *)workspace;
    uint8_t *d_one = ws + align_up(eval);
    void *d_b = d_one + align_up(n);
    int32_t *d_path = (int32_t *)((uint8_t *)d_b + align_up(n * (size_t)T));
    uint8_t *d_small = (uint8_t *)d_path + align_up((size_t)info.L * sizeof(int32_t));
    int64_t *d_cp = (int64_t *)d_small;
    int32_t *d_len = (int32_t *)(d_small + 8);
    hipStream_t st = (hipStream_t)stream;
    // the ranks know no devices: one device of speed 1, nothing is transferred
    rc = launch_zero_bytes(d_one, (int64_t)n, stream);
    if (rc) return rc;
    const int64_t unit = 1;
    uint8_t *chain = chain_bytes && workspace_bytes >= need + jump_bytes + chain_bytes ? ws + need + jump_bytes : nullptr;
    rc = eval_one(g, 1, d_one, &unit, &unit, ws, align_up(eval), stream, d_cp, d_b, nullptr, T, CP_OUT_VERTEX_MAJOR,
                  status_out, chain, chain_bytes);
    if (rc) return rc;
    int32_t *jumps = jump_bytes && workspace_bytes >= need + jump_bytes ? (int32_t *)(ws + need) : nullptr;
    rc = critical_path(g, 1, 1, d_one, CP_ASSIGN_PARTITION_MAJOR, &unit, &unit, d_b, d_cp, T, CP_OUT_VERTEX_MAJOR, ws,
                       align_up(eval), stream, info.L, d_path, d_len, status_out, jumps);
    if (rc) return rc;
    SeedArgs a{};
    a.c = (const uint8_t *)g->device_blob + p.c_off;
    a.path = d_path;
    a.len = d_len;
    a.assign = assignment_out;
    a.n = info.n;
    a.k = k;
    a.fastest = 0;
    for (int d = 1; d < k; ++d)
        if (speeds[d] > speeds[a.fastest]) a.fastest = d;
    for (int d = 0; d < k; ++d) {
        a.mg[d] = tabs.magic[2 * (size_t)k * k + d];
        a.speed[d] = speeds[d];
    }
    hipLaunchKernelGGL(seed_mark_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
    hipLaunchKernelGGL(seed_path_kernel, dim3(64), dim3(256), 0, st, a);
    // (16 devices a register of the chain's wavefront)
    if (tabs.magic_ok && k <= 16) hipLaunchKernelGGL((seed_keys_kernel<1, 4>), dim3(1), dim3(256), 0, st, a);
    else if (tabs.magic_ok && k <= 32) hipLaunchKernelGGL((seed_keys_kernel<2, 5>), dim3(1), dim3(256), 0, st, a);
    else if (tabs.magic_ok) hipLaunchKernelGGL((seed_keys_kernel<4, 6>), dim3(1), dim3(256), 0, st, a);
    else if (p.narrow) hipLaunchKernelGGL(seed_greedy_kernel<uint32_t>, dim3(1), dim3(64), 0, st, a);
    else hipLaunchKernelGGL(seed_greedy_kernel<int64_t>, dim3(1), dim3(64), 0, st, a);
    return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_HIP;
}

}  // extern "C"
