// Whole-graph sweep: a call on a small graph in one launch.
//
// Under the lane-window plan a call is four launches (tables, device ids by group, sweeps, mask), and on graphs of some
// thousand vertices the launches take longer than the sweeps.  Where the values of all vertices fit LDS for both sweeps side
// by side, one workgroup of 4 or 8 consecutive partitions does everything: it reads its partitions' ids as they are, takes the cost
// tables from the kernel's arguments, walks both sweeps tick by tick (half of its wavefronts each), and writes
// outputs and mask from LDS, along the rows that the caller asked for.
//
// A ring word is value << 6 | device id as in the lane-window plan, at row v of the sweep's array, so nothing is ever
// overwritten and no vertex is far.  Lanes: G partitions x 64 / G units; a unit is up to four edges of a vertex, read from the
// graph's stream four ticks ahead (the lanes of a partition group share the load), and vertices of several units meet in an
// LDS maximum.  The word and the execution time of a unit's own vertex are looked up a tick ahead.
//
// Whole calls, the lane-window plan -> this one: 64 vertices in 8 levels, 16 partitions 26 -> 12 us (the launch 6.4 of them);
// 2,016 in 195 levels, 1,024 and 4,096 partitions 106 -> 62 and 390 -> 138; 1,400 in 112, 1,024 partitions 71 -> 40.
// Bound by the chain of a tick, 0.27 us: two LDS round trips, the maximum, a barrier, and some 75 vector instructions of a
// wavefront that has its SIMD for itself; with more than four wavefronts on a compute unit by their issue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "device_math.hpp"
#include "launch.hpp"

namespace cpeval {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct WholeArgs {
    const u32x4 *units[2];     // [ticks][units][2] of either sweep, see WholeDir
    void *out[2];              // b, tl: ticks of (v, q) at v * out_sv + q * out_sq, or NULL
    int64_t out_sv, out_sq;
    int64_t *cp_out;
    uint64_t *mask;
    int32_t *status;
    const uint8_t *assign;
    int64_t a_sp, a_sv;
    const uint32_t *c;
    const void *edge_tab, *vert_tab;         // where they are not among the arguments
    int32_t n, P, k, ticks, units_a_tick, out64, by_partition, sweeps;
    int32_t check_all;         // workgroup 0 looks at all ids and writes the status; else it has been cleared
};

// Edge entries by (own device, neighbour) of the b sweep, then the vertices'.
struct alignas(8) WholeTable { uint32_t v[kWholeTableWords]; };
struct NoTable {};

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename Word, int G, typename Tab, typename Table>
__global__ __launch_bounds__(1024) void whole_kernel(WholeArgs a, Table table) {
    constexpr int S = G + 1, kAhead = kWholeAhead, RPW = 64 / G;
    constexpr uint32_t ID = (1u << kLaneIdBits) - 1, kWord = sizeof(Word);
    extern __shared__ uint4 lds16[];
    __shared__ unsigned long long red[G];
    __shared__ int32_t any_bad;
    const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x, n = a.n, k = a.k;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = nt / 64;
    const int32_t q0 = blockIdx.x * G, live = min(G, a.P - q0);
    const int per_sweep = a.sweeps == 3 ? nt / 2 : nt;
    const bool second = a.sweeps == 3 ? tid >= per_sweep : a.sweeps == 2;
    const size_t ring_words = (size_t)(n + 2) * S;
    Word *const rings = (Word *)lds16;
    Word *const ring_b = rings, *const ring_t = rings + (a.sweeps == 3 ? ring_words : 0);
    Tab *const tabs = (Tab *)(rings + (((a.sweeps == 3 ? 2 : 1) * ring_words + 1) & ~(size_t)1));
    const int kk = k * k;

    // tables: the b sweep's, the same transposed for the t sweep, the vertices'
    {
        const Tab *edges = (const Tab *)a.edge_tab, *verts = (const Tab *)a.vert_tab;
        if constexpr (std::is_same_v<Table, WholeTable>) {
            edges = (const Tab *)table.v;
            verts = edges + kk;
        }
        for (int i = tid; i < kk; i += nt) {
            const Tab x = edges[i];
            tabs[i] = x;
            tabs[kk + i % k * k + i / k] = x;
        }
        for (int i = tid; i < k; i += nt) tabs[2 * kk + i] = verts[i];
    }
    if (tid < G) red[tid] = 0;
    if (tid == 0) any_bad = 0;
    for (int i = tid; i < 2 * S; i += nt) {
        ring_b[(size_t)n * S + i] = 0;
        ring_t[(size_t)n * S + i] = 0;
    }
    // device ids
    bool bad = false;
    constexpr int kAtOnce = 4;               // vertices a lane asks for together: a round trip for each would add up
    for (int v0 = tid; v0 < n; v0 += kAtOnce * nt) {
        uint32_t d[kAtOnce][G];
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i)
#pragma unroll
            for (int g = 0; g < G; ++g)
                d[i][g] = a.assign[(int64_t)min(q0 + g, a.P - 1) * a.a_sp + (int64_t)min(v0 + i * nt, n - 1) * a.a_sv];
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i)
#pragma unroll
            for (int g = 0; g < G; ++g) {
                bad |= d[i][g] >= (uint32_t)k;
                const Word x = (Word)min(d[i][g], (uint32_t)k - 1);
                const size_t row = (size_t)min(v0 + i * nt, n - 1) * S + g;      // (the last one once more past the end)
                ring_b[row] = x;
                ring_t[row] = x;
            }
    }
    if (a.check_all && blockIdx.x == 0) {
        const int32_t bytes = n * a.P;
        const u32x4 *all = (const u32x4 *)a.assign;
        for (int i = tid; i < bytes / 16; i += nt) {
            const u32x4 x = all[i];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int h = 0; h < 4; ++h) bad |= (x[j] >> (8 * h) & 0xffu) >= (uint32_t)k;
        }
        for (int i = bytes / 16 * 16 + tid; i < bytes; i += nt) bad |= a.assign[i] >= (uint32_t)k;
    }

    const Tab base = round_up(Tab());        // (no variable divisions behind this)
    // this lane's unit of a tick
    const int t_lane = second && a.sweeps == 3 ? tid - per_sweep : tid, g = lane % G, unit = t_lane / G;
    const Tab *const etab = tabs + (second ? kk : 0), *const vtab = tabs + 2 * kk;
    char *const ring = (char *)(second ? ring_t : ring_b);
    const u32x4 *stream = a.units[second ? 1 : 0] + 2 * unit;
    u32x4 from[kAhead], wt[kAhead];
    auto load = [&](int r) {
        from[r] = stream[0];
        wt[r] = stream[1];
        stream += 2 * a.units_a_tick;
    };
#pragma unroll
    for (int r = 0; r < kAhead; ++r) {
        load(r);
        __builtin_amdgcn_sched_barrier(0);   // (the waits count loads in the order of the loop)
    }
    auto at = [&](uint32_t row) { return (Word *)(ring + __umul24(row, S * kWord) + (uint32_t)g * kWord); };
    lds_barrier();
    if (bad) any_bad = 1;

    // Places of a tick's words; the id of a unit's own vertex, known a tick ahead, gives its row of the table and its w.
    Word *near[4], *mine, best = 0;
    const Tab *erow;
    Word own;
    auto places = [&](const u32x4 &x) {
        near[0] = at(x.x & 0xffffu);
        near[1] = at(x.x >> 16);
        near[2] = at(x.y & 0xffffu);
        near[3] = at(x.y >> 16);
        mine = at(x.z);
    };
    auto vertex = [&](uint32_t id, uint32_t c, Tab m) {
        erow = etab + __umul24(id, (uint32_t)k);
        own = add_quotient((Word)id, c, m, base);
    };
    {
        places(from[0]);
        const uint32_t id = (uint32_t)*mine & ID;
        vertex(id, from[0].w, vtab[id]);
    }
    for (int t0 = 0; t0 < a.ticks; t0 += kAhead) {
#pragma unroll
        for (int r = 0; r < kAhead; ++r) {
            const u32x4 next = from[(r + 1) % kAhead];
            Word v[4];
            Tab m[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = *near[j];
            const Word next_own = *at(next.z);
#pragma unroll
            for (int j = 0; j < 4; ++j) m[j] = erow[(uint32_t)v[j] & ID];
            const uint32_t next_id = (uint32_t)next_own & ID;
            const Tab next_m = vtab[next_id];
            Word acc = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = max(acc, add_quotient(v[j], wt[r][j], m[j], base));
            const Word fin = (acc & ~(Word)ID) + own;
            atomicMax(mine, fin);
            __builtin_amdgcn_sched_barrier(0);       // (nothing in front of what the next tick waits for)
            best = max(best, fin);
            load(r);
            places(next);
            vertex(next_id, next.w, next_m);
            lds_barrier();
        }
    }
    if (!second && a.sweeps != 2) atomicMax(&red[g], (unsigned long long)(best >> kLaneIdBits));
    lds_barrier();
    if (tid < live && a.cp_out) a.cp_out[q0 + tid] = (int64_t)red[tid];
    if (tid == 0) {
        if (a.check_all) {
            if (blockIdx.x == 0) *a.status = any_bad ? CP_STATUS_BAD_DEVICE_ID : CP_STATUS_OK;
        } else if (any_bad) {
            *a.status = CP_STATUS_BAD_DEVICE_ID;
        }
    }

    // outputs
    const Word *ids = a.sweeps == 2 ? ring_t : ring_b;
    auto put = [&](int32_t v, uint32_t c, int gl, bool there) {
        const int64_t to = (int64_t)v * a.out_sv + (int64_t)(q0 + gl) * a.out_sq;
        const size_t row = (size_t)v * S + gl;
        Word b = 0, tl = 0;
        if (a.sweeps != 2) b = ring_b[row] >> kLaneIdBits;
        if (a.sweeps != 1) tl = (ring_t[row] >> kLaneIdBits) - (Word)inverse_div(c, vtab[(uint32_t)ids[row] & ID], base);
        if (there) {
            if (a.out64) {
                if (a.out[0]) ((int64_t *)a.out[0])[to] = (int64_t)b;
                if (a.out[1]) ((int64_t *)a.out[1])[to] = (int64_t)tl;
            } else {
                if (a.out[0]) ((int32_t *)a.out[0])[to] = (int32_t)b;
                if (a.out[1]) ((int32_t *)a.out[1])[to] = (int32_t)tl;
            }
        }
        return __ballot(there && (unsigned long long)(b + tl) == red[gl]);
    };
    if (a.by_partition) {
        const size_t words = ((size_t)n + 63) / 64;
        const int parts = max(1, waves / G), step = parts * 64;      // (more wavefronts than partitions share a row)
        for (int gl = wave % G; gl < live && wave < parts * G; gl += waves)
            for (int32_t v0 = wave / G * 64; v0 < n; v0 += kAtOnce * step) {
                uint32_t c[kAtOnce];
#pragma unroll
                for (int i = 0; i < kAtOnce; ++i) c[i] = a.c[min(v0 + i * step + lane, n - 1)];
#pragma unroll
                for (int i = 0; i < kAtOnce; ++i) {
                    const int32_t first = v0 + i * step, v = first + lane;
                    const unsigned long long bits = put(min(v, n - 1), c[i], gl, v < n);
                    if (a.mask && lane == 0 && first < n) a.mask[(size_t)(q0 + gl) * words + first / 64] = bits;
                }
            }
    } else {
        const size_t words = ((size_t)a.P + 63) / 64;
        const bool final = q0 + G >= a.P;                    // (its bytes and those behind them, up to the word's end)
        const int step = waves * RPW;
        for (int32_t v0 = wave * RPW + lane / G; v0 - lane / G < n; v0 += kAtOnce * step) {
            uint32_t c[kAtOnce];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) c[i] = a.c[min(v0 + i * step, n - 1)];
#pragma unroll
            for (int i = 0; i < kAtOnce; ++i) {
                const int32_t v = v0 + i * step;
                const unsigned long long bits = put(min(v, n - 1), c[i], g, v < n && g < live);
                if (a.mask && v < n) {                       // (G = 8: a byte a vertex)
                    const size_t byte = (size_t)q0 / 8 + (size_t)g;
                    const uint8_t x = g == 0 ? (uint8_t)(bits >> (lane & ~7)) : 0;
                    if (g == 0 || (final && byte < words * 8)) ((uint8_t *)a.mask)[(size_t)v * words * 8 + byte] = x;
                }
            }
        }
    }
}

template <typename Word, typename Tab, typename Table>
int launch_whole_k(const WholeArgs &a, const Table &table, const WholeCfg &cfg, hipStream_t st) {
    const auto kernel = cfg.groups == 8 ? whole_kernel<Word, 8, Tab, Table> : whole_kernel<Word, 4, Tab, Table>;
    if (cfg.lds_bytes > 64 * 1024 && hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                         (int)cfg.lds_bytes) != hipSuccess)
        return CP_ERR_HIP;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((a.P + cfg.groups - 1) / cfg.groups)), dim3((unsigned)cfg.threads),
                       cfg.lds_bytes, st, a, table);
    return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_HIP;
}

template <typename Table>
int launch_whole_t(const WholeArgs &a, const Table &table, const WholeCfg &cfg, hipStream_t st) {
    if (cfg.word == 8)
        return cfg.floats ? launch_whole_k<unsigned long long, float>(a, table, cfg, st)
                          : launch_whole_k<unsigned long long, double>(a, table, cfg, st);
    return cfg.floats ? launch_whole_k<uint32_t, float>(a, table, cfg, st) : launch_whole_k<uint32_t, double>(a, table, cfg, st);
}

}  // namespace

bool whole_config(const WholeDir &d, int32_t n, int32_t k, int groups, int word_bytes, bool floats, int sweeps,
                  size_t lds_limit, WholeCfg &out) {
    const size_t entry_bytes = floats ? 4 : 8;
    out.groups = groups;
    out.word = word_bytes;
    out.floats = floats;
    out.table_bytes = ((size_t)k * k + k) * entry_bytes;
    const size_t ring = (size_t)(n + 2) * (groups + 1);
    out.lds_bytes = align_up(((sweeps * ring + 1) & ~(size_t)1) * word_bytes + ((size_t)2 * k * k + k) * entry_bytes, 16);
    const int per_sweep = d.units_a_tick * groups;
    out.threads = per_sweep * sweeps;
    return per_sweep % kWave == 0 && out.threads <= 1024 && out.lds_bytes + 256 <= lds_limit;
}

int launch_whole(const SweepLaunch &sb, const SweepLaunch &st, const WholeDir &d, const WholeCfg &cfg, bool want_b,
                 bool want_t, bool by_partition, const void *table, bool check_all, void *stream) {
    WholeArgs a{};
    a.units[0] = (const u32x4 *)(sb.blob + d.units_b);
    a.units[1] = (const u32x4 *)(sb.blob + d.units_t);
    a.out[0] = sb.val;
    a.out[1] = st.val;
    a.out_sv = sb.out_sv;
    a.out_sq = sb.out_sq;
    a.cp_out = sb.cp_out;
    a.mask = sb.mask_out;
    a.status = sb.status;
    a.assign = sb.assign;
    a.a_sp = sb.a_stride_p;
    a.a_sv = sb.a_stride_v;
    a.c = (const uint32_t *)(sb.blob + sb.c_off);
    a.n = sb.n;
    a.P = sb.P;
    a.k = sb.k;
    a.ticks = d.ticks;
    a.units_a_tick = d.units_a_tick;
    a.out64 = sb.tick_bytes == 8;
    a.sweeps = (want_b ? 1 : 0) | (want_t ? 2 : 0);
    a.check_all = check_all;
    a.by_partition = by_partition;
    a.edge_tab = cfg.floats ? (const void *)sb.edge_tab4 : sb.edge_tab;
    a.vert_tab = cfg.floats ? (const void *)sb.vert_tab4 : sb.vert_tab;
    if (!table) return launch_whole_t(a, NoTable{}, cfg, (hipStream_t)stream);
    WholeTable args;
    std::memcpy(args.v, table, cfg.table_bytes);
    return launch_whole_t(a, args, cfg, (hipStream_t)stream);
}

}  // namespace cpeval
