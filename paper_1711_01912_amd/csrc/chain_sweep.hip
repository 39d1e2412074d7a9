// Chain sweep: both sweeps of a handful of partitions, each by one workgroup that does nothing but the chain.
//
// One partition of a deep graph is a chain of levels, and the window plans put everything a level needs on it or
// beside it in the same workgroup: packet, device ids, cost tables, division.  With a few partitions the rest of the GPU is
// idle meanwhile.  Here a first launch on the whole GPU writes what every edge and vertex costs under every
// partition (chain_cost_kernel), and the second walks the levels with what is left of a relaxation: an addition and a
// maximum.  A lane takes four edges of a vertex, read as one record of ring slots (the graph's, packed by
// cp_graph_create) and one of costs (the partition's), eight ticks ahead into registers.
//
//   ring      w(v) + max over v's edges of (ring value of the neighbour + cost), by position in sweep order modulo R;
//             that is b in the b sweep and tl + w in the t sweep, whose output takes w off again.  w is part of the
//             costs, so that what a tick adds is one number an edge
//   tick      four ring reads, four additions, maxima (over the lanes of a row by register permutations, one step for
//             up to 8 edges, 16, 32, 64), one ring write, barrier; beside it the last tick's outputs are stored
//
// Costs take 18 or 36 bytes a lane of a tick and partition for both sweeps; where there is room for fewer partitions' than the
// call has, it goes in rounds over one block of them.
//
// R covers the largest distance of an edge in positions and two ticks, so a slot is written after its last reader.  Both sweeps of
// a call run side by side.  Whole calls, the plan before -> this one, one and 32 partitions: 211,000 vertices in 1,000 levels 799
// -> 223 us and 803 -> 484 (rows per vertex 1,486 -> 241, 1,485 -> 710), 121,000 in 701 levels 503 -> 139 and 508 -> 257,
// 19,800 in 660 levels 725 -> 105 and 691 -> 133, 18,000 in 300 levels with 64-bit ticks 219 -> 76 and 228 -> 106.
// Bound by the chain of a tick: 0.11 us with one wavefront, 0.2 with five, of which an LDS round trip, the instructions
// of the wavefront with the most lanes a row and the barrier are about a third each; from 16 wavefronts on by the 24 bytes a lane
// that pass the L1 (with 48, ring slots as byte offsets of 32 bits and costs of 32, 300 levels of 600 vertices took 149 us,
// 112 with these, and 1,500 levels of 20, which save the unpacking, 175 and 191).  With 16 partitions or more
// chain_cost_kernel takes over, by its gathers of device ids.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_math.hpp"
#include "launch.hpp"

namespace cpeval {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct ChainArgs {
    const u32x4 *units;        // [ticks][width], see ChainDir
    const uint2 *edges;        // [ticks][width]
    const int32_t *idx;        // CSR in the sweep's direction
    const uint32_t *wt;
    const void *edge_tab;
    void *cost;                // [P][ticks][width] four of a lane's edges, w of its vertex included; 16 bits each or 32
    void *w;                   // [P][ticks][width] the same bits, t sweep only
    void *out;                 // ticks of (v, q) at v * out_sv + q * out_sq, or NULL
    int64_t out_sv, out_sq;
    int64_t *cp_out;           // [P] or NULL
    int32_t ticks, slots;      // ticks: kChainAhead of them empty, behind the last one
};

struct ChainShape {
    const uint8_t *assign;
    int64_t a_sp, a_sv;
    const uint32_t *c;
    const void *vert_tab;
    int32_t *status;
    int32_t n, P, k, width, sweeps;
};

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int CTRL>
__device__ __forceinline__ uint32_t lane_of(uint32_t x) { return dpp_row<CTRL>(x); }
template <int CTRL>
__device__ __forceinline__ unsigned long long lane_of(unsigned long long x) {
    return (unsigned long long)dpp_row<CTRL>((uint32_t)(x >> 32)) << 32 | dpp_row<CTRL>((uint32_t)x);
}

// Byte offset of the ring slot in the upper or lower half of a word.
template <int HALF, uint32_t SHIFT>
__device__ __forceinline__ uint32_t word_at(uint32_t x) {
    uint32_t off;
    if constexpr (HALF == 0)
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
            : "=v"(off) : "v"(SHIFT), "v"(x));
    else
        asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
            : "=v"(off) : "v"(SHIFT), "v"(x));
    return off;
}

// What a partition's edges and vertices cost, a thread per unit.
template <bool MAGIC, bool C16>
__global__ __launch_bounds__(256) void chain_cost_kernel(ChainArgs b, ChainArgs t, ChainShape sh) {
    const bool second = sh.sweeps == 3 ? blockIdx.z != 0 : sh.sweeps == 2;
    const ChainArgs &a = second ? t : b;
    const uint32_t all = (uint32_t)a.ticks * (uint32_t)sh.width, i = blockIdx.x * 256 + threadIdx.x;
    if (i >= all) return;
    const uint2 from = a.edges[i];
    const uint32_t v = from.y & 0x7fffffffu;
    u32x4 cost = {0, 0, 0, 0};
    uint32_t own = 0;
    if (v < (uint32_t)sh.n) {
        const u32x4 u = a.units[i];
        const uint32_t from_slot[4] = {u.x & 0xffffu, u.x >> 16, u.y & 0xffffu, u.y >> 16};
        const uint8_t *ids = sh.assign + (int64_t)blockIdx.y * sh.a_sp;
        uint32_t d = ids[(int64_t)v * sh.a_sv];
        const uint32_t cv = from.y >> 31 ? 0 : sh.c[v];
        uint32_t at[4], wt[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            const bool there = from_slot[j] != (uint32_t)a.slots && !(from.x >> 31);
            at[j] = there ? ids[(int64_t)a.idx[from.x + j] * sh.a_sv] : 0;
            wt[j] = there ? a.wt[from.x + j] : 0;
        }
        if (d >= (uint32_t)sh.k) {
            *sh.status = CP_STATUS_BAD_DEVICE_ID;
            d = (uint32_t)sh.k - 1;
        }
        auto div = [&](uint32_t x, const void *tab, uint32_t row) {
            return MAGIC ? magic_div(x, ((const Magic *)tab)[row])
                         : (uint32_t)plain_div(x, (uint64_t)((const int64_t *)tab)[row]);
        };
        own = div(cv, sh.vert_tab, d);
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)             // (an edge that is not there: t = 0, which costs nothing)
            cost[j] = own + div(wt[j], a.edge_tab, d * (uint32_t)sh.k + min(at[j], (uint32_t)sh.k - 1));
    }
    const size_t to = (size_t)blockIdx.y * all + i;
    if constexpr (C16) {
        ((u32x2 *)a.cost)[to] = u32x2{cost.x | cost.y << 16, cost.z | cost.w << 16};
        if (second) ((uint16_t *)a.w)[to] = (uint16_t)own;
    } else {
        ((u32x4 *)a.cost)[to] = cost;
        if (second) ((uint32_t *)a.w)[to] = own;
    }
}

template <typename Word, bool T64, bool ONE, bool C16, bool TSWEEP>
__device__ __forceinline__ void chain_sweep(const ChainArgs &a, const ChainShape &sh, int32_t q) {
    constexpr int kAhead = kChainAhead;
    constexpr uint32_t kShift = sizeof(Word) == 8 ? 3 : 2, kTick = T64 ? 8 : 4, kNowhere = 0xffffffffu;
    const uint32_t tid = threadIdx.x, width = (uint32_t)sh.width;
    const uint32_t words = (uint32_t)a.slots + 1 + kWave;
    // (the kernel's LDS is the launch's alone, so that a byte offset is an address)
    typedef __attribute__((address_space(3))) Word LdsWord;
    auto at = [](uint32_t off) { return (LdsWord *)(uintptr_t)off; };
    for (uint32_t i = tid; i < words; i += width) *at(i << kShift) = 0;
    // (a single wavefront's LDS accesses are carried out in their order)
    auto tick_barrier = []() {
        if constexpr (ONE) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            __builtin_amdgcn_wave_barrier();
        } else {
            lds_barrier();
        }
    };
    // Buffer accesses: streams read at an offset that only the scalar unit moves, and stores that are not to be made sent past
    // the end, where the hardware drops them (a branch around them would leave the number of stores in flight open, and the
    // waits for loads would have to assume none).
    const size_t per = (size_t)a.ticks * width;
    const auto buffer = [](const void *base, uint32_t bytes) {
        return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000);
    };
    constexpr uint32_t kCost = C16 ? 8 : 16, kW = kCost / 4;
    const __amdgpu_buffer_rsrc_t units = buffer(a.units, (uint32_t)(per * 16)),
                                 costs = buffer((uint8_t *)a.cost + (size_t)q * per * kCost, (uint32_t)(per * kCost)),
                                 ws = buffer((uint8_t *)a.w + (TSWEEP ? (size_t)q * per * kW : 0), TSWEEP ? (uint32_t)(per * kW) : 0);
    const uint32_t sv = (uint32_t)a.out_sv * kTick;
    const __amdgpu_buffer_rsrc_t rows =
        buffer((uint8_t *)a.out + (a.out ? (int64_t)q * a.out_sq * kTick : 0), a.out ? (uint32_t)(sh.n - 1) * sv + kTick : 0);

    typedef std::conditional_t<C16, u32x2, u32x4> Cost;
    u32x4 unit[kAhead];
    Cost cost[kAhead];
    uint32_t w[kAhead], next = 0;                    // next: first lane of the tick to be read next
    auto load = [&](int r) {
        unit[r] = __builtin_amdgcn_raw_buffer_load_b128(units, (int)(tid * 16), (int)(next * 16), 0);
        if constexpr (C16) cost[r] = __builtin_amdgcn_raw_buffer_load_b64(costs, (int)(tid * 8), (int)(next * 8), 0);
        else cost[r] = __builtin_amdgcn_raw_buffer_load_b128(costs, (int)(tid * 16), (int)(next * 16), 0);
        if constexpr (TSWEEP) {
            if constexpr (C16) w[r] = __builtin_amdgcn_raw_buffer_load_b16(ws, (int)(tid * 2), (int)(next * 2), 0);
            else w[r] = __builtin_amdgcn_raw_buffer_load_b32(ws, (int)(tid * 4), (int)(next * 4), 0);
        }
        next += width;
        __builtin_amdgcn_sched_barrier(0);           // (the waits count loads in the order of the loop)
    };
    uint32_t from[4], mine;                          // of the tick at hand: its neighbours' places in LDS, its row's
    auto unpack = [&](const u32x4 &x) {
        from[0] = word_at<0, kShift>(x.x);
        from[1] = word_at<1, kShift>(x.x);
        from[2] = word_at<0, kShift>(x.y);
        from[3] = word_at<1, kShift>(x.y);
        mine = word_at<0, kShift>(x.z);
    };
#pragma unroll
    for (int r = 0; r < kAhead; ++r) load(r);
    unpack(unit[0]);
    uint32_t put_at = kNowhere;                      // output of the last tick
    Word put = 0, best = 0;
    const int T = a.ticks - kAhead;
    tick_barrier();
    for (int t0 = 0; t0 < T; t0 += kAhead) {
#pragma unroll
        for (int r = 0; r < kAhead; ++r) {
            const Word v0 = *at(from[0]), v1 = *at(from[1]), v2 = *at(from[2]), v3 = *at(from[3]);
            if constexpr (T64) {
                const u32x2 two = {(uint32_t)put, (uint32_t)((uint64_t)put >> 32)};
                __builtin_amdgcn_raw_buffer_store_b64(two, rows, (int)put_at, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32((uint32_t)put, rows, (int)put_at, 0, 0);
            }
            Word x;
            if constexpr (C16)
                x = max(max(v0 + (Word)(cost[r].x & 0xffffu), v1 + (Word)(cost[r].x >> 16)),
                        max(v2 + (Word)(cost[r].y & 0xffffu), v3 + (Word)(cost[r].y >> 16)));
            else
                x = max(max(v0 + (Word)cost[r].x, v1 + (Word)cost[r].y), max(v2 + (Word)cost[r].z, v3 + (Word)cost[r].w));
            // log2 of its row's lanes, and of the widest row's in the wavefront
            const uint32_t lanes = unit[r].z >> 16 & 0xfu;
            const uint32_t steps = (uint32_t)__builtin_amdgcn_readfirstlane((int)unit[r].z) >> 20;
            if (steps) {
                auto fold = [&](Word y, uint32_t step) { x = lanes > step ? max(x, y) : x; };
                fold(lane_of<0xB1>(x), 0);
                if (steps > 1) {
                    fold(lane_of<0x4E>(x), 1);
                    if (steps > 2) {
                        fold(lane_of<0x141>(x), 2);
                        if (steps > 3) fold(lane_of<0x140>(x), 3);
                    }
                }
            }
            *at(mine) = x;
            __builtin_amdgcn_sched_barrier(0);       // (nothing in front of what the next tick waits for)
            put = TSWEEP ? x - (Word)w[r] : x;
            put_at = __umul24(unit[r].w, sv);         // (vertex 2^24 - 1 lies past the end)
            if constexpr (!TSWEEP) best = max(best, x);
            load(r);
            unpack(unit[(r + 1) % kAhead]);
            tick_barrier();
        }
    }
    if (!TSWEEP && a.cp_out) {
        const uint32_t to = (uint32_t)a.slots << kShift;         // (0 so far)
        __hip_atomic_fetch_max(at(to), best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        lds_barrier();
        if (tid == 0) a.cp_out[q] = (int64_t)*at(to);
    }
}

template <typename Word, bool T64, bool ONE, bool C16>
__global__ __launch_bounds__(ONE ? 64 : 1024) void chain_kernel(ChainArgs b, ChainArgs t, ChainShape sh) {
    const bool second = sh.sweeps == 3 ? (blockIdx.x & 1) != 0 : sh.sweeps == 2;
    const int32_t q = sh.sweeps == 3 ? (int32_t)(blockIdx.x >> 1) : (int32_t)blockIdx.x;
    if (second) chain_sweep<Word, T64, ONE, C16, true>(t, sh, q);
    else chain_sweep<Word, T64, ONE, C16, false>(b, sh, q);
}

}  // namespace

size_t chain_work_bytes(const ChainDir *db, const ChainDir *dt, int32_t width, int32_t P, bool cost16) {
    size_t bytes = 0;
    for (const ChainDir *d : {db, dt})
        if (d) bytes += align_up((size_t)P * d->ticks * width * (d == dt ? 20 : 16) / (cost16 ? 2 : 1));
    return bytes;
}

size_t chain_lds_bytes(const ChainDir &d, int word_bytes) { return ((size_t)(d.slots + 1 + kWave) * word_bytes + 15) & ~(size_t)15; }

int launch_chain(const SweepLaunch &sb, const SweepLaunch &st, const ChainDir &db, const ChainDir &dt, int32_t width,
                 int word_bytes, bool cost16, bool want_b, bool want_t, uint8_t *work, int32_t at_once, void *stream) {
    ChainArgs args[2]{};
    const SweepLaunch *launch[2] = {&sb, &st};
    const ChainDir *dir[2] = {&db, &dt};
    const bool want[2] = {want_b, want_t};
    for (int i = 0; i < 2; ++i) {
        const SweepLaunch &s = *launch[i];
        const ChainDir &d = *dir[i];
        ChainArgs &a = args[i];
        if (!want[i]) continue;
        a.units = (const u32x4 *)(s.blob + d.unit_off);
        a.edges = (const uint2 *)(s.blob + d.edge_off);
        a.idx = (const int32_t *)(s.blob + s.dir->idx_off);
        a.wt = (const uint32_t *)(s.blob + s.dir->wt_off);
        a.edge_tab = s.edge_tab;
        const size_t items = (size_t)at_once * d.ticks * width;
        a.cost = work;
        a.w = work + items * (cost16 ? 8 : 16);
        work += align_up(items * (i ? 20 : 16) / (cost16 ? 2 : 1));
        a.out_sv = s.out_sv;
        a.out_sq = s.out_sq;
        a.ticks = d.ticks;
        a.slots = d.slots;
    }
    ChainShape sh{};
    sh.a_sp = sb.a_stride_p;
    sh.a_sv = sb.a_stride_v;
    sh.c = (const uint32_t *)(sb.blob + sb.c_off);
    sh.vert_tab = sb.vert_tab;
    sh.status = sb.status;
    sh.n = sb.n;
    sh.k = sb.k;
    sh.width = width;
    sh.sweeps = (want_b ? 1 : 0) | (want_t ? 2 : 0);
    const unsigned both = sh.sweeps == 3 ? 2 : 1;
    const int32_t most = std::max(want_b ? db.ticks : 0, want_t ? dt.ticks : 0);
    const size_t lds = std::max(want_b ? chain_lds_bytes(db, word_bytes) : 0, want_t ? chain_lds_bytes(dt, word_bytes) : 0);
    hipStream_t s = (hipStream_t)stream;
    for (int32_t q0 = 0; q0 < sb.P; q0 += at_once) {
        sh.P = std::min(at_once, sb.P - q0);
        sh.assign = sb.assign + (int64_t)q0 * sb.a_stride_p;
        for (int i = 0; i < 2; ++i) {
            const SweepLaunch &l = *launch[i];
            if (!want[i]) continue;
            args[i].out = l.val ? (uint8_t *)l.val + (int64_t)q0 * l.out_sq * l.tick_bytes : nullptr;
            args[i].cp_out = l.cp_out ? l.cp_out + q0 : nullptr;
        }
        const dim3 grid((unsigned)(((int64_t)most * width + 255) / 256), (unsigned)sh.P, both);
#define CP_COST(MAGIC, C16) hipLaunchKernelGGL((chain_cost_kernel<MAGIC, C16>), grid, dim3(256), 0, s, args[0], args[1], sh)
        if (sb.magic && cost16) CP_COST(true, true);
        else if (sb.magic) CP_COST(true, false);
        else if (cost16) CP_COST(false, true);
        else CP_COST(false, false);
#undef CP_COST
        const dim3 groups((unsigned)sh.P * both), lanes((unsigned)width);
#define CP_CHAIN(WORD, T64, ONE, C16)                                                                                \
    do {                                                                                                             \
        const auto kernel = chain_kernel<WORD, T64, ONE, C16>;                                                       \
        if (hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) \
            return CP_ERR_HIP;                                                                                       \
        hipLaunchKernelGGL(kernel, groups, lanes, lds, s, args[0], args[1], sh);                                     \
    } while (0)
#define CP_CHAIN_OF(WORD, T64)                                                                                       \
    do {                                                                                                             \
        if (width == kWave && cost16) CP_CHAIN(WORD, T64, true, true);                                               \
        else if (width == kWave) CP_CHAIN(WORD, T64, true, false);                                                   \
        else if (cost16) CP_CHAIN(WORD, T64, false, true);                                                           \
        else CP_CHAIN(WORD, T64, false, false);                                                                      \
    } while (0)
        if (word_bytes == 8) CP_CHAIN_OF(unsigned long long, true);
        else if (sb.tick_bytes == 8) CP_CHAIN_OF(uint32_t, true);
        else CP_CHAIN_OF(uint32_t, false);
#undef CP_CHAIN_OF
#undef CP_CHAIN
        if (hipGetLastError() != hipSuccess) return CP_ERR_HIP;
    }
    return CP_OK;
}

}  // namespace cpeval
