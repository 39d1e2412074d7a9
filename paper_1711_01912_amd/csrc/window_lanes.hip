// Lane-window sweep: the resident-window idea with the partitions in the lanes.
//
// The resident-window kernel puts the vertices of a level into the lanes of one partition's
// workgroup.  On graphs whose levels are a few dozen vertices wide that leaves most lanes idle, and
// every partition pays the tick's chain of dependent LDS reads and its barrier for itself (19,800
// vertices in 660 levels, 4,096 partitions: 1.6 ms per sweep, 0.78 us a tick, three rounds of
// workgroups).  Here a workgroup owns G = 4 or 8 consecutive partitions, a wavefront relaxes
// 64 / G sub-rows (runs of at most LaneDir::width edges of a vertex) for all of them at once, and the
// lanes of a partition group share the packet entry they read, so a narrow level fills the
// lanes and the tick's chain is paid once per G partitions.  Both sweeps of a call run side by
// side in one launch.  Whole calls, before -> now: 2,016 vertices in 195 levels, 1,024 partitions 300 ->
// 105 us; 121,000 in 701 levels, 777 partitions, rows per vertex 2.84 -> 1.08 ms; 29,000 in 301 levels with
// 64-bit ticks (a launch per level before), 320 partitions 3.65 -> 0.28 ms.  What bounds it: on narrow ticks
// the chain of a tick (two LDS round trips, publication, barrier: 0.2 to 0.3 us; with far reads, 660 levels, 1.0 us with one
// workgroup on a compute unit, 1.3, 1.7 and 2.3 with two, three and four; there vector ALUs and LDS pipe are busy 36 and 37 % of
// the time and wavefronts wait 68 % of theirs), on wide ones the LDS pipe of a compute unit (121,000 vertices: 77 % busy, a
// third of it bank conflicts; vector ALUs 60 %, 25 instructions per 64 relaxations with what loaders and stores add).
// Divisions are one multiply-add (inverse_div): floats where no volume reaches 2^23, doubles above.  Against multiply-shift
// constants, whose 64-bit product alone takes four times as long: 121,000 vertices in 701 levels, 777 partitions
// 1,155 -> 1,077 us a call; 19,800 in 660, 4,096 partitions 1,685 -> 1,511; 29,000 in 301 with 64-bit words, 320
// partitions 315 -> 274; narrow ticks, which wait for their chain, gain least (1,578 levels of 34 vertices, 118 partitions
// 797 -> 763), and b alone of two vertices a level takes up to a tenth longer (530 levels, 908 partitions 141 -> 156).
//
// A ring word is value << 6 | device id, one LDS read per relaxation; x << 6 is added to it and the
// maximum taken over whole words, whose upper bits are the maximum of the sums.  Words are 32 bits while
// every value is below 2^26, else 64.
//
// LDS: [ring, (R+2) rows of G + 1 words, then 2 x far_cap rows][4 stage slots][cost tables][tick words].  The extra word of a
// row spreads the rows over the banks, both for lanes that read G words of a row and for lanes that
// read one partition's words of many rows.  Row R holds 0 (padding entries read it), row R+1 takes what
// padding sub-rows write.
//
// Roles (t = the tick between two barriers):
//   loaders   write packet t+2 into its stage slot and the device ids of its vertices into their
//             ring rows (both requested kDepth ticks earlier, held in registers)
//   compute   relax tick t; the next item's records and entries are read ahead, across the barrier
//   stores    write tick t-1 from the ring to the outputs: along a partition's row, or along a
//             vertex's row, as the caller asked.  The t sweep's ring holds tl + w, they take w off again.
//   far       where the ring cannot hold every neighbour: the store wavefronts also keep a copy of the words
//             that far reads will ask for in the workspace ([groups][numbers][G], 32 or 16 bytes together);
//             far wavefronts load the numbers of tick t + 1 + 2X, the words of tick t + 1 + X, and write
//             those of tick t + 1 behind the ring.  A word is copied in the iteration after its tick, every
//             store wavefront waits each iteration until its copies of kFarWait iterations ago have
//             reached the L2, and the fetch, past the L1, is issued X + 1 iterations before the tick that
//             reads it: a distance of kFarWait + X + 3 = 15 ticks or more is safe; kLaneFarTicks is 16.
// A vertex with several sub-rows needs no care: words are published with LDS maxima into rows that hold
// the device ids already.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "device_math.hpp"
#include "launch.hpp"

namespace cpeval {
namespace {

constexpr int kFarLead = 4;      // X: ticks between the requests of a far wavefront
constexpr int kFarWait = 8;      // iterations a copy may be on its way
constexpr int kFarPieces = 4;    // far reads a far wavefront serves per tick: this many times 64 / G
static_assert(kFarWait + kFarLead + 3 < kLaneFarTicks, "far reads need their distance");
constexpr int kSlots = 4;        // stage slots: being stored, computed, read ahead, filled

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct LaneArgs {
    const uint4 *stream;
    const uint32_t *tick_tab;
    const uint8_t *ids;        // [groups][n][G], by position
    void *out;                 // ticks of (v, q) at v * out_sv + q * out_sq, or NULL
    int64_t out_sv, out_sq;
    uint32_t off_sv, off_sq;   // the strides in bytes
    int32_t out64;             // outputs are 64-bit
    int64_t *cp_out;           // [P] or NULL
    const void *edge_tab, *vert_tab;
    const int32_t *far_list;   // [T][far_cap]
    void *far;                 // words [groups][far_count][G]
    int32_t far_cap, far_count;
    int32_t n, P, k, T, R;
};

struct LaneShape {
    int32_t nc, nlw, nsw, nfw; // compute, loader, store and far wavefronts (no kernel reads the last; without it the struct
                               // is no 32 bytes, registers are given out otherwise, and calls with far reads or
                               // 64-bit words take 3 % longer, those with narrow 32-bit ticks 2 % less)
    uint32_t stage_off, stage_bytes, tab_off, ticks_off;
};

__device__ __forceinline__ uint32_t tick_units(uint32_t word) { return word & 0x3fffu; }
__device__ __forceinline__ uint32_t tick_verts(uint32_t word) { return word >> 14 & 0x1ffu; }
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

template <typename Word, bool TSWEEP, int G, int W, typename Tab, int NL, bool FAR>
__device__ __forceinline__ void lane_sweep(const LaneArgs &a, const LaneShape &sh, uint8_t *lds,
                                           unsigned long long *red, int32_t grp) {
    constexpr int kDepth = 8 / NL;           // ticks a loader runs ahead of the stage, NL 16-byte loads a lane each
    constexpr int RPW = 64 / G;              // sub-rows a wavefront relaxes at a time
    constexpr int IU = RPW / kLaneUnit;      // units of an item
    constexpr int VS = G + 1;                // words between two rows of the ring
    constexpr int UNIT = 64 * (1 + W);       // bytes of a unit
    constexpr uint32_t ID = (1u << kLaneIdBits) - 1;
    const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = a.T, R = a.R, k = a.k;
    Word *ring = (Word *)lds;
    uint8_t *stage = lds + sh.stage_off;
    const Tab *etab = (const Tab *)(lds + sh.tab_off);
    const Tab *vtab = etab + k * k;
    const uint32_t *words = (const uint32_t *)(lds + sh.ticks_off);
    {
        Tab *to = (Tab *)(lds + sh.tab_off);
        for (int i = tid; i < k * k; i += nt) to[i] = ((const Tab *)a.edge_tab)[i];
        for (int i = tid; i < k; i += nt) to[k * k + i] = ((const Tab *)a.vert_tab)[i];
        for (int i = tid; i < (2 + 2 * a.far_cap) * VS; i += nt) ring[(size_t)R * VS + i] = 0;
        uint32_t *dst = (uint32_t *)(lds + sh.ticks_off);
        for (int i = tid; i < T + 2; i += nt) dst[i] = i < T ? a.tick_tab[i] : 0;     // two empty ticks behind the last
        if (tid < G) red[tid] = 0;
    }
    lds_barrier();                           // tables and tick words are there
    // iterations of every role's loop: the ticks, one more for the last tick's stores, rounded up
    // so that the loaders' registers can be named
    static_assert(4 % kDepth == 0 && kFarLead == 4, "one rounding for all");
    const int N = (T + 1 + 3) / 4 * 4;
    const int32_t q0 = grp * G;

    if (FAR && wave >= sh.nc + sh.nlw + sh.nsw) {
        // ------------------------------------------------ far wavefronts
        constexpr int X = kFarLead;
        const int fw = wave - sh.nc - sh.nlw - sh.nsw;
        const int g = lane % G, cap = a.far_cap;
        if (cap == 0) {                      // (the other sweep has far reads)
            for (int t = -1; t < N; ++t) lds_barrier();
        } else {
        const Word *words_of = (const Word *)a.far + (size_t)grp * (size_t)a.far_count * G + g;
        uint32_t lst[X][kFarPieces];
        Word got[X][kFarPieces];
        int row[kFarPieces];                 // (past the cap: its last row once more)
#pragma unroll
        for (int i = 0; i < kFarPieces; ++i) row[i] = min((fw * kFarPieces + i) * RPW + lane / G, cap - 1);
        auto list_load = [&](int s, int r) {
#pragma unroll
            for (int i = 0; i < kFarPieces; ++i)
                lst[r][i] = (uint32_t)a.far_list[(size_t)min(s, T - 1) * (size_t)cap + (size_t)row[i]];
        };
#pragma unroll
        for (int j = 1; j <= X; ++j) {
            // (a first word each, in the order of the loop: the waits for what the loop asked for earlier would
            // otherwise have to cover a first iteration with fewer requests behind)
#pragma unroll
            for (int i = 0; i < kFarPieces; ++i)
                got[j % X][i] = __hip_atomic_load(words_of, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            list_load(j + X, j % X);
        }
        lds_barrier();
        for (int t0 = 0; t0 < N; t0 += X) {
#pragma unroll
            for (int r = 0; r < X; ++r) {
                const int t = t0 + r, sl = (r + 1) % X;
                lds_barrier();
                Word *to = ring + (size_t)(R + 2 + ((t + 1) & 1) * cap) * VS + g;
#pragma unroll
                for (int i = 0; i < kFarPieces; ++i) to[row[i] * VS] = got[sl][i];
#pragma unroll
                for (int i = 0; i < kFarPieces; ++i)
                    got[sl][i] = __hip_atomic_load(words_of + (size_t)lst[sl][i] * G, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
                list_load(t + 1 + 2 * X, sl);
            }
        }
        }
    } else if (wave >= sh.nc + sh.nlw) {
        // ------------------------------------------------ store wavefronts
        // Two pieces at a time, so that their LDS reads overlap; a piece is up to 64 outputs.
        const int sw = wave - sh.nc - sh.nlw, nsw = sh.nsw;
        const int32_t live = min(G, a.P - q0);
        const uint32_t sv = a.off_sv, sq = a.off_sq;           // bytes; a group's outputs span less than 4 GB
        char *base = (char *)a.out + (size_t)q0 * (size_t)a.out_sq * (a.out64 ? 8 : 4);
        const bool by_row = a.out_sv == 1;
        const Tab up = round_up(Tab());    // (no variable divisions behind this)
        uint32_t slot0 = 0;                  // of the tick being stored
        int copied = 0;                      // numbers given to far copies so far
        uint64_t recent = 0;                 // stores of each of the last kFarWait iterations, a byte each
        auto ring_slot = [&](int vi) {
            const uint32_t s = slot0 + (uint32_t)vi;
            return s >= (uint32_t)R ? s - (uint32_t)R : s;
        };
        auto put2 = [&](uint32_t slot_a, int ga, uint2 ra, bool ok_a, uint32_t slot_b, int gb, uint2 rb, bool ok_b) {
            Word xa = ring[__umul24(slot_a, (uint32_t)VS) + ga], xb = ring[__umul24(slot_b, (uint32_t)VS) + gb];
            const uint32_t at_a = ra.x * sv + (uint32_t)ga * sq, at_b = rb.x * sv + (uint32_t)gb * sq;
            if constexpr (TSWEEP) {
                const Tab ma = vtab[(uint32_t)xa & ID], mb = vtab[(uint32_t)xb & ID];
                xa = (xa >> kLaneIdBits) - (Word)inverse_div(word_for<Tab>(ra.y), ma, up);
                xb = (xb >> kLaneIdBits) - (Word)inverse_div(word_for<Tab>(rb.y), mb, up);
            } else {
                xa >>= kLaneIdBits;
                xb >>= kLaneIdBits;
            }
            if (a.out64) {
                if (ok_a) *(int64_t *)(base + at_a) = (int64_t)xa;
                if (ok_b) *(int64_t *)(base + at_b) = (int64_t)xb;
            } else {
                if (ok_a) *(int32_t *)(base + at_a) = (int32_t)xa;
                if (ok_b) *(int32_t *)(base + at_b) = (int32_t)xb;
            }
        };
        lds_barrier();
        uint32_t word = words[0];
        for (int t = 0; t < N; ++t) {
            lds_barrier();
            if (t < 1 || t > T) continue;
            const uint32_t tick = uniform(word);
            word = words[t];                 // of the next iteration's tick
            const int w = (int)tick_verts(tick);
            const uint2 *verts = (const uint2 *)(stage + (size_t)((t - 1) % kSlots) * sh.stage_bytes + tick_units(tick) * UNIT);
            uint32_t sure = 0;               // stores this iteration issues, at least
            if (FAR && a.far_cap > 0) {
                // the copies first: what is left of this iteration's stores may stay on its way
                const int copies = (int)(tick >> 23);
                const uint32_t *slots = (const uint32_t *)(verts + w);
                Word *to = (Word *)a.far + ((size_t)grp * (size_t)a.far_count + (size_t)copied) * G + lane % G;
                for (int f0 = sw * RPW; f0 < copies; f0 += nsw * RPW) {
                    const int f = f0 + lane / G;
                    const uint32_t slot = slots[min(f, copies - 1)];
                    const Word x = ring[__umul24(slot, (uint32_t)VS) + lane % G];
                    if (f < copies) __hip_atomic_store(to + (size_t)f * G, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ++sure;
                }
                copied += copies;
            }
            if (!a.out) {
            } else if (by_row) {
                // along the partitions' rows: 2^wl vertices x 2^(6-wl) partitions a piece
                const int wl = w >= 64 ? 6 : 32 - __clz(w - 1);
                const int vl = lane & ((1 << wl) - 1), gl = lane >> wl, gs = 64 >> wl;
                for (int v0 = 0; v0 < w; v0 += 64) {
                    const int vi = min(v0 + vl, w - 1);
                    const uint2 r = verts[vi];
                    const uint32_t slot = ring_slot(vi);
                    const bool mine = v0 + vl < w;
                    for (int g0 = sw * gs; g0 < G; g0 += 2 * nsw * gs) {
                        const int ga = g0 + gl, gb = ga + nsw * gs;
                        put2(slot, min(ga, G - 1), r, mine && ga < live, slot, min(gb, G - 1), r, mine && gb < live);
                        if (FAR) sure += (uint32_t)(g0 < live) + (uint32_t)(g0 + nsw * gs < live);
                    }
                }
            } else {
                // along the vertices' rows: the G partitions of 64 / G vertices a piece
                const int g = lane % G, vl = lane / G;
                for (int v0 = sw * RPW; v0 < w; v0 += 2 * nsw * RPW) {
                    const int va = v0 + vl, vb = va + nsw * RPW;
                    const int ca = min(va, w - 1), cb = min(vb, w - 1);
                    const uint2 ra = verts[ca], rb = verts[cb];
                    put2(ring_slot(ca), g, ra, va < w && g < live, ring_slot(cb), g, rb, vb < w && g < live);
                    if (FAR) sure += 1u + (uint32_t)(v0 + nsw * RPW < w);
                }
            }
            slot0 += (uint32_t)w;
            if (slot0 >= (uint32_t)R) slot0 -= (uint32_t)R;
            if (FAR && a.far_cap > 0) {
                // copies of kFarWait iterations ago have arrived once no more stores are on their way than
                // the later iterations issued
                recent = recent << 8 | min(sure, 31u);
                uint32_t later = 0;
#pragma unroll
                for (int i = 0; i < kFarWait; ++i) later += (uint32_t)(recent >> (8 * i)) & 0xffu;
#define CP_WAIT(N)                                                                  \
    if (later >= N) {                                                               \
        asm volatile("s_waitcnt vmcnt(" #N ")" ::: "memory");                       \
    } else
                CP_WAIT(48) CP_WAIT(32) CP_WAIT(24) CP_WAIT(20) CP_WAIT(16) CP_WAIT(12) CP_WAIT(8) CP_WAIT(6) CP_WAIT(4)
                CP_WAIT(2) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
#undef CP_WAIT
            }
        }
    } else if (wave >= sh.nc) {
        // ------------------------------------------------ loader wavefronts
        const int lw = wave - sh.nc;
        const int vi = lw * 64 + lane;                         // this lane's vertex of a tick
        const uint4 *stream = a.stream;
        const uint8_t *gids = a.ids + (size_t)grp * (size_t)a.n * G;
        u32x4 buf[kDepth][NL];
        uint32_t idr[kDepth][G / 4];
        uint32_t verts[kDepth];              // of the ticks on their way (uniform)
        uint32_t put_slot = 0;               // ring slot of the first vertex of the tick to be put next
        // Packet and device ids of tick s (of the last tick once more past the end: no branch around a
        // load, or the waits for loads would have to cover both ways and end up waiting for the youngest;
        // the tick words come from LDS because a scalar load's wait is a wait for LDS too).
        auto issue = [&](int s, int r) {
            const uint32_t word = uniform(words[min(s, T - 1)]);
            verts[r] = tick_verts(word);
            const uint32_t chunks = (tick_units(word) * UNIT + 8 * verts[r] + 4 * (word >> 23) + 15) / 16;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
                const uint32_t c = (uint32_t)((i * sh.nlw + lw) * 64 + lane);
                buf[r][i] = *(const u32x4 *)(stream + min(c, chunks - 1));
            }
            const uint32_t *row = (const uint32_t *)(gids + min((uint32_t)vi, verts[r] - 1) * (uint32_t)G);
            if constexpr (G == 8) {
                const uint2 x = *(const uint2 *)row;
                idr[r][0] = x.x;
                idr[r][1] = x.y;
            } else {
                idr[r][0] = *row;
            }
            if (s < T - 1) {
                stream += chunks;
                gids += (size_t)verts[r] * G;
            }
        };
        auto put = [&](int s, int r) {
            u32x4 *dst = (u32x4 *)(stage + (size_t)(s % kSlots) * sh.stage_bytes);
#pragma unroll
            for (int i = 0; i < NL; ++i) dst[(i * sh.nlw + lw) * 64 + lane] = buf[r][i];
            if ((uint32_t)vi < verts[r] && s < T) {
                uint32_t slot = put_slot + (uint32_t)vi;
                if (slot >= (uint32_t)R) slot -= (uint32_t)R;
                Word *row = ring + __umul24(slot, (uint32_t)VS);
#pragma unroll
                for (int g = 0; g < G; ++g) row[g] = (Word)((idr[r][g / 4] >> (8 * (g % 4))) & 0xffu);
            }
            put_slot += verts[r];
            if (put_slot >= (uint32_t)R) put_slot -= (uint32_t)R;
        };
#pragma unroll
        for (int r = 0; r < kDepth; ++r) issue(r, r);
        put(0, 0);
        issue(kDepth, 0);
        put(1, 1);
        issue(kDepth + 1, 1);
        lds_barrier();
        for (int t0 = 0; t0 < N; t0 += kDepth) {
#pragma unroll
            for (int r = 0; r < kDepth; ++r) {
                lds_barrier();
                put(t0 + r + 2, (r + 2) % kDepth);
                issue(t0 + r + 2 + kDepth, (r + 2) % kDepth);
            }
        }
    } else {
        // ------------------------------------------------ compute wavefronts
        // An item = RPW sub-rows of a unit: two dependent LDS round trips (ring words, table entries) and a
        // publication; the next item's records and entries are on their way meanwhile.
        __builtin_amdgcn_s_setprio(1);
        const Tab up = round_up(Tab());
        const int g = lane % G, rg = lane / G;
        uint2 rec, ent[W];
        const uint32_t lane_off = (uint32_t)(rg / kLaneUnit) * UNIT + (uint32_t)(rg % kLaneUnit) * 8;
        auto ask = [&](uint32_t at) {
            const uint2 *p = (const uint2 *)(stage + at + lane_off);
            rec = p[0];
#pragma unroll
            for (int j = 0; j < W; ++j) ent[j] = p[(1 + j) * kLaneUnit];
        };
        auto item_at = [&](int t, int i) {
            return (uint32_t)(t % kSlots) * sh.stage_bytes + (uint32_t)i * (IU * UNIT);
        };
        Word best = 0;
        lds_barrier();
        int items = (int)tick_units(uniform(words[0])) / IU;
        ask(item_at(0, wave));               // (past the tick's last item: stage bytes nobody uses)
        for (int t = 0; t < N; ++t) {
            lds_barrier();
            const uint32_t word_next = words[min(t + 1, T)];
            int i = wave;
            if (i >= items) ask(item_at(t + 1, wave));
            while (i < items) {
                const uint2 rec_c = rec;
                uint32_t x_t[W];
                Word v[W];
                Word *mine = ring + __umul24(rec_c.x, (uint32_t)VS) + g;
                const Word own_w = *mine;
#pragma unroll
                for (int j = 0; j < W; ++j) {
                    v[j] = ring[__umul24(ent[j].x, (uint32_t)VS) + g];
                    x_t[j] = ent[j].y;
                }
                i += sh.nc;
                ask(i < items ? item_at(t, i) : item_at(t + 1, wave));
                // (before the ring's words are waited for: left to itself the compiler asks between them and the table, and the
                // division by floats waits for all three; 1,578 levels of 34 vertices, 118 partitions 830 -> 765 us a call)
                __builtin_amdgcn_sched_barrier(0);
                const uint32_t own = (uint32_t)own_w & ID;
                const Tab *erow = etab + __umul24(own, (uint32_t)k);
                Tab m[W];
#pragma unroll
                for (int j = 0; j < W; ++j) m[j] = erow[(uint32_t)v[j] & ID];
                const Tab mw = vtab[own];
                Word acc = 0;
#pragma unroll
                for (int j = 0; j < W; ++j) acc = max(acc, add_quotient(v[j], x_t[j], m[j], up));
                const Word fin = add_quotient((acc & ~(Word)ID) | own, rec_c.y, mw, up);
                atomicMax(mine, fin);
                best = max(best, fin);
            }
            items = (int)tick_units(uniform(word_next)) / IU;
        }
        if (a.cp_out) atomicMax(&red[g], (unsigned long long)(best >> kLaneIdBits));
    }

    if (a.cp_out) {
        lds_barrier();
        if (tid < G && q0 + tid < a.P) a.cp_out[q0 + tid] = (int64_t)red[tid];
    }
}

// Both sweeps (sweeps = 3) or one of them; workgroups of one partition group sit side by side, and an
// XCD gets consecutive groups, so that lines of a vertex's row meet in one L2.
template <typename Word, int G, int W, typename Tab, int NL, bool FAR>
__global__ __launch_bounds__(kWindowMaxWaves * 64, FAR && sizeof(Word) == 4 ? 8 : 4) void window_lanes_kernel(LaneArgs b, LaneArgs t, LaneShape sh,
                                                                            int32_t sweeps, int32_t total,
                                                                            int32_t per_xcd) {
    extern __shared__ uint4 lds16[];
    __shared__ unsigned long long red[G];
    const int32_t id = (int32_t)(blockIdx.x % 8) * per_xcd + (int32_t)(blockIdx.x / 8);
    if (id >= total) return;                   // whole workgroup: no barrier has been reached yet
    const bool second = sweeps == 3 ? (id & 1) != 0 : sweeps == 2;
    const int32_t grp = sweeps == 3 ? id >> 1 : id;
    if (second) lane_sweep<Word, true, G, W, Tab, NL, FAR>(t, sh, (uint8_t *)lds16, red, grp);
    else lane_sweep<Word, false, G, W, Tab, NL, FAR>(b, sh, (uint8_t *)lds16, red, grp);
}

// Device ids as the loaders want them: [groups][n][G] by position of either sweep, groups past the batch
// filled up with its last partition.  An id >= k is reported and replaced by k - 1.
template <int G>
__global__ __launch_bounds__(256) void group_ids_kernel(const uint8_t *__restrict__ assign, int64_t sp, int64_t sv,
                                                        int32_t n, int32_t P, int32_t k,
                                                        const int32_t *__restrict__ pos_b,
                                                        const int32_t *__restrict__ pos_t, uint8_t *__restrict__ out_b,
                                                        uint8_t *__restrict__ out_t, int32_t *status) {
    const int32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    bool bad = false;
    uint32_t w[G / 4];
#pragma unroll
    for (int i = 0; i < G / 4; ++i) w[i] = 0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int32_t q = min((int32_t)blockIdx.y * G + g, P - 1);
        uint32_t d = assign[(int64_t)q * sp + (int64_t)v * sv];
        if (d >= (uint32_t)k) { bad = true; d = (uint32_t)k - 1; }
        w[g / 4] |= d << (8 * (g % 4));
    }
    const size_t at = (size_t)blockIdx.y * (size_t)n;
    auto write = [&](uint8_t *row) {
        if constexpr (G == 8) *(uint2 *)row = make_uint2(w[0], w[1]);
        else *(uint32_t *)row = w[0];
    };
    if (out_b) write(out_b + (at + (size_t)pos_b[v]) * G);
    if (out_t) write(out_t + (at + (size_t)pos_t[v]) * G);
    if (bad) *status = CP_STATUS_BAD_DEVICE_ID;
}

LaneArgs lane_args(const SweepLaunch &s, const LaneDir &d, const uint8_t *ids, bool floats, uint8_t *far) {
    LaneArgs a{};
    a.stream = (const uint4 *)(s.blob + d.stream_off);
    a.tick_tab = (const uint32_t *)(s.blob + d.tick_off);
    a.ids = ids;
    a.out = s.val;
    a.out_sv = s.out_sv;
    a.out_sq = s.out_sq;
    a.out64 = s.tick_bytes == 8;
    a.off_sv = (uint32_t)(s.out_sv * s.tick_bytes);
    a.off_sq = (uint32_t)(s.out_sq * s.tick_bytes);
    a.cp_out = s.cp_out;
    a.edge_tab = floats ? (const void *)s.edge_tab4 : s.edge_tab;
    a.vert_tab = floats ? (const void *)s.vert_tab4 : s.vert_tab;
    a.far_list = (const int32_t *)(s.blob + d.far_off);
    a.far = far;
    a.far_cap = d.far_cap;
    a.far_count = d.far_count;
    a.n = s.n; a.P = s.P; a.k = s.k; a.T = d.ticks; a.R = d.slots;
    return a;
}

template <typename Word, int G, int W, typename Tab, int NL, bool FAR>
int launch_lanes_k(const LaneArgs &b, const LaneArgs &t, const LaneCfg &cfg, int sweeps, int32_t P, hipStream_t st) {
    auto kern = window_lanes_kernel<Word, G, W, Tab, NL, FAR>;
    if (cfg.lds_bytes > 64 * 1024 &&
        hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)cfg.lds_bytes) !=
            hipSuccess)
        return CP_ERR_HIP;
    LaneShape sh{};
    sh.nc = cfg.nc; sh.nlw = cfg.nlw; sh.nsw = cfg.nsw; sh.nfw = cfg.nfw;
    sh.stage_off = (uint32_t)cfg.stage_off;
    sh.stage_bytes = (uint32_t)cfg.stage_bytes;
    sh.tab_off = (uint32_t)cfg.tab_off;
    sh.ticks_off = (uint32_t)cfg.ticks_off;
    const int32_t total = (P + G - 1) / G * (sweeps == 3 ? 2 : 1), per_xcd = (total + 7) / 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * per_xcd)), dim3((cfg.nc + cfg.nlw + cfg.nsw + cfg.nfw) * 64), cfg.lds_bytes, st,
                       b, t, sh, (int32_t)sweeps, total, per_xcd);
    return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_HIP;
}

template <typename Word, int G, int W, typename Tab>
int launch_lanes_n(const LaneArgs &b, const LaneArgs &t, const LaneCfg &cfg, int sweeps, int32_t P, hipStream_t st) {
    if (cfg.nfw > 0) return launch_lanes_k<Word, G, W, Tab, 2, true>(b, t, cfg, sweeps, P, st);
    return cfg.nl == 4 ? launch_lanes_k<Word, G, W, Tab, 4, false>(b, t, cfg, sweeps, P, st)
                       : launch_lanes_k<Word, G, W, Tab, 2, false>(b, t, cfg, sweeps, P, st);
}

template <typename Word, int G, typename Tab>
int launch_lanes_g(const LaneArgs &b, const LaneArgs &t, const LaneCfg &cfg, int sweeps, int32_t P, hipStream_t st) {
    return cfg.width == 2 ? launch_lanes_n<Word, G, 2, Tab>(b, t, cfg, sweeps, P, st)
                          : launch_lanes_n<Word, G, 4, Tab>(b, t, cfg, sweeps, P, st);
}

template <typename Word, typename Tab>
int launch_lanes_w(const LaneArgs &b, const LaneArgs &t, const LaneCfg &cfg, int sweeps, int32_t P, hipStream_t st) {
    return cfg.groups == 8 ? launch_lanes_g<Word, 8, Tab>(b, t, cfg, sweeps, P, st)
                           : launch_lanes_g<Word, 4, Tab>(b, t, cfg, sweeps, P, st);
}

}  // namespace

bool lane_config(const LaneDir &db, const LaneDir &dt, int32_t n, int32_t k, int groups, int word_bytes, bool with_out,
                 int64_t workgroups, size_t lds_limit, LaneCfg &out) {
    const size_t static_lds = 512;
    const size_t G = (size_t)groups, rows = (size_t)std::max(db.slots + 2 * db.far_cap, dt.slots + 2 * dt.far_cap) + 2;
    const int chunks = std::max(db.max_chunks, dt.max_chunks), verts = std::max(db.max_verts, dt.max_verts);
    if (db.width != dt.width) return false;
    LaneCfg c;
    c.groups = groups;
    c.width = db.width;
    c.word = word_bytes;
    const int far_cap = std::max(db.far_cap, dt.far_cap);
    c.nfw = far_cap > 0 ? (far_cap * groups / 64 + kFarPieces - 1) / kFarPieces : 0;
    // wide ticks: fewer loaders with more loads each, which need not run as far ahead
    c.nl = chunks > 256 && c.nfw == 0 ? 4 : 2;
    c.nlw = std::max((verts + 63) / 64, (chunks + 64 * c.nl - 1) / (64 * c.nl));
    if (c.nlw > 8) return false;
    c.stage_off = align_up(rows * (G + 1) * (size_t)word_bytes, 16);
    c.stage_bytes = (size_t)c.nlw * c.nl * 1024;
    c.tab_off = c.stage_off + kSlots * c.stage_bytes;
    // a wavefront without items still reads the place of its first one: stage bytes, or what lies behind them
    c.ticks_off = c.tab_off + sizeof(Magic) * ((size_t)k * k + k);
    const size_t reach = c.tab_off + (size_t)(kWindowMaxWaves + 1) * (8 / groups) * lane_unit_bytes(c.width);
    c.lds_bytes = std::max(c.ticks_off + 4 * ((size_t)std::max(db.ticks, dt.ticks) + 2), reach);
    if (c.lds_bytes + static_lds > lds_limit || rows * (G + 1) >= (1u << 24)) return false;
    // Workgroups that will share a compute unit share its 32 wavefronts (24 with far reads and 64-bit
    // words).  Compute wavefronts for half of an average tick's items, store wavefronts for two pieces of
    // its outputs each: more of either only adds idle instructions to a unit that is short of issue slots
    // (19,800 vertices, 4,096 partitions: 5 + 1 of them 2.11 ms, 3 + 2 1.59 ms; 29,000 vertices with 64-bit
    // words: 11 + 2 of them 325 us, 4 + 3 285 us).
    const int waves = far_cap > 0 && word_bytes == 8 ? 24 : 32;
    const int share = (int)std::max<int64_t>(1, std::min<int64_t>((workgroups + 255) / 256,
                                                                  (int64_t)(kLdsBudget / (c.lds_bytes + static_lds))));
    const int most = std::min(kWindowMaxWaves, std::max(waves / share, c.nlw + c.nfw + 2));
    const double ticks = (double)std::min(db.ticks, dt.ticks);
    const int outs = (int)std::ceil((double)n / ticks * groups / 64 / 2);
    const int items = (int)std::ceil((double)std::max(db.units, dt.units) / ticks * groups / 8 * 0.55);
    c.nsw = with_out || far_cap > 0 ? std::max(1, std::min({4, outs, most - c.nlw - c.nfw - 1})) : 0;
    c.nc = std::max(1, std::min(most - c.nlw - c.nsw - c.nfw, items));
    out = c;
    return true;
}

size_t lane_ids_bytes(int32_t n, int32_t P, int groups) {
    return align_up((size_t)((P + groups - 1) / groups) * groups * (size_t)n);
}

size_t lane_work_bytes(const LaneDir *db, const LaneDir *dt, int32_t n, int32_t P, int groups, int word_bytes) {
    size_t bytes = 0;
    for (const LaneDir *d : {db, dt})
        if (d)
            bytes += lane_ids_bytes(n, P, groups) +
                     align_up((size_t)((P + groups - 1) / groups) * groups * (size_t)d->far_count * (size_t)word_bytes);
    return bytes;
}

int launch_window_lanes(const SweepLaunch &sb, const SweepLaunch &st, const LaneDir &db, const LaneDir &dt,
                        const LaneCfg &cfg, bool want_b, bool want_t, uint8_t *ids, void *stream) {
    hipStream_t hs = (hipStream_t)stream;
    const dim3 grid((unsigned)((sb.n + 255) / 256), (unsigned)((sb.P + cfg.groups - 1) / cfg.groups)), block(256);
    const int sweeps = (want_b ? 1 : 0) | (want_t ? 2 : 0);
    if (grid.y > 65535 || sweeps == 0) return CP_ERR_ARG;
    uint8_t *ids_b = want_b ? ids : nullptr;
    uint8_t *ids_t = want_t ? ids + (want_b ? lane_ids_bytes(sb.n, sb.P, cfg.groups) : 0) : nullptr;
    uint8_t *far_b = ids + (size_t)(want_b + want_t) * lane_ids_bytes(sb.n, sb.P, cfg.groups);
    uint8_t *far_t = far_b + (want_b ? lane_work_bytes(&db, nullptr, sb.n, sb.P, cfg.groups, cfg.word) -
                                           lane_ids_bytes(sb.n, sb.P, cfg.groups) : 0);
    const int32_t *pos_b = (const int32_t *)(sb.blob + db.pos_off), *pos_t = (const int32_t *)(sb.blob + dt.pos_off);
#define CP_GROUP(G)                                                                                           \
    hipLaunchKernelGGL(group_ids_kernel<G>, grid, block, 0, hs, sb.assign, sb.a_stride_p, sb.a_stride_v, sb.n, \
                       sb.P, sb.k, pos_b, pos_t, ids_b, ids_t, sb.status)
    if (cfg.groups == 8) CP_GROUP(8);
    else if (cfg.groups == 4) CP_GROUP(4);
    else return CP_ERR_ARG;
#undef CP_GROUP
    if (hipGetLastError() != hipSuccess) return CP_ERR_HIP;
    const LaneArgs b = lane_args(sb, db, ids_b, cfg.floats, far_b), t = lane_args(st, dt, ids_t, cfg.floats, far_t);
    if (cfg.word == 8)
        return cfg.floats ? launch_lanes_w<unsigned long long, float>(b, t, cfg, sweeps, sb.P, hs)
                          : launch_lanes_w<unsigned long long, double>(b, t, cfg, sweeps, sb.P, hs);
    return cfg.floats ? launch_lanes_w<uint32_t, float>(b, t, cfg, sweeps, sb.P, hs)
                      : launch_lanes_w<uint32_t, double>(b, t, cfg, sweeps, sb.P, hs);
}

}  // namespace cpeval
