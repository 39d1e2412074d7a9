// List-scheduling simulation of one iteration for a batch of partitions: the paper's
// scheduling criteria (section 4, (1)-(6)) with its PCT rule (section 4.1) or the FIFO
// baseline (section 5.1), on the cost model of section 2 in integer ticks.  The result is
// the start time of every vertex and the makespan, the quantity the paper's evaluation
// plots (section 5).
//
// One wavefront simulates one partition, lane d being device d; with 32 devices or fewer it
// simulates 64 / k partitions side by side, k lanes each.  A device keeps the vertices
// whose predecessors have all started -- their ready time is final by then -- in a
// min-heap keyed by ready time ("pending"); under PCT the ones that are executable at the
// device's decision time move on to a second heap keyed by descending b ("available").
// Devices only interact through tensors that arrive: a vertex that starts at time T on
// one device reaches another device no earlier than T + (shortest execution time) +
// (shortest transfer time).  So with T_min the earliest decision time over all devices,
// every device whose decision time lies less than that sum after T_min already knows all
// it needs, and those lanes decide in the same step.  A lane that starts a vertex lowers
// the open-input count of each successor and raises its ready time; the lane that takes
// the last open input hands the successor to its owner's inbox, which the owner drains at
// the top of its next step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "cpeval_internal.hpp"
#include "device_math.hpp"
#include "launch.hpp"

namespace cpeval {

namespace {

constexpr uint32_t kNever = 0xffffffffu;
constexpr size_t kSimWaves = 32;         // wavefronts a compute unit holds
constexpr size_t kSimStaticLds = 1024;   // static LDS of a wavefront with a near inbox, the most there is
constexpr int kWideRow = 32;      // out-edges from which a started vertex's row is shared out over the wavefront

// All lanes of a partition sit in one wavefront, so everything they exchange passes through
// one compute unit's vector L1 and one L2; no fence wider than the workgroup is ever needed (a
// release at device scope would write the L2 back on every step).  Ready times and open-input
// counts are only changed by read-modify-write atomics, which execute in the L2 and leave the
// L1 stale: a ready time is read back with a load of device scope, which goes past the L1.
// Inbox slots are written with ordinary stores and read afterwards by another lane of the wavefront; where the
// first of a step wait in LDS they are written again every step.  Either is safe because one wavefront writes and reads
// them: its accesses to an address keep their order in its compute unit's L1, which writes through, and step_fence
// waits for the stores before the next step's loads.
__device__ __forceinline__ int32_t l2_read(int32_t *p) {
    // a device-scope load goes past the L1 like the atomics do, and unlike an atomic it writes nothing
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t inbox_load(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void inbox_store(int32_t *p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
// Every memory operation of the wavefront issued so far has completed.
__device__ __forceinline__ void step_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// Four-ary min-heaps of 64-bit keys (children of i: 4i+1 .. 4i+4): half the levels of a binary
// heap, and the four children of a node are loaded together.  A lane's heap is touched by that
// lane only.  A heap never holds more keys than its device has vertices, so 16 levels bound
// every loop.
__device__ __forceinline__ void heap_push(uint64_t *h, int32_t &size, uint64_t key) {
    int32_t i = size++;
    for (int depth = 0; depth < 16 && i > 0; ++depth) {
        const int32_t up = (i - 1) >> 2;
        const uint64_t uk = h[up];
        if (uk <= key) break;
        h[i] = uk;
        i = up;
    }
    h[i] = key;
}

__device__ __forceinline__ uint64_t heap_pop(uint64_t *h, int32_t &size) {
    const uint64_t top = h[0];
    const int32_t left = --size;
    if (left > 0) {
        const uint64_t last = h[left];
        int32_t i = 0;
        for (int depth = 0; depth < 16; ++depth) {
            const int32_t c0 = 4 * i + 1;
            if (c0 >= left) break;
            uint64_t ck[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) ck[j] = h[min(c0 + j, left - 1)];     // in range; masked below
            uint64_t best = ck[0];
            int32_t at = c0;
#pragma unroll
            for (int j = 1; j < 4; ++j) {
                if (c0 + j < left && ck[j] < best) {
                    best = ck[j];
                    at = c0 + j;
                }
            }
            if (last <= best) break;
            h[i] = best;
            i = at;
        }
        h[i] = last;
    }
    return top;
}

// A queue = its three smallest keys in registers, in order, + the heap above in memory for the rest.  Device
// queues are short most of the time (a handful of executable vertices), so most pushes and
// pops never touch memory, and the decision time is read from a register.  Three, because with four three partitions
// of a wavefront need more registers than the wavefronts of a full unit have (20,000 partitions on 3 devices: 5.8 ms, 4.4
// with three); on 50 devices one to six differ by 3 %.
constexpr uint64_t kNoKey = ~0ull;         // above every key: times and 2^31 - 1 - b lie below 2^31
constexpr int kHeld = 3;

struct Queue {
    uint64_t key[kHeld];
    uint32_t b[kHeld];         // pending under PCT: b of each, so that it is loaded once
    int32_t in_memory = 0;
    __device__ Queue() {
        for (int i = 0; i < kHeld; ++i) { key[i] = kNoKey; b[i] = 0; }
    }
};

__device__ __forceinline__ void queue_push(uint64_t *h, Queue &q, uint64_t key, uint32_t b = 0) {
#pragma unroll
    for (int i = 0; i < kHeld; ++i) {
        const uint64_t k0 = q.key[i];
        const uint32_t b0 = q.b[i];
        const bool before = key < k0;
        q.key[i] = before ? key : k0;
        q.b[i] = before ? b : b0;
        key = before ? k0 : key;
        b = before ? b0 : b;
    }
    if (key != kNoKey) heap_push(h, q.in_memory, key);
}

// Taking the smallest key and bringing the next one into the registers are two calls, so that
// the caller can start the loads that depend on the key before the heap in memory is put in
// order again.  Nothing else may touch the queue in between.
__device__ __forceinline__ uint64_t queue_take(Queue &q) {
    const uint64_t out = q.key[0];
#pragma unroll
    for (int i = 0; i + 1 < kHeld; ++i) {
        q.key[i] = q.key[i + 1];
        q.b[i] = q.b[i + 1];
    }
    q.key[kHeld - 1] = kNoKey;
    return out;
}

// Whether a key came from memory, whose b the caller then has to ask for.
__device__ __forceinline__ bool queue_refill(uint64_t *h, Queue &q) {
    if (q.in_memory == 0) return false;
    q.key[kHeld - 1] = heap_pop(h, q.in_memory);
    return true;
}

// b(z) of the lane's partition as it is in memory, anything outside 32 bits as ~0; used, a value outside [0, 2^31) is
// reported and replaced by 0.  Two steps, so that several loads of 32 bits can be on their way.
__device__ __forceinline__ uint32_t load_b(const uint8_t *bq, int32_t z, int64_t bsv, int32_t b_bytes) {
    if (b_bytes == 4) return *(const uint32_t *)(bq + (int64_t)z * bsv * 4);
    const uint64_t wide = *(const uint64_t *)(bq + (int64_t)z * bsv * 8);
    return wide >> 32 ? 0xffffffffu : (uint32_t)wide;
}
__device__ __forceinline__ uint64_t available_key(uint32_t b, int32_t z, bool &bad) {
    if (b > 0x7fffffffu) { bad = true; b = 0; }
    return ((uint64_t)(0x7fffffffu - b) << 32) | (uint32_t)z;
}

// How much of a partition's state a wavefront with one partition keeps in LDS.  A step is a chain of dependent
// memory round trips, and the batch's state is far larger than the L2: what sits in LDS leaves that chain and
// the traffic.  kOwnersAndInputs (1.5 bytes a vertex, 2 with in-degrees past 15): the device of every vertex and
// the open inputs, which every edge of a started vertex asks for.  kAll (6 bytes more): the ready times and the
// inboxes too; then nothing that two lanes exchange is in memory, and a step waits for no store.  Measured
// against the state in memory: 5,271 vertices, 50 devices, 4,096 partitions (16 wavefronts
// per compute unit, owners and inputs kept; 3.93 with the near inbox below) 5.73 -> 4.55 ms; 1,124 vertices, 26 devices, 1,957 partitions (all
// kept) 1.83 -> 0.90 ms.
enum Resident { kNothing, kOwnersAndInputs, kNearInboxToo, kAll };

// kNearInboxToo: the first two vertices handed to a device in a step wait in LDS, the others in its inbox in memory,
// which then costs most steps neither a store to wait for nor a round trip (5,271 vertices, 50 devices, 4,096
// partitions: PCT 4.46 -> 3.93 ms, FIFO 3.88 -> 3.40, before the records).  From kNearFrom wavefronts a compute unit on: one alone finds its
// inbox in the L1 (24,000 vertices, 8 devices: 64 and 256 partitions 1.02 times as long with it, 512 as long,
// 1,024 0.98, on 50 devices 0.96).  Two, because the static LDS then still is kSimStaticLds; 16 bits, because state in LDS
// means at most 43,690 vertices.
constexpr size_t kNearFrom = 3;
constexpr int32_t kNearInbox = 2;
static_assert(3 * 64 * sizeof(int32_t) + 64 * kNearInbox * sizeof(uint16_t) <= kSimStaticLds, "fits() counts on it");

// An entry of the cost tables, and ceil(a / d) by it.
template <bool MAGIC> struct DivisorOf {
    Magic m = {0, 0};
};
template <> struct DivisorOf<false> {
    int64_t d = 1;
};
template <typename WT> __device__ __forceinline__ uint32_t quotient(WT a, const DivisorOf<true> &by) {
    return magic_div((uint32_t)a, by.m);
}
template <typename WT> __device__ __forceinline__ uint32_t quotient(WT a, const DivisorOf<false> &by) {
    return (uint32_t)plain_div((uint64_t)a, (uint64_t)by.d);
}

struct SimArgs {
    const int32_t *ptr;        // successor CSR over original ids
    const int32_t *idx;
    const void *wt;            // t(e) in that order
    const void *c;
    const uint4 *records;      // [n][2] or null: see simulate_records_kernel
    const int32_t *pred_ptr;   // predecessor CSR row bounds: the in-degrees
    const uint8_t *assign;
    int64_t a_stride_p, a_stride_v;
    const void *b;             // PCT: ticks, b(v, q) at v * b_sv + q * b_sq
    int64_t b_sv, b_sq;
    int32_t b_bytes;
    const int32_t *tie;        // FIFO: rank of a vertex among equal ready times, null = its number
    const int32_t *tie_inv;    //       vertex of a rank
    const void *edge_tab;      // row = device of the edge's source vertex
    const void *vert_tab;
    int32_t *ready;            // [P][n] latest arrival so far
    int32_t *need;             // [P][n] inputs whose producer has not started
    int32_t *inbox;            // [P][n], one segment per device
    uint64_t *pending;         // [P][n], one segment per device
    uint64_t *available;       // [P][n], PCT only
    long long *makespan;       // [P]
    int32_t *start;            // [P][n] or null
    int32_t *status;
    int32_t n, P, k;
    int32_t groups;            // partitions per wavefront, <= 64 / k
    uint32_t window;           // lanes with T - T_min <= window decide together
    int32_t need_bits;         // LDS: bits of an open-input count, 4 or 8
};

// What a step reads of a vertex, 32 bytes: c, its out-edges' number, and up to kRecordEdges of them as (head, t), or the
// number of the first one.  A lane's loads go to lines of their own, and the address unit and the L1 were busy two thirds
// of the time: one line in place of four (c, row bounds, heads, t), and a round trip less where the edges are in it.
// 5,271 vertices on 50 devices, ms as it is, without the records, with one key of a queue in a register, and with b asked for
// only where a vertex becomes available:
//   out-edges 1 to 3, PCT,    256 partitions  1.38  1.47  1.49  1.42
//                           1,024             1.53  1.63  1.64  1.58
//                           4,096             3.10  3.36  3.67  3.33
//                     FIFO, 4,096             2.90  3.17  3.06  2.90
//   out-edges 1 to 7, PCT,  4,096             4.47  4.63  4.95  4.71   (four in seven have too many for the record)
// Not where the mean row is longer than a record holds: the record is then one more line to most steps.  Over 600 calls (100 to 25,000
// vertices, 1 to 64 devices) records took 0.96 times as long as none at 2 to 3 edges a vertex, 1.00 at 3 to 5 and 1.03 at 5
// to 9 (11,500 vertices of nine edges, one device, ten partitions, FIFO 70 ms a call, 61 before there were records).
// The launch that writes them takes some 5 us; they stand where the open inputs would be in memory, so not beside those.
constexpr int32_t kRecordEdges = 3, kRecordsFrom = 8;       // (8 words a vertex, one for each of 8 partitions)
__global__ __launch_bounds__(256) void simulate_records_kernel(const int32_t *__restrict__ ptr,
                                                               const int32_t *__restrict__ idx,
                                                               const uint32_t *__restrict__ wt,
                                                               const uint32_t *__restrict__ c, int32_t n,
                                                               uint4 *__restrict__ records) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    const int32_t e0 = ptr[v], degree = ptr[v + 1] - e0;
    uint32_t w[2 * kRecordEdges] = {};
    if (degree > kRecordEdges) {
        w[0] = (uint32_t)e0;
    } else {
#pragma unroll
        for (int j = 0; j < kRecordEdges; ++j) {
            if (j < degree) {
                w[2 * j] = (uint32_t)idx[e0 + j];
                w[2 * j + 1] = wt[e0 + j];
            }
        }
    }
    records[2 * v] = make_uint4(c[v], (uint32_t)degree, w[0], w[1]);
    records[2 * v + 1] = make_uint4(w[2], w[3], w[4], w[5]);
}

template <typename WT, bool MAGIC, bool PCT, int KEEP, bool RECORDS>
__global__ __launch_bounds__(64) void simulate_kernel(SimArgs a) {
    extern __shared__ uint32_t sim_lds[];
    __shared__ int32_t count[64];      // vertices per device, then handed to it so far (kNearInboxToo: in this step)
    __shared__ int32_t seg[64];        // first slot of the device's segment
    __shared__ int32_t gbad[64];       // per group: a device id >= k was seen
    __shared__ uint16_t near_in[64][kNearInbox];       // kNearInboxToo: the first vertices handed over in a step
    const int lane = threadIdx.x;
    const int32_t n = a.n, k = a.k;
    // with k <= 32 devices a wavefront can hold up to 64 / k partitions side by side: group g =
    // lanes g*k .. g*k + k-1.  Lanes past the last group, and groups past the batch, idle.
    const int groups = a.groups;
    const int grp = lane / k, dev = lane - grp * k;
    const int first = grp * k;
    const int64_t q = (int64_t)blockIdx.x * groups + grp;
    bool alive = grp < groups && q < a.P;
    // Idle lanes keep their pointers in range; with state in LDS (one partition) they help to set it up.
    const int64_t qq = KEEP != kNothing ? (int64_t)blockIdx.x : (alive ? q : 0);
    const uint8_t *row = a.assign + qq * a.a_stride_p;
    const int64_t asv = a.a_stride_v;
    const WT *wt = (const WT *)a.wt;
    const WT *cw = (const WT *)a.c;
    using Divisor = DivisorOf<MAGIC>;
    const Divisor *etab = (const Divisor *)a.edge_tab, *vtab = (const Divisor *)a.vert_tab;
    int32_t *ready = a.ready + qq * n;
    int32_t *need = a.need + qq * n;
    int32_t *start = a.start ? a.start + qq * n : nullptr;
    // LDS (one partition per wavefront): counts packed into words, [ready times,] devices, [inboxes]
    const int nb_sh = a.need_bits == 4 ? 3 : 2;                    // counts per word, as a shift
    uint32_t *l_need = sim_lds;
    uint32_t *l_ready = l_need + ((n + (1 << nb_sh) - 1) >> nb_sh);
    uint8_t *l_dev = (uint8_t *)(l_ready + (KEEP == kAll ? n : 0));
    uint16_t *l_inbox = (uint16_t *)(l_dev + ((n + 3) & ~3));
    auto need_at = [&](int32_t v) { return (v & ((1 << nb_sh) - 1)) * a.need_bits; };
    auto owner = [&](int32_t v) { return KEEP != kNothing ? (uint32_t)l_dev[v] : (uint32_t)row[(int64_t)v * asv]; };

    if (*a.status & CP_STATUS_BAD_TIE) {          // set by the check of the tie ranks, same stream
        if (alive && dev == 0) a.makespan[q] = -1;
        return;
    }

    // ---- set-up: vertices per device, state of every vertex
    count[lane] = 0;
    gbad[lane] = 0;
    __syncthreads();
    if (KEEP != kNothing) {
        for (int32_t i = lane; i < (n + (1 << nb_sh) - 1) >> nb_sh; i += 64) l_need[i] = 0;
        __syncthreads();
        for (int32_t v = lane; v < n; v += 64) {
            const uint32_t d = row[(int64_t)v * asv];
            l_dev[v] = (uint8_t)d;
            atomicOr(&l_need[v >> nb_sh], (uint32_t)(a.pred_ptr[v + 1] - a.pred_ptr[v]) << need_at(v));
            if (KEEP == kAll) l_ready[v] = 0;
            else ready[v] = 0;
            if (d >= (uint32_t)k) gbad[grp < groups ? grp : 0] = 1;
            else atomicAdd(&count[d], 1);
        }
    } else if (alive) {
        for (int32_t v = dev; v < n; v += k) {
            const uint32_t d = row[(int64_t)v * asv];
            if (d >= (uint32_t)k) { gbad[grp] = 1; continue; }
            atomicAdd(&count[first + d], 1);
            ready[v] = 0;
            need[v] = a.pred_ptr[v + 1] - a.pred_ptr[v];
        }
    }
    __syncthreads();
    if (alive && gbad[grp]) {
        alive = false;
        if (dev == 0) {
            atomicOr(a.status, CP_STATUS_BAD_DEVICE_ID);
            a.makespan[q] = -1;
        }
    }
    {
        const int32_t mine = alive ? count[lane] : 0;
        int32_t incl = mine;
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t other = __shfl_up(incl, off);
            if (lane >= off) incl += other;
        }
        const int32_t below = __shfl(incl, first > 0 ? first - 1 : 0);   // total of the groups before this one
        __syncthreads();
        seg[lane] = incl - mine - (first > 0 ? below : 0);
        count[lane] = 0;
    }
    step_fence();
    int32_t *inbox = a.inbox + qq * n;
    const int64_t bsv = a.b_sv;
    const uint8_t *bq = (const uint8_t *)a.b + (PCT ? qq * a.b_sq * a.b_bytes : 0);
    bool b_bad = false;
    if (alive) {
        for (int32_t v = dev; v < n; v += k) {
            if (a.pred_ptr[v + 1] == a.pred_ptr[v]) {
                const uint32_t d = owner(v);
                const int32_t pos = atomicAdd(&count[first + d], 1);
                if (KEEP == kAll) l_inbox[seg[first + d] + pos] = (uint16_t)v;
                else if (KEEP == kNearInboxToo && pos < kNearInbox) near_in[d][pos] = (uint16_t)v;
                else inbox_store(inbox + seg[first + d] + pos, v);
            }
        }
    }
    step_fence();

    // ---- the event loop
    const int32_t base = seg[lane];
    uint64_t *hp = a.pending + qq * n + base;
    uint64_t *ha = PCT ? a.available + qq * n + base : nullptr;
    const int32_t *my_inbox = inbox + base;
    const int last_lane = min(first + k - 1, 63);
    Queue pending, available;
    const Divisor my_speed = vtab[dev];
    int32_t taken = 0, done = 0;
    uint32_t free_at = 0;
    // what a started vertex does to a successor of its own partition
    auto raise_ready = [&](int32_t z, uint32_t arrival) {
        if (KEEP == kAll) atomicMax(&l_ready[z], arrival);
        else __hip_atomic_fetch_max(ready + z, (int32_t)arrival, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto take_input = [&](int32_t z) -> int32_t {
        if (KEEP == kNothing)
            return __hip_atomic_fetch_add(need + z, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const uint32_t old = atomicSub(&l_need[z >> nb_sh], 1u << need_at(z));
        return (int32_t)((old >> need_at(z)) & ((1u << a.need_bits) - 1));
    };
    auto hand_over = [&](int32_t z, uint32_t d) {
        const int to = (KEEP != kNothing ? 0 : first) + (int)d;    // idle lanes help with wide rows: not their first
        const int32_t pos = atomicAdd(&count[to], 1);
        if (KEEP == kAll) l_inbox[seg[to] + pos] = (uint16_t)z;
        else if (KEEP == kNearInboxToo && pos < kNearInbox) near_in[to][pos] = (uint16_t)z;
        else inbox_store(inbox + seg[to] + pos, z);
    };
    // vertices of its inbox that a device looks at side by side: large graphs hand over many in a step (200,000 vertices of up
    // to 7 out-edges on 8 devices, 64 partitions: one at a time 1.2 % slower), small ones one or two (5,271 vertices, 50
    // devices, 256 partitions: three at a time 5 % slower)
    constexpr int32_t kDrain = KEEP == kNothing ? 4 : 1;
    // every step with work left starts at least one vertex in every unfinished group, so
    // n + 1 steps always suffice
    for (int64_t step = 0; step <= n; ++step) {
        if (alive) {   // vertices handed to this device since its last step
            const int32_t have = count[lane];
            if (KEEP == kNearInboxToo) {            // what is handed over in a step is numbered from 0
                taken = 0;
                count[lane] = 0;
            }
            while (taken < have) {
                const int32_t cnt = min(kDrain, have - taken);
                int32_t z[kDrain];
                uint32_t rz[kDrain], bz[kDrain], low[kDrain];
#pragma unroll
                for (int j = 0; j < kDrain; ++j) {
                    const int32_t at = taken + min(j, cnt - 1);
                    if (KEEP == kAll) z[j] = (int32_t)l_inbox[base + at];
                    else if (KEEP == kNearInboxToo && at < kNearInbox) z[j] = (int32_t)near_in[lane][at];
                    else z[j] = inbox_load(my_inbox + at);
                }
#pragma unroll
                for (int j = 0; j < kDrain; ++j) {
                    rz[j] = KEEP == kAll ? l_ready[z[j]] : (uint32_t)l2_read(ready + z[j]);
                    bz[j] = PCT ? load_b(bq, z[j], bsv, a.b_bytes) : 0u;
                    low[j] = !PCT && a.tie ? (uint32_t)a.tie[z[j]] : (uint32_t)z[j];
                }
#pragma unroll
                for (int j = 0; j < kDrain; ++j) {
                    if (j < cnt) {
                        if (PCT && rz[j] <= free_at)    // executable at every decision this device has still to take
                            queue_push(ha, available, available_key(bz[j], z[j], b_bad));
                        else
                            queue_push(hp, pending, ((uint64_t)rz[j] << 32) | low[j], bz[j]);
                    }
                }
                taken += cnt;
            }
        }
        uint32_t T = kNever;
        if (PCT && available.key[0] != kNoKey) T = free_at;
        else if (pending.key[0] != kNoKey) T = max(free_at, (uint32_t)(pending.key[0] >> 32));
        // the group's earliest decision time (several groups: a running minimum over each
        // group's lanes, read from its last lane)
        uint32_t tmin = T;
        if (groups == 1) {
            // one partition in the wavefront: the minimum of each row of 16 lanes by register
            // permutations, then the four rows' minima through scalar registers
            tmin = min(tmin, dpp_u32<0xB1>(tmin));      // swap neighbours
            tmin = min(tmin, dpp_u32<0x4E>(tmin));      // swap pairs
            tmin = min(tmin, dpp_u32<0x141>(tmin));     // mirror halves of 8
            tmin = min(tmin, dpp_u32<0x140>(tmin));     // mirror the row
            tmin = min(min((uint32_t)__builtin_amdgcn_readlane((int)tmin, 0),
                           (uint32_t)__builtin_amdgcn_readlane((int)tmin, 16)),
                       min((uint32_t)__builtin_amdgcn_readlane((int)tmin, 32),
                           (uint32_t)__builtin_amdgcn_readlane((int)tmin, 48)));
        } else {
            for (int off = 1; off < k; off <<= 1) {
                const uint32_t other = (uint32_t)__shfl_up((int)tmin, off);
                if (dev >= off) tmin = min(tmin, other);
            }
            tmin = (uint32_t)__shfl((int)tmin, last_lane);
        }
        if (__all(tmin == kNever)) break;
        int32_t wide_e0 = 0, wide_e1 = 0;     // a long row is left to the whole wavefront below
        if (T != kNever && T - tmin <= a.window) {
            int32_t v;
            if (PCT) {
                for (int32_t moved = 0; (uint32_t)(pending.key[0] >> 32) <= T && moved < n; ++moved) {
                    const uint32_t bz = pending.b[0];
                    const int32_t z = (int32_t)(uint32_t)queue_take(pending);
                    if (queue_refill(hp, pending))
                        pending.b[kHeld - 1] = load_b(bq, (int32_t)(uint32_t)pending.key[kHeld - 1], bsv, a.b_bytes);
                    queue_push(ha, available, available_key(bz, z, b_bad));
                }
                v = (int32_t)(uint32_t)queue_take(available);
            } else {
                const uint32_t low = (uint32_t)queue_take(pending);
                v = a.tie_inv ? a.tie_inv[low] : (int32_t)low;
            }
            // what the vertex needs from the graph is on its way while the queue is put in order
            uint4 r0, r1;
            WT cv;
            int32_t e0, degree;
            if (RECORDS) {
                r0 = a.records[2 * (int64_t)v];
                r1 = a.records[2 * (int64_t)v + 1];
                cv = (WT)r0.x;
                degree = (int32_t)r0.y;
                e0 = (int32_t)r0.z;
            } else {
                cv = cw[v];
                e0 = a.ptr[v];
                degree = a.ptr[v + 1] - e0;
            }
            if (PCT) queue_refill(ha, available);
            else queue_refill(hp, pending);
            if (start) start[v] = (int32_t)T;
            ++done;
            const uint32_t w = quotient(cv, my_speed);
            free_at = T + w;
            // the out-edges four at a time, so that the dependent loads of four edges (successor,
            // its device, the table entry) and their atomics overlap; slots past the row's end take
            // no part but for the table's first entries, whose loads need no branch
            const bool held = RECORDS && degree <= kRecordEdges;      // in the record
            if (degree >= kWideRow) {
                wide_e0 = e0;
                wide_e1 = e0 + degree;
                degree = 0;
            }
            for (int32_t i = 0; i < degree; i += 4) {
                const int32_t cnt = min(4, degree - i), e = e0 + i;
                int32_t z[4], before[4];
                WT te[4];
                uint32_t dz[4], arrive[4];
                Divisor by[4];
                if (held) {
                    z[0] = (int32_t)r0.z; te[0] = (WT)r0.w;
                    z[1] = (int32_t)r1.x; te[1] = (WT)r1.y;
                    z[2] = (int32_t)r1.z; te[2] = (WT)r1.w;
                    z[3] = 0; te[3] = 0;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int32_t ej = e + min(j, cnt - 1);
                        z[j] = a.idx[ej];
                        te[j] = wt[ej];
                    }
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) dz[j] = owner(z[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j) by[j] = etab[dev * k + dz[j]];
#pragma unroll
                for (int j = 0; j < 4; ++j) arrive[j] = free_at + quotient(te[j], by[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (j < cnt) raise_ready(z[j], arrive[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    before[j] = 0;
                    if (j < cnt) before[j] = take_input(z[j]);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (before[j] == 1) hand_over(z[j], dz[j]);
            }
        }
        // long rows (hubs), one after the other, 64 edges at a time: every lane of the wavefront,
        // whatever its own partition, works for the lane that started the hub
        for (unsigned long long wide = __ballot(wide_e1 > wide_e0); wide; wide &= wide - 1) {
            const int src = __ffsll((long long)wide) - 1;
            const int32_t he0 = __shfl(wide_e0, src), he1 = __shfl(wide_e1, src);
            const uint32_t hfree = (uint32_t)__shfl((int)free_at, src);
            const int hdev = __shfl(dev, src), hfirst = __shfl(first, src);
            const int64_t hq = ((int64_t)__shfl((int)(qq >> 32), src) << 32) | (uint32_t)__shfl((int)(uint32_t)qq, src);
            const uint8_t *hrow = a.assign + hq * a.a_stride_p;
            int32_t *hready = a.ready + hq * n, *hneed = a.need + hq * n, *hinbox = a.inbox + hq * n;
            for (int32_t e = he0 + lane; e < he1; e += 64) {
                const int32_t z = a.idx[e];
                const WT te = wt[e];
                const uint32_t dz = KEEP != kNothing ? (uint32_t)l_dev[z] : (uint32_t)hrow[(int64_t)z * asv];
                const uint32_t x = quotient(te, etab[hdev * k + dz]);
                if (KEEP != kNothing) {              // the wavefront's only partition
                    raise_ready(z, hfree + x);
                    if (take_input(z) == 1) hand_over(z, dz);
                    continue;
                }
                __hip_atomic_fetch_max(hready + z, (int32_t)(hfree + x), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                const int32_t before = __hip_atomic_fetch_add(hneed + z, -1, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_WORKGROUP);
                if (before == 1) {
                    const int32_t pos = atomicAdd(&count[hfirst + dz], 1);
                    inbox_store(hinbox + seg[hfirst + dz] + pos, z);
                }
            }
        }
        if (KEEP == kAll) {
            // what lanes exchange is in LDS, which serves a wavefront in order
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");
            __builtin_amdgcn_wave_barrier();
        } else {
            step_fence(); // everything this step wrote is in place before the next step reads it
        }
    }
    uint32_t last = free_at;
    int32_t total = done;
    for (int off = 1; off < k; off <<= 1) {
        const uint32_t o1 = (uint32_t)__shfl_up((int)last, off);
        const int32_t o2 = __shfl_up(total, off);
        if (dev >= off) {
            last = max(last, o1);
            total += o2;
        }
    }
    if (__any(b_bad) && lane == 0) atomicOr(a.status, CP_STATUS_B_OUT_OF_RANGE);
    if (alive && dev == k - 1) {
        if (total != n) {
            atomicOr(a.status, CP_STATUS_INCOMPLETE);
            a.makespan[q] = -1;
        } else {
            a.makespan[q] = (long long)last;
        }
    }
}

// tie_inv[tie[v]] = v; a rank outside [0, n) is reported.  tie_inv starts at -1.
__global__ __launch_bounds__(256) void tie_scatter_kernel(const int32_t *tie, int32_t n, int32_t *tie_inv,
                                                          int32_t *status) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    const int32_t r = tie[v];
    if (r < 0 || r >= n) atomicOr(status, CP_STATUS_BAD_TIE);
    else tie_inv[r] = (int32_t)v;
}

// A rank nobody has means another rank was given twice: not a permutation.
__global__ __launch_bounds__(256) void tie_check_kernel(const int32_t *tie_inv, int32_t n, int32_t *status) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r < n && tie_inv[r] < 0) atomicOr(status, CP_STATUS_BAD_TIE);
}

__global__ __launch_bounds__(256) void fill_minus_one_kernel(int32_t *dst, int32_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = -1;
}

}  // namespace

int launch_simulate(const SimulateLaunch &s, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    if (s.n < 1 || s.P < 1 || s.k < 1 || s.k > kWave) return CP_ERR_SIZE;
    if (s.tie) {
        const dim3 grid((unsigned)((s.n + 255) / 256)), block(256);
        hipLaunchKernelGGL(fill_minus_one_kernel, grid, block, 0, st, s.tie_inv, s.n);
        hipLaunchKernelGGL(tie_scatter_kernel, grid, block, 0, st, s.tie, s.n, s.tie_inv, s.status);
        hipLaunchKernelGGL(tie_check_kernel, grid, block, 0, st, s.tie_inv, s.n, s.status);
    }
    SimArgs a{};
    a.ptr = (const int32_t *)(s.blob + s.succ->ptr_off);
    a.idx = (const int32_t *)(s.blob + s.succ->idx_off);
    a.wt = s.blob + s.succ->wt_off;
    a.c = s.blob + s.c_off;
    a.pred_ptr = (const int32_t *)(s.blob + s.pred->ptr_off);
    a.assign = s.assign;
    a.a_stride_p = s.a_stride_p;
    a.a_stride_v = s.a_stride_v;
    a.b = s.b;
    a.b_sv = s.b_sv;
    a.b_sq = s.b_sq;
    a.b_bytes = s.b_bytes;
    a.tie = s.tie;
    a.tie_inv = s.tie ? s.tie_inv : nullptr;
    a.edge_tab = s.edge_tab;
    a.vert_tab = s.vert_tab;
    a.ready = s.ready;
    a.need = s.need;
    a.inbox = s.inbox;
    a.pending = s.pending;
    a.available = s.available;
    a.makespan = (long long *)s.makespan;
    a.start = s.start;
    a.status = s.status;
    a.n = s.n; a.P = s.P; a.k = s.k;
    a.window = s.window;
    const int groups = std::max(1, std::min(s.groups, kWave / s.k));      // partitions per wavefront
    a.groups = groups;
    // The most that fits the LDS beside every wavefront the batch puts on a compute unit, at most kSimWaves of
    // them: more wavefronts in flight hide more of the round trips than the state in LDS saves.  Wavefronts
    // that share themselves out over several partitions (past 8,192) would need the room of each, and
    // in-degrees past 255 a wider count: their state stays in memory.
    a.need_bits = s.max_in_degree <= 15 ? 4 : 8;
    const size_t owners = (((size_t)s.n * a.need_bits / 8 + 7) & ~(size_t)3) + (((size_t)s.n + 3) & ~(size_t)3);
    const size_t all = owners + (size_t)s.n * 6;
    const size_t there = std::min<size_t>(kSimWaves, ((size_t)s.P + 255) / 256);
    auto fits = [&](size_t bytes) { return there * (bytes + kSimStaticLds) <= kLdsBudget && bytes <= 64 * 1024; };
    int keep = kNothing;
    if (groups == 1 && s.max_in_degree <= 255) {
        if (s.n <= 65535 && fits(all)) keep = kAll;
        else if (fits(owners)) keep = there < kNearFrom ? kOwnersAndInputs : kNearInboxToo;
    }
    // (the open inputs sit in LDS, and their array holds the records)
    if (keep != kNothing && s.narrow && s.P >= kRecordsFrom && s.m <= (int64_t)kRecordEdges * s.n) {
        a.records = (const uint4 *)s.need;
        hipLaunchKernelGGL(simulate_records_kernel, dim3((unsigned)((s.n + 255) / 256)), dim3(256), 0, st, a.ptr, a.idx,
                           (const uint32_t *)a.wt, (const uint32_t *)a.c, s.n, (uint4 *)s.need);
    }
    const size_t lds = keep == kAll ? all : (keep != kNothing ? owners : 0);
    const dim3 grid((unsigned)((s.P + groups - 1) / groups)), block(64);
#define CP_SIM_R(WT, MAGIC, PCT, KEEP)                                                                              \
    do {                                                                                                            \
        constexpr bool kCan = sizeof(WT) == 4;                                                                      \
        if (kCan && a.records)                                                                                      \
            hipLaunchKernelGGL((simulate_kernel<WT, MAGIC, PCT, KEEP, kCan>), grid, block, lds, st, a);             \
        else                                                                                                        \
            hipLaunchKernelGGL((simulate_kernel<WT, MAGIC, PCT, KEEP, false>), grid, block, lds, st, a);            \
    } while (0)
#define CP_SIM_K(WT, MAGIC, PCT)                                                                                    \
    do {                                                                                                            \
        if (keep == kAll) CP_SIM_R(WT, MAGIC, PCT, kAll);                                                           \
        else if (keep == kNearInboxToo) CP_SIM_R(WT, MAGIC, PCT, kNearInboxToo);                                    \
        else if (keep == kOwnersAndInputs) CP_SIM_R(WT, MAGIC, PCT, kOwnersAndInputs);                              \
        else hipLaunchKernelGGL((simulate_kernel<WT, MAGIC, PCT, kNothing, false>), grid, block, 0, st, a);         \
    } while (0)
#define CP_SIM(WT, MAGIC)                       \
    do {                                        \
        if (s.pct) CP_SIM_K(WT, MAGIC, true);   \
        else CP_SIM_K(WT, MAGIC, false);        \
    } while (0)
    if (s.magic) CP_SIM(uint32_t, true);
    else if (s.narrow) CP_SIM(uint32_t, false);
    else CP_SIM(int64_t, false);
#undef CP_SIM
#undef CP_SIM_K
#undef CP_SIM_R
    return hipGetLastError() == hipSuccess ? CP_OK : CP_ERR_HIP;
}

}  // namespace cpeval
