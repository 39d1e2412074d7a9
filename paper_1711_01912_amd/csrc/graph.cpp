// Host side of cp_graph_create: validation of the caller's arrays and packing
// into the device image used by the two kernel families.  No GPU call here.
#include <algorithm>
#include <cstring>
#include <future>
#include <memory>
#include <new>
#include <numeric>
#include <system_error>

#include "cpeval_internal.hpp"

namespace cpeval {
namespace {

struct BlobWriter {
    std::vector<uint8_t> &buf;
    explicit BlobWriter(std::vector<uint8_t> &b) : buf(b) {}
    size_t reserve(size_t bytes) {
        size_t off = align_up(buf.size());
        buf.resize(off + bytes, 0);
        return off;
    }
    template <typename T> T *at(size_t off) { return reinterpret_cast<T *>(buf.data() + off); }
};

struct Csr {
    const int32_t *ptr;
    const int32_t *idx;
    std::vector<int64_t> wt;  // t(e) in this CSR's order
};

int check_csr(int32_t n, int64_t m, const int32_t *ptr, const int32_t *idx) {
    if (ptr[0] != 0 || (int64_t)ptr[n] != m) return CP_ERR_CSR;
    for (int32_t v = 0; v < n; ++v)
        if (ptr[v + 1] < ptr[v]) return CP_ERR_CSR;
    for (int64_t e = 0; e < m; ++e)
        if (idx[e] < 0 || idx[e] >= n) return CP_ERR_CSR;
    return CP_OK;
}

// Vertices in sweep order: levels first-to-last (forward) or last-to-first, and
// inside a level the longest rows first, so that hubs lead and rows of similar
// length share a wavefront.
void sweep_order(int32_t n, int32_t L, const int32_t *level_ptr, const int32_t *level_vtx,
                 const int32_t *ptr, bool forward, std::vector<int32_t> &order, ColumnDir &dir) {
    order.resize(n);
    dir.lvl_begin.assign(L, 0);
    dir.lvl_hubs.assign(L, 0);
    dir.lvl_count.assign(L, 0);
    dir.lvl_longest.assign(L, 0);
    dir.lvl_split.assign(L, 0);
    int32_t pos = 0;
    for (int32_t s = 0; s < L; ++s) {
        int32_t l = forward ? s : L - 1 - s;
        int32_t a = level_ptr[l], b = level_ptr[l + 1];
        std::copy(level_vtx + a, level_vtx + b, order.begin() + pos);
        std::stable_sort(order.begin() + pos, order.begin() + pos + (b - a),
                         [&](int32_t x, int32_t y) {
                             return ptr[x + 1] - ptr[x] > ptr[y + 1] - ptr[y];
                         });
        int32_t hubs = 0;
        while (hubs < b - a) {
            int32_t v = order[pos + hubs];
            if (ptr[v + 1] - ptr[v] < kHubDegree) break;
            ++hubs;
        }
        int32_t split = hubs;
        while (split < b - a && ptr[order[pos + split] + 1] - ptr[order[pos + split]] >= kColumnSplit) ++split;
        dir.lvl_split[s] = split - hubs;
        dir.lvl_begin[s] = pos;
        dir.lvl_hubs[s] = hubs;
        dir.lvl_count[s] = b - a;
        if (hubs < b - a) dir.lvl_longest[s] = ptr[order[pos + hubs] + 1] - ptr[order[pos + hubs]];
        pos += b - a;
    }
}

void pack_column_dir(BlobWriter &w, int32_t n, int64_t m, bool narrow, const Csr &csr,
                     const std::vector<int32_t> &order, ColumnDir &dir) {
    dir.ptr_off = w.reserve(sizeof(int32_t) * ((size_t)n + 1));
    std::memcpy(w.at<int32_t>(dir.ptr_off), csr.ptr, sizeof(int32_t) * ((size_t)n + 1));
    dir.idx_off = w.reserve(sizeof(int32_t) * (size_t)std::max<int64_t>(m, 1));
    if (m) std::memcpy(w.at<int32_t>(dir.idx_off), csr.idx, sizeof(int32_t) * (size_t)m);
    if (narrow) {
        dir.wt_off = w.reserve(sizeof(uint32_t) * (size_t)std::max<int64_t>(m, 1));
        uint32_t *p = w.at<uint32_t>(dir.wt_off);
        for (int64_t e = 0; e < m; ++e) p[e] = (uint32_t)csr.wt[e];
    } else {
        dir.wt_off = w.reserve(sizeof(int64_t) * (size_t)std::max<int64_t>(m, 1));
        if (m) std::memcpy(w.at<int64_t>(dir.wt_off), csr.wt.data(), sizeof(int64_t) * (size_t)m);
    }
    dir.order_off = w.reserve(sizeof(int32_t) * (size_t)n);
    std::memcpy(w.at<int32_t>(dir.order_off), order.data(), sizeof(int32_t) * (size_t)n);
    dir.rows_off = w.reserve(sizeof(int32_t) * 4 * (size_t)n);
    int32_t *rows = w.at<int32_t>(dir.rows_off);
    const size_t L = dir.lvl_begin.size();
    for (size_t l = 0; l < L; ++l)
        for (int32_t i = dir.lvl_begin[l]; i < dir.lvl_begin[l] + dir.lvl_count[l]; ++i) {
            const int32_t v = order[i];
            rows[4 * (size_t)i] = v;
            rows[4 * (size_t)i + 1] = csr.ptr[v];
            rows[4 * (size_t)i + 2] = csr.ptr[v + 1];
            rows[4 * (size_t)i + 3] = (int32_t)l;
        }
    dir.lvl_off = w.reserve(sizeof(int32_t) * 4 * std::max<size_t>(L, 1));
    int32_t *lvl = w.at<int32_t>(dir.lvl_off);
    for (size_t l = 0; l < L; ++l) {
        lvl[4 * l] = dir.lvl_begin[l];
        lvl[4 * l + 1] = dir.lvl_hubs[l];
        lvl[4 * l + 2] = dir.lvl_count[l];
        lvl[4 * l + 3] = 0;
    }
}

// A slice with few rows spreads each row over several lanes: log2 of the lanes
// per row for a slice of `rows` vertices.
int lanes_per_row_log2(int rows) {
    int sh = 0;
    while ((rows << (sh + 1)) <= kWave) ++sh;
    return sh;
}

// Resident-window packing for one direction (layout: see WindowDir).  Returns
// false if the graph does not suit that plan.
bool pack_window_dir(BlobWriter &w, int32_t n, int32_t L, const int64_t *c, int64_t max_t,
                     bool ticks32, const Csr &csr, const std::vector<int32_t> &level_order,
                     const ColumnDir &col, WindowDir &dir) {
    // A slice is 64 consecutive positions of a level in the order the wave-column plan uses
    // (long rows first).  Inside a slice the order is free: by vertex number, so that the
    // lanes of an output store (and of the mask's reads of b) walk memory in one direction
    // and neighbouring lanes share cache lines.
    std::vector<int32_t> order(level_order);
    std::vector<int32_t> slice_deg((size_t)n, 0);       // longest row of the slice that starts at this position
    for (size_t s = 0; s < col.lvl_begin.size(); ++s) {
        const int32_t a = col.lvl_begin[s], b = a + col.lvl_count[s];
        for (int32_t p0 = a; p0 < b; p0 += kWave) {
            const int32_t e = std::min(b, p0 + kWave);
            int32_t deg = 0;
            for (int32_t i = p0; i < e; ++i) deg = std::max(deg, csr.ptr[order[i] + 1] - csr.ptr[order[i]]);
            slice_deg[p0] = deg;
            std::sort(order.begin() + p0, order.begin() + e);
        }
    }
    std::vector<int32_t> pos(n);
    for (int32_t i = 0; i < n; ++i) pos[order[i]] = i;

    auto slice_entries = [&](int32_t p0, int32_t rows) -> uint64_t {
        int64_t deg0 = slice_deg[p0];
        int sh = lanes_per_row_log2(rows);
        return (uint64_t)((deg0 + (1 << sh) - 1) >> sh) * kWave;
    };
    // Far edges: a neighbour computed kWindowFarTicks or more ticks earlier is not kept in
    // the ring; its value is read back from the output array by a far wavefront (32-bit
    // ticks only: the far values are staged as {value, device} pairs like the ring's).
    // Before the ticks are known the level distance stands in for the tick distance (a
    // level is at least one tick), which can only overestimate the ring.
    std::vector<int32_t> lvl_of((size_t)n);
    for (int32_t s = 0; s < L; ++s)
        for (int32_t i = col.lvl_begin[s]; i < col.lvl_begin[s] + col.lvl_count[s]; ++i) lvl_of[i] = s;
    // An upper bound of the ring capacity (exact value below, once the ticks are known)
    // fixes the entry format: the ring holds {value, device} pairs if that leaves room
    // for two stage slots and small cost tables, else separate arrays.
    auto ring_bound = [&](bool skip_far) {
        int64_t bound = 1;
        for (int32_t i = 0; i < n; ++i) {
            int32_t v = order[i];
            int32_t end = col.lvl_begin[lvl_of[i]] + col.lvl_count[lvl_of[i]];
            for (int32_t e = csr.ptr[v]; e < csr.ptr[v + 1]; ++e) {
                int32_t pn = pos[csr.idx[e]];
                if (skip_far && lvl_of[i] - lvl_of[pn] >= kWindowFarTicks) continue;
                bound = std::max<int64_t>(bound, (int64_t)end - pn);
            }
        }
        return bound;
    };
    auto pairs_fit = [&](int64_t slots, uint64_t far_bytes) {
        return 8 * ((uint64_t)slots + 1) + far_bytes + 2 * (kWindowTickBytes + 1024) + 4096 <= kLdsBudget - 512;
    };
    // far reads only where a ring of pairs for every neighbour does not fit
    int64_t need_ub = ring_bound(false);
    const bool far_allowed = ticks32 && !pairs_fit(need_ub, 0);
    if (far_allowed) need_ub = ring_bound(true);
    const uint64_t far_bytes_ub = far_allowed ? 2 * 8 * (uint64_t)kWave * kWindowMaxFarWaves : 0;
    dir.packed = ticks32 && pairs_fit(need_ub, far_bytes_ub);
    const uint64_t field_max = dir.packed ? 8 * (uint64_t)need_ub + 32 + far_bytes_ub : (uint64_t)need_ub;
    dir.ent4 = field_max < 65536 && max_t < 65536;
    const uint64_t esz = dir.ent4 ? 4 : 8;

    // Ticks: a level is cut into runs of at most kWindowTickSlices slices and about
    // kWindowTickBytes of packet, so that one typical packet size fits every tick
    // (vertices of one level do not depend on each other, so any cut is valid).
    std::vector<int32_t> tick_a, tick_b;
    for (int32_t s = 0; s < L; ++s) {
        int32_t a = col.lvl_begin[s], b = a + col.lvl_count[s];
        if (a == b) continue;
        int32_t start = a, nsl = 0;
        uint64_t bytes = 0;
        for (int32_t p0 = a; p0 < b; p0 += kWave) {
            int32_t rows = std::min(kWave, b - p0);
            uint64_t add = 8 * (uint64_t)kWave + esz * slice_entries(p0, rows);
            if (nsl > 0 && (nsl == kWindowTickSlices || bytes + add > kWindowTickBytes)) {
                tick_a.push_back(start);
                tick_b.push_back(p0);
                start = p0;
                nsl = 0;
                bytes = 0;
            }
            ++nsl;
            bytes += add;
        }
        tick_a.push_back(start);
        tick_b.push_back(b);
    }
    const int32_t T = (int32_t)tick_a.size();
    dir.ticks = T;

    std::vector<int32_t> tick_of((size_t)n);
    for (int32_t s = 0; s < T; ++s)
        for (int32_t i = tick_a[s]; i < tick_b[s]; ++i) tick_of[i] = s;
    // A neighbour far_ticks or more ticks back is a far read.  The smallest distance is the
    // one the far wavefronts' timing needs; it is doubled until the far reads of every tick
    // fit the far wavefronts (a longer ring for fewer far reads).
    const bool far_on = far_allowed && dir.packed;
    int32_t far_ticks = kWindowFarTicks;
    auto is_far = [&](int32_t s, int32_t pn) { return far_on && s - tick_of[pn] >= far_ticks; };
    int64_t need = 1, far_max = 0;
    for (;;) {
        need = 1;
        far_max = 0;
        for (int32_t s = 0; s < T; ++s) {
            int32_t a = tick_a[s], b = tick_b[s];
            int64_t far_here = 0;
            // a tick's vertices take consecutive slots with at most one wrap, whether or not
            // anything reads them: the ring is at least as long as the widest tick
            need = std::max<int64_t>(need, (int64_t)b - a);
            for (int32_t i = a; i < b; ++i) {
                int32_t v = order[i];
                for (int32_t e = csr.ptr[v]; e < csr.ptr[v + 1]; ++e) {
                    int32_t pn = pos[csr.idx[e]];
                    if (is_far(s, pn)) ++far_here;
                    else need = std::max<int64_t>(need, (int64_t)b - pn);
                }
            }
            far_max = std::max(far_max, far_here);
        }
        if (!far_on || far_max <= (int64_t)kWave * kWindowMaxFarWaves || far_ticks > T) break;
        far_ticks *= 2;
    }
    if (far_on && !pairs_fit(need, 2 * 8 * (uint64_t)((far_max + kWave - 1) / kWave * kWave))) return false;
    if (dir.ent4 && dir.packed && 8 * ((uint64_t)need + 1) + 32 + far_bytes_ub >= 65536) return false;

    int32_t wmax = 1;
    int64_t idspan = 1;
    std::vector<uint32_t> tick_tab(4 * ((size_t)T + 1), 0);   // {first chunk, chunks, lowest id, id span}
    uint64_t total = 0;
    uint32_t max_chunks = 1;
    for (int32_t s = 0; s < T; ++s) {
        int32_t a = tick_a[s], b = tick_b[s];
        wmax = std::max(wmax, b - a);
        int32_t lo = order[a], hi = order[a];
        for (int32_t i = a; i < b; ++i) { lo = std::min(lo, order[i]); hi = std::max(hi, order[i]); }
        idspan = std::max<int64_t>(idspan, (int64_t)hi - lo + 1);
        tick_tab[4 * s + 2] = (uint32_t)lo;
        tick_tab[4 * s + 3] = (uint32_t)(hi - lo + 1);
    }
    dir.slots = (int32_t)need;
    dir.far_cap = (int32_t)((far_max + kWave - 1) / kWave * kWave);
    if (dir.far_cap > kWave * kWindowMaxFarWaves) return false;    // too many far reads per tick
    dir.smax = (wmax + kWave - 1) / kWave;
    dir.wpad = dir.smax * kWave;
    if (dir.smax > kWindowMaxWaves - 1) return false;   // only when one slice alone exceeds every limit
    // the device ids of a tick can be staged straight from the caller's row when its
    // vertices occupy a short id range
    dir.direct_ok = idspan + 15 <= 4 * (int64_t)dir.wpad;
    dir.idpad = dir.direct_ok ? std::max<int32_t>(dir.wpad, (int32_t)((idspan + 15 + 15) / 16 * 16)) : dir.wpad;

    for (int32_t s = 0; s < T; ++s) {
        int32_t a = tick_a[s], b = tick_b[s];
        uint64_t nsl = (uint64_t)(b - a + kWave - 1) / kWave, entries = 0;
        for (int32_t p0 = a; p0 < b; p0 += kWave) entries += slice_entries(p0, std::min(kWave, b - p0));
        uint64_t bytes = 16 * (uint64_t)dir.smax + 8 * kWave * nsl + esz * entries;
        uint64_t chunks = (bytes + 15) / 16;
        if (chunks > (1u << 16)) return false;      // a 1 MB tick never fits LDS
        tick_tab[4 * s] = (uint32_t)total;
        tick_tab[4 * s + 1] = (uint32_t)chunks;
        total += chunks;
        if (total >= (1ull << 31)) return false;
        max_chunks = std::max<uint32_t>(max_chunks, (uint32_t)chunks);
    }
    tick_tab[4 * (size_t)T] = (uint32_t)total;
    dir.total_chunks = (int64_t)total;
    dir.max_chunks = (int32_t)max_chunks;

    // the stream is followed by slack: a wavefront that streams its own slices always fetches a
    // fixed number of entry rows, whatever the slice's width
    dir.stream_off = w.reserve(16 * ((size_t)std::max<uint64_t>(total, 1) + kStreamSlackChunks));
    const bool with_stab = dir.ent4 && dir.packed && dir.far_cap == 0;
    // ... and runs kStreamTailTicks ticks past the end with empty slices
    dir.stab_off = with_stab ? w.reserve(32 * ((size_t)T + kStreamTailTicks) * (size_t)dir.smax) : 0;
    dir.tick_off = w.reserve(sizeof(uint32_t) * tick_tab.size());
    std::memcpy(w.at<uint32_t>(dir.tick_off), tick_tab.data(), sizeof(uint32_t) * tick_tab.size());
    dir.gmap_off = w.reserve(sizeof(int32_t) * (size_t)std::max(T, 1) * dir.wpad);
    dir.far_off = w.reserve(8 * (size_t)std::max(dir.far_cap, 1) * (size_t)std::max(T, 1));
    // every reservation is made: the blob does not move any more
    int32_t *gmap = w.at<int32_t>(dir.gmap_off);
    uint32_t *far_list = w.at<uint32_t>(dir.far_off);
    uint32_t *stab = with_stab ? w.at<uint32_t>(dir.stab_off) : nullptr;
    dir.max_width = 0;
    std::fill(gmap, gmap + (size_t)std::max(T, 1) * dir.wpad, -1);

    // far reads of a tick: {vertex, c} per read, padded with vertex 0; the pairs they are
    // turned into sit behind the ring, one region per tick parity
    const uint32_t ring_bytes = (uint32_t)((8 * ((uint64_t)dir.slots + 1) + 15) & ~(uint64_t)15);
    if (dir.far_cap > 0 && dir.ent4 && ring_bytes + 2 * 8 * (uint64_t)dir.far_cap >= 65536) return false;

    const uint32_t pad_field = (uint32_t)(dir.packed ? 8 * (uint64_t)dir.slots : (uint64_t)dir.slots);
    for (int32_t s = 0; s < T; ++s) {
        int32_t a = tick_a[s], b = tick_b[s];
        uint32_t nsl = (uint32_t)(b - a + kWave - 1) / kWave;
        uint32_t far_next = 0;
        const uint32_t far_base = ring_bytes + (uint32_t)(s & 1) * 8u * (uint32_t)dir.far_cap;
        uint8_t *pk = w.at<uint8_t>(dir.stream_off + 16 * (size_t)tick_tab[4 * s]);
        uint32_t *desc = (uint32_t *)pk;
        uint32_t *rec = (uint32_t *)(pk + 16 * (size_t)dir.smax);         // nsl*64 x {v, c}
        const uint32_t ent_start = 16 * (uint32_t)dir.smax + 8 * kWave * nsl;
        uint32_t *ent = (uint32_t *)(pk + ent_start);
        uint32_t ebase = 0;                                               // in entries
        for (uint32_t j = 0; j < nsl; ++j) {
            int32_t p0 = a + (int32_t)j * kWave;
            int32_t rows = std::min(kWave, b - p0);
            int sh = lanes_per_row_log2(rows);
            int32_t lpr = 1 << sh;
            uint64_t width = (uint64_t)((slice_deg[p0] + lpr - 1) >> sh);
            if (width >= 65536) return false;
            desc[4 * j] = ent_start + (uint32_t)esz * ebase;
            desc[4 * j + 1] = (uint32_t)width | ((uint32_t)rows << 16) | ((uint32_t)sh << 24);
            desc[4 * j + 2] = tick_tab[4 * s + 2];
            desc[4 * j + 3] = (uint32_t)(p0 % dir.slots);
            dir.max_width = std::max(dir.max_width, (int32_t)width);
            if (stab) {
                uint32_t *e = stab + 8 * ((size_t)s * dir.smax + j);
                e[0] = tick_tab[4 * s] + (uint32_t)dir.smax + 32u * j;                  // 64 records of 8 bytes per slice
                e[1] = tick_tab[4 * s] + (ent_start + (uint32_t)esz * ebase) / 16;      // whole chunks: 64 entries a row
                e[2] = desc[4 * j + 1];
                e[3] = desc[4 * j + 2];
                e[4] = desc[4 * j + 3];
            }
            for (int32_t r = 0; r < kWave; ++r) {       // records: one per row
                uint32_t *rc = rec + 2 * ((size_t)j * kWave + r);
                if (r < rows) {
                    int32_t v = order[p0 + r];
                    rc[0] = (uint32_t)v;
                    rc[1] = (uint32_t)c[v];
                    gmap[(size_t)s * dir.wpad + (size_t)j * kWave + r] = v;
                } else {                                // padding row: never published
                    rc[0] = tick_tab[4 * s + 2];
                    rc[1] = 0;
                }
            }
            for (int32_t l = 0; l < kWave; ++l) {       // entries: lane l serves row l >> sh
                int32_t r = l >> sh, sub = l & (lpr - 1);
                int32_t v = r < rows ? order[p0 + r] : -1;
                int32_t d = v >= 0 ? csr.ptr[v + 1] - csr.ptr[v] : 0;
                for (uint32_t jj = 0; jj < (uint32_t)width; ++jj) {
                    const size_t at = (size_t)ebase + (size_t)jj * kWave + l;
                    int64_t ei = (int64_t)jj * lpr + sub;
                    uint32_t field = pad_field, te = 0;    // padding: the constant-zero slot
                    if (ei < d) {
                        int64_t e = (int64_t)csr.ptr[v] + ei;
                        int32_t pn = pos[csr.idx[e]];
                        if (is_far(s, pn)) {
                            uint32_t *fl = far_list + 2 * ((size_t)s * dir.far_cap + far_next);
                            fl[0] = (uint32_t)csr.idx[e];
                            fl[1] = (uint32_t)c[csr.idx[e]];
                            field = far_base + 8 * far_next;
                            ++far_next;
                        } else {
                            uint32_t slot = (uint32_t)(pn % dir.slots);
                            field = dir.packed ? 8 * slot : slot;
                        }
                        te = (uint32_t)csr.wt[e];
                    }
                    if (dir.ent4) {
                        ent[at] = field | (te << 16);
                    } else {
                        ent[2 * at] = field;
                        ent[2 * at + 1] = te;
                    }
                }
            }
            ebase += (uint32_t)width * kWave;
        }
        for (uint32_t j = nsl; stab && j < (uint32_t)dir.smax; ++j) {   // slices this tick does not have
            uint32_t *e = stab + 8 * ((size_t)s * dir.smax + j);
            e[0] = e[1] = tick_tab[4 * s];
            e[3] = tick_tab[4 * s + 2];
        }
    }
    return true;
}

// Positions and ticks of the lane-window plan, made level by level as far as somebody asks: a graph whose ring turns
// out too long costs its first levels, not all of them.  Positions go by level, inside a level by vertex number,
// so that outputs are written along rows; a tick is a run of at most kLaneTickVerts vertices of a level, and about
// kLaneTickBytes of packet.
struct LaneTicks {
    const ColumnDir &col;
    const Csr &csr;
    const int32_t *level_ptr, *level_vtx;
    const bool forward;
    const uint32_t row_bytes;            // of the packet, per sub-row
    const int shift;                     // log2 of the entries per sub-row
    std::unique_ptr<int32_t[]> order, pos, tick_of;      // filled for the levels made so far
    std::vector<int32_t> begin, end;     // positions of the ticks made so far
    size_t levels = 0;                   // made so far

    LaneTicks(int32_t n, const ColumnDir &col_, const Csr &csr_, const int32_t *lp, const int32_t *lv, bool fwd, int width)
        : col(col_), csr(csr_), level_ptr(lp), level_vtx(lv), forward(fwd), row_bytes(lane_unit_bytes(width) / kLaneUnit),
          shift(width == 4 ? 2 : 1), order(new int32_t[(size_t)n]), pos(new int32_t[(size_t)n]),
          tick_of(new int32_t[(size_t)n]) {}

    int32_t degree(int32_t v) const { return csr.ptr[v + 1] - csr.ptr[v]; }
    int32_t pieces(int32_t v) const { return std::max(1, (degree(v) + (1 << shift) - 1) >> shift); }

    void next_level() {
        const size_t l = forward ? levels : col.lvl_begin.size() - 1 - levels;
        const int32_t first = col.lvl_begin[levels], count = col.lvl_count[levels];
        int32_t *const to = order.get() + first;
        std::copy(level_vtx + level_ptr[l], level_vtx + level_ptr[l + 1], to);
        if (!std::is_sorted(to, to + count)) std::sort(to, to + count);
        int64_t bytes = 0;
        for (int32_t i = first; i < first + count; ++i) {
            const int32_t v = order[i];
            const int64_t add = 8 + (int64_t)pieces(v) * row_bytes;
            if (i == first || i - begin.back() == kLaneTickVerts || bytes + add > kLaneTickBytes) {
                begin.push_back(i);
                end.push_back(i);
                bytes = 0;
            }
            bytes += add;
            end.back() = i + 1;
            pos[v] = i;
            tick_of[v] = (int32_t)begin.size() - 1;
        }
        ++levels;
    }
    // Makes ticks up to number s; false if there are fewer.
    bool have(size_t s) {
        while (begin.size() <= s && levels < col.lvl_begin.size()) next_level();
        return s < begin.size();
    }
};

// Lane-window packing for one direction (layout: see LaneDir).  Returns false if the ring of a
// workgroup of 8 partitions would be too long.
bool pack_lane_dir(BlobWriter &w, int32_t n, const int64_t *c, size_t word_bytes, int width, const Csr &csr,
                   const int32_t *level_ptr, const int32_t *level_vtx, bool forward, const ColumnDir &col, LaneDir &dir) {
    LaneTicks ticks(n, col, csr, level_ptr, level_vtx, forward, width);
    const size_t row_bytes = (8 + 1) * word_bytes;
    const uint32_t unit_bytes = lane_unit_bytes(width);
    // Ring: while tick s runs, the values its edges read and those of tick s - 1 (on their way to the
    // output) are live, and the device ids of the two ticks after s are written already.  far_ticks = 0:
    // every neighbour in the ring.  Returns false if that is too long, or a tick has too many far reads.
    int64_t need = 0;
    std::vector<int32_t> far_of_tick;
    auto ring_fits = [&](int32_t far_ticks) {
        need = 1;
        dir.far_cap = 0;
        for (int32_t s = 0; ticks.have((size_t)s); ++s) {
            ticks.have((size_t)s + 2);
            int32_t oldest = ticks.begin[std::max(s - 1, 0)];
            far_of_tick.clear();
            for (int32_t i = ticks.begin[s]; i < ticks.end[s]; ++i) {
                const int32_t v = ticks.order[i];
                for (int32_t e = csr.ptr[v]; e < csr.ptr[v + 1]; ++e) {
                    const int32_t u = csr.idx[e];
                    if (far_ticks == 0 || s - ticks.tick_of[u] < far_ticks) oldest = std::min(oldest, ticks.pos[u]);
                    else far_of_tick.push_back(u);
                }
            }
            if (far_of_tick.size() > 16) {               // (up to 16 the cap is the same whatever repeats)
                std::sort(far_of_tick.begin(), far_of_tick.end());
                far_of_tick.erase(std::unique(far_of_tick.begin(), far_of_tick.end()), far_of_tick.end());
            }
            need = std::max<int64_t>(need, (int64_t)ticks.end[std::min<size_t>((size_t)s + 2, ticks.end.size() - 1)] - oldest);
            dir.far_cap = std::max(dir.far_cap, ((int32_t)far_of_tick.size() + 15) / 16 * 16);
            if ((uint64_t)(need + 2 * dir.far_cap) * row_bytes > kLaneRingBytes || dir.far_cap > kLaneMaxFar) return false;
        }
        return true;
    };
    int32_t far_ticks = 0;
    if (!ring_fits(0)) {
        far_ticks = kLaneFarTicks;
        while (!ring_fits(far_ticks)) {
            // a longer ring helps against too many far reads only
            if (dir.far_cap <= kLaneMaxFar || ticks.begin.size() <= (size_t)far_ticks) return false;
            far_ticks *= 2;
        }
        if (far_ticks >= (int32_t)ticks.begin.size()) return false;
    }
    const int32_t T = (int32_t)ticks.begin.size();
    const int32_t *const order = ticks.order.get(), *const tick_of = ticks.tick_of.get();
    dir.ticks = T;
    dir.slots = (int32_t)need;
    dir.width = width;
    std::unique_ptr<int32_t[]> slot(new int32_t[(size_t)n]);
    for (int32_t i = 0, at = 0; i < n; ++i) {
        slot[order[i]] = at;
        if (++at == dir.slots) at = 0;
    }

    // vertices that far reads ask for, numbered in the order they are computed
    std::vector<int32_t> far_no, far_list, far_seen;
    if (far_ticks) {
        far_no.assign((size_t)n, -1);
        for (int32_t i = 0; i < n; ++i)
            for (int32_t e = csr.ptr[order[i]]; e < csr.ptr[order[i] + 1]; ++e)
                if (tick_of[order[i]] - tick_of[csr.idx[e]] >= far_ticks) far_no[csr.idx[e]] = 0;
        for (int32_t i = 0; i < n; ++i)
            if (far_no[order[i]] == 0) far_no[order[i]] = dir.far_count++;
        far_list.assign((size_t)T * dir.far_cap, 0);
        far_seen.assign((size_t)n, -1);                  // last tick with a far read of the vertex
    }
    std::vector<int32_t> far_row(far_ticks ? (size_t)n : 0);     // row of the vertex among the current tick's far reads
    // what each tick takes of the stream, then the packets in place
    std::vector<uint32_t> tab((size_t)std::max(T, 1), 0);
    size_t total = 0;
    for (int32_t s = 0; s < T; ++s) {
        int64_t rows = 0;
        uint32_t far_out = 0;
        for (int32_t i = ticks.begin[s]; i < ticks.end[s]; ++i) {
            rows += ticks.pieces(order[i]);
            far_out += far_ticks && far_no[order[i]] >= 0;
        }
        const int64_t units = (rows + 2 * kLaneUnit - 1) / (2 * kLaneUnit) * 2;
        if (units >= (1 << 14)) return false;
        const uint32_t verts = (uint32_t)(ticks.end[s] - ticks.begin[s]);
        const uint32_t chunks = ((uint32_t)units * unit_bytes + 8u * verts + 4 * far_out + 15) / 16;
        tab[s] = (uint32_t)units | verts << 14 | far_out << 23;
        total += chunks;
        if (total >= (1ull << 31)) return false;
        dir.units += units;
        dir.max_chunks = std::max(dir.max_chunks, (int32_t)chunks);
        dir.max_verts = std::max(dir.max_verts, (int32_t)verts);
    }
    dir.stream_off = w.reserve(16 * std::max<size_t>(total, 1));
    uint32_t *packet = w.at<uint32_t>(dir.stream_off);
    const uint32_t pad_from = (uint32_t)dir.slots;
    for (int32_t s = 0; s < T; ++s) {
        const int32_t a = ticks.begin[s], b = ticks.end[s];
        const uint32_t units = tab[s] & 0x3fffu, far_out = tab[s] >> 23;
        uint32_t far_in = 0;
        auto source = [&](int32_t u) {
            if (!far_ticks || s - tick_of[u] < far_ticks) return (uint32_t)slot[u];
            if (far_seen[u] != s) {
                far_seen[u] = s;
                far_row[u] = (int32_t)far_in;
                far_list[(size_t)s * dir.far_cap + far_in++] = far_no[u];
            }
            return (uint32_t)(dir.slots + 2 + (s & 1) * dir.far_cap + far_row[u]);
        };
        uint32_t row = 0;
        auto put_row = [&](uint32_t to, uint32_t cv, int32_t e, int32_t len) {
            uint32_t *x = packet + (size_t)(row / kLaneUnit) * (unit_bytes / 4) + 2 * (row % kLaneUnit);
            x[0] = to;
            x[1] = cv;
            for (int j = 0; j < width; ++j) {
                x += 2 * kLaneUnit;
                x[0] = j < len ? source(csr.idx[e + j]) : pad_from;
                x[1] = j < len ? (uint32_t)csr.wt[e + j] : 0;
            }
            ++row;
        };
        for (int32_t i = a; i < b; ++i) {
            const int32_t v = order[i], d = ticks.degree(v);
            for (int32_t j = 0; j == 0 || j < d; j += width) put_row((uint32_t)slot[v], (uint32_t)c[v], csr.ptr[v] + j, d - j);
        }
        while (row < units * kLaneUnit) put_row(pad_from + 1, 0, 0, 0);
        uint32_t *verts = packet + (size_t)units * unit_bytes / 4;
        for (int32_t i = a; i < b; ++i) {
            verts[2 * (i - a)] = (uint32_t)order[i];
            verts[2 * (i - a) + 1] = (uint32_t)c[order[i]];
        }
        uint32_t *out = verts + 2 * (b - a);
        for (int32_t i = a; far_out && i < b; ++i)
            if (far_no[order[i]] >= 0) *out++ = (uint32_t)slot[order[i]];
        packet += ((size_t)units * unit_bytes + 8u * (uint32_t)(b - a) + 4 * far_out + 15) / 16 * 4;
    }
    dir.tick_off = w.reserve(4 * tab.size());
    std::memcpy(w.at<uint32_t>(dir.tick_off), tab.data(), 4 * tab.size());
    if (far_ticks) {
        dir.far_off = w.reserve(4 * far_list.size());
        std::memcpy(w.at<int32_t>(dir.far_off), far_list.data(), 4 * far_list.size());
    }
    dir.pos_off = w.reserve(4 * (size_t)n);
    std::memcpy(w.at<int32_t>(dir.pos_off), ticks.pos.get(), 4 * (size_t)n);
    return true;
}

// Rows of the chain sweep in one direction (see ChainDir), level by level in sweep order, and inside a level stage by stage:
// a vertex of more than kChainRow edges is put together from rows of the stages before its own.
struct ChainRows {
    struct Row {
        int32_t vertex;
        int32_t first, count;    // its edges in the CSR, or, `joins`, the rows that it is put together from
        int8_t lanes_log2;
        bool joins, part;        // part: a later row is put together from it
    };
    std::vector<Row> rows;
    std::vector<int32_t> begin, lanes;       // of the stages: first row (and the end of the last one), lanes that its rows take
    std::vector<int32_t> row_of;             // row of a vertex

    ChainRows(int32_t n, int32_t L, const Csr &csr, const int32_t *level_ptr, const int32_t *level_vtx, bool forward)
        : row_of((size_t)n) {
        rows.reserve((size_t)n);
        std::vector<Row> now, later;
        for (int32_t s = 0; s < L; ++s) {
            const int32_t l = forward ? s : L - 1 - s;
            now.clear();
            for (int32_t i = level_ptr[l]; i < level_ptr[l + 1]; ++i) {
                const int32_t v = level_vtx[i], d = csr.ptr[v + 1] - csr.ptr[v];
                int8_t lg = 0;
                while (4 << lg < std::min(d, kChainRow)) ++lg;
                now.push_back({v, csr.ptr[v], d, lg, false, false});
            }
            for (; !now.empty(); now.swap(later)) put_stage(now, later);
        }
        begin.push_back((int32_t)rows.size());
    }

  private:
    // Parts first, then rows of most lanes: the lanes of a row are an aligned group.
    void put_stage(const std::vector<Row> &now, std::vector<Row> &later) {
        constexpr int8_t kMost = 4;
        static_assert(4 << kMost == kChainRow, "a row's lanes hold four edges each");
        begin.push_back((int32_t)rows.size());
        int32_t taken = 0, of[kMost + 1] = {};
        later.clear();
        for (const Row &r : now) {
            if (r.count <= kChainRow) {
                ++of[r.lanes_log2];
                continue;
            }
            const int32_t parts = (r.count + kChainRow - 1) / kChainRow;
            int8_t lg = 0;
            while (4 << lg < std::min(parts, kChainRow)) ++lg;
            later.push_back({r.vertex, (int32_t)rows.size(), parts, lg, true, false});
            for (int32_t i = 0; i < parts; ++i)
                rows.push_back({r.vertex, r.first + i * kChainRow, std::min(kChainRow, r.count - i * kChainRow), kMost,
                                r.joins, true});
            taken += parts << kMost;
        }
        int32_t at[kMost + 1];
        int32_t next = (int32_t)rows.size();
        for (int lg = kMost; lg >= 0; --lg) {
            at[lg] = next;
            next += of[lg];
            taken += of[lg] << lg;
        }
        rows.resize((size_t)next);
        for (const Row &r : now) {
            if (r.count > kChainRow) continue;
            const int32_t to = at[r.lanes_log2]++;
            rows[to] = r;
            row_of[r.vertex] = to;
        }
        lanes.push_back(taken);
    }
};

// Lanes of a workgroup for these stages: a tick costs 0.1 us and 0.016 a wavefront, whether its lanes are filled or not.
int32_t chain_width(const ChainRows &b, const ChainRows &t) {
    int32_t best = 0;
    double best_us = 0;
    for (int32_t waves : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16}) {
        double us = 0;
        for (const ChainRows *r : {&b, &t}) {
            int64_t ticks = 0;
            for (int32_t u : r->lanes) ticks += (u + 64 * waves - 1) / (64 * waves);
            us = std::max(us, (double)ticks * (0.1 + 0.016 * waves));
        }
        if (best == 0 || us < best_us) {
            best_us = us;
            best = 64 * waves;
        }
    }
    return best;
}

// Packing of one direction for the chain sweep (layout: see ChainDir).  Returns false if its ring would be too long.
bool pack_chain_dir(BlobWriter &w, size_t word_bytes, const Csr &csr, const ChainRows &r, int32_t width, ChainDir &dir) {
    int64_t ticks = 0, all = 0;
    int32_t far = 0;
    for (int32_t u : r.lanes) {
        ticks += (u + width - 1) / width;
        all += u;
    }
    for (int32_t i = 0; i < (int32_t)r.rows.size(); ++i) {
        const ChainRows::Row &x = r.rows[i];
        if (x.joins && x.count > 0) far = std::max(far, i - x.first);
        else
            for (int32_t e = x.first; e < x.first + x.count; ++e) far = std::max(far, i - r.row_of[csr.idx[e]]);
    }
    const int64_t slots = (int64_t)far + 2 * std::min<int64_t>(width, (int64_t)r.rows.size());
    if ((size_t)(slots + 1 + kWave) * word_bytes > kChainLdsBytes) return false;
    ticks = (ticks + 1 + kChainAhead - 1) / kChainAhead * kChainAhead + kChainAhead;
    if (ticks * width >= (int64_t)1 << 27 || ticks * width > 8 * all + (1 << 20)) return false;
    dir.ticks = (int32_t)ticks;
    dir.slots = (int32_t)slots;
    dir.unit_off = w.reserve((size_t)ticks * width * 16);
    dir.edge_off = w.reserve((size_t)ticks * width * 8);
    uint32_t *const units = w.at<uint32_t>(dir.unit_off), *const edges = w.at<uint32_t>(dir.edge_off);
    const uint32_t none = (uint32_t)slots;
    // ring slots of the rows, and of the vertices (one look at an edge's neighbour instead of two and a division)
    std::unique_ptr<uint16_t[]> slot_of(new uint16_t[r.rows.size()]), slot_at(new uint16_t[r.row_of.size()]);
    for (size_t i = 0, at = 0; i < r.rows.size(); ++i, at = at + 1 == (size_t)slots ? 0 : at + 1) {
        slot_of[i] = (uint16_t)at;
        if (!r.rows[i].part) slot_at[r.rows[i].vertex] = (uint16_t)at;
    }
    int64_t at = 0;                          // units so far
    uint32_t steps = 0;                      // of the wavefront at hand: its first row has the most lanes
    auto put = [&](uint32_t slot, uint32_t lg, uint32_t leads, uint32_t first, uint32_t vertex) {
        uint32_t *u = units + 4 * at, *x = edges + 2 * at;
        if (at % kWave == 0) steps = lg;
        u[0] = u[1] = none | none << 16;
        u[2] = (slot == none ? none + 1 + (uint32_t)(at % kWave) : slot) | lg << 16 | steps << 20;
        u[3] = leads;
        x[0] = first;
        x[1] = vertex;
        ++at;
        return (uint16_t *)u;
    };
    for (size_t s = 0; s < r.lanes.size(); ++s) {
        for (int32_t i = r.begin[s]; i < r.begin[s + 1]; ++i) {
            const ChainRows::Row &x = r.rows[i];
            const uint32_t flags = (uint32_t)x.vertex | (x.part ? 1u << 31 : 0);
            for (int32_t j = 0; j < 1 << x.lanes_log2; ++j) {
                const int32_t first = x.first + 4 * j;
                uint16_t *u = put(j == 0 ? (uint32_t)slot_of[i] : none, (uint32_t)x.lanes_log2,
                                  j == 0 && !x.part ? (uint32_t)x.vertex : kChainNobody,
                                  (uint32_t)first | (x.joins ? 1u << 31 : 0), flags);
                const int32_t cnt = std::min(4, x.count - 4 * j);
                for (int32_t e = 0; e < cnt; ++e) u[e] = x.joins ? slot_of[first + e] : slot_at[csr.idx[first + e]];
            }
        }
        while (at % width) put(none, 0, kChainNobody, 0, kChainNobody);
    }
    while (at < ticks * width) put(none, 0, kChainNobody, 0, kChainNobody);
    return true;
}

// Packing for the whole-graph sweep (layout: see WholeDir).
void pack_whole(BlobWriter &w, int32_t n, int32_t L, const int64_t *c, const Csr &succ, const Csr &pred,
                const int32_t *level_ptr, const int32_t *level_vtx, WholeDir &dir) {
    const Csr *csr[2] = {&succ, &pred};
    std::vector<int32_t> units[2];           // of the levels
    for (int i = 0; i < 2; ++i)
        for (int32_t l = 0; l < L; ++l) {
            int32_t count = 0;
            for (int32_t j = level_ptr[l]; j < level_ptr[l + 1]; ++j)
                count += std::max(1, (csr[i]->ptr[level_vtx[j] + 1] - csr[i]->ptr[level_vtx[j]] + 3) / 4);
            units[i].push_back(count);
        }
    // units of a tick: a tick costs 0.28 us, and 0.006 for every unit past 32, whether it is filled or not
    double best_us = 0;
    for (int32_t a_tick : {8, 16, 32, 48, 64}) {
        int64_t ticks = 0;
        for (int i = 0; i < 2; ++i) {
            int64_t sum = 0;
            for (int32_t u : units[i]) sum += (u + a_tick - 1) / a_tick;
            ticks = std::max(ticks, sum);
        }
        const double us = (double)ticks * (0.28 + 0.006 * std::max(0, a_tick - 32));
        if (dir.units_a_tick == 0 || us < best_us) {
            best_us = us;
            dir.units_a_tick = a_tick;
            dir.ticks = (int32_t)((ticks + kWholeAhead - 1) / kWholeAhead * kWholeAhead);
        }
    }
    const int64_t room = (int64_t)(dir.ticks + kWholeAhead) * dir.units_a_tick;
    for (int i = 0; i < 2; ++i) {
        const size_t off = w.reserve((size_t)room * 32);
        (i ? dir.units_t : dir.units_b) = off;
        uint32_t *to = w.at<uint32_t>(off), *const end = to + room * 8;
        const uint32_t none = (uint32_t)n | (uint32_t)n << 16;
        auto put = [&](uint32_t v, uint32_t cv) {
            uint32_t *u = to;
            u[0] = u[1] = none;
            u[2] = v;
            u[3] = cv;
            u[4] = u[5] = u[6] = u[7] = 0;
            to += 8;
            return u;
        };
        for (int32_t s = 0; s < L; ++s) {
            const int32_t l = i ? s : L - 1 - s;
            for (int32_t j = level_ptr[l]; j < level_ptr[l + 1]; ++j) {
                const int32_t v = level_vtx[j], e0 = csr[i]->ptr[v], e1 = csr[i]->ptr[v + 1];
                for (int32_t e = e0; e < e1 || e == e0; e += 4) {
                    uint32_t *u = put((uint32_t)v, (uint32_t)c[v]);
                    for (int32_t x = 0; x < std::min(4, e1 - e); ++x) {
                        ((uint16_t *)u)[x] = (uint16_t)csr[i]->idx[e + x];
                        u[4 + x] = (uint32_t)csr[i]->wt[e + x];
                    }
                }
            }
            for (int32_t pad = (dir.units_a_tick - units[i][l] % dir.units_a_tick) % dir.units_a_tick; pad > 0; --pad)
                put((uint32_t)n + 1, 0);
        }
        while (to < end) put((uint32_t)n + 1, 0);
    }
}

// Both directions for the chain sweep, offsets from the start of a piece of the blob of their own; `ok` false and nothing in
// it where either is refused.
struct ChainPacked {
    std::vector<uint8_t> blob;
    ChainDir b, t;
    int32_t width = 0;
    bool ok = false;
};
ChainPacked pack_chain(int32_t n, int32_t L, size_t word_bytes, const Csr &succ, const Csr &pred, const int32_t *level_ptr,
                       const int32_t *level_vtx) {
    ChainPacked p;
    BlobWriter w(p.blob);
    const ChainRows rows_b(n, L, succ, level_ptr, level_vtx, false), rows_t(n, L, pred, level_ptr, level_vtx, true);
    p.width = chain_width(rows_b, rows_t);
    p.ok = pack_chain_dir(w, word_bytes, succ, rows_b, p.width, p.b) && pack_chain_dir(w, word_bytes, pred, rows_t, p.width, p.t);
    if (!p.ok) p.blob.clear();
    return p;
}

}  // namespace

int pack_graph(int32_t n, int64_t m, int32_t L,
               const int32_t *succ_ptr, const int32_t *succ_idx, const int64_t *succ_t,
               const int32_t *pred_ptr, const int32_t *pred_idx, const int32_t *pred_eid,
               const int64_t *c, const int32_t *level_ptr, const int32_t *level_vtx,
               Packed &out) {
    if (n < 1 || m < 0 || L < 1 || m >= (int64_t)0x7fffffff) return CP_ERR_SIZE;
    if (!succ_ptr || !pred_ptr || !c || !level_ptr || !level_vtx) return CP_ERR_NULL;
    if (m > 0 && (!succ_idx || !succ_t || !pred_idx || !pred_eid)) return CP_ERR_NULL;

    int rc = check_csr(n, m, succ_ptr, succ_idx);
    if (rc) return rc;
    rc = check_csr(n, m, pred_ptr, pred_idx);
    if (rc) return rc;

    // both CSRs must describe the same multiset of edges
    std::vector<int32_t> edge_src((size_t)m);
    for (int32_t v = 0; v < n; ++v)
        for (int32_t e = succ_ptr[v]; e < succ_ptr[v + 1]; ++e) edge_src[e] = v;
    {
        std::vector<uint8_t> seen((size_t)m, 0);
        for (int32_t v = 0; v < n; ++v)
            for (int32_t j = pred_ptr[v]; j < pred_ptr[v + 1]; ++j) {
                int32_t e = pred_eid[j];
                if (e < 0 || e >= m || seen[e]) return CP_ERR_CSR;
                seen[e] = 1;
                if (succ_idx[e] != v || edge_src[e] != pred_idx[j]) return CP_ERR_CSR;
            }
    }

    // level index: a partition of V in which every edge climbs
    if (level_ptr[0] != 0 || level_ptr[L] != n) return CP_ERR_LEVELS;
    std::vector<int32_t> level((size_t)n, -1);
    for (int32_t l = 0; l < L; ++l) {
        if (level_ptr[l + 1] < level_ptr[l]) return CP_ERR_LEVELS;
        for (int32_t i = level_ptr[l]; i < level_ptr[l + 1]; ++i) {
            int32_t v = level_vtx[i];
            if (v < 0 || v >= n || level[v] >= 0) return CP_ERR_LEVELS;
            level[v] = l;
        }
    }
    double per_level = 0;
    out.reach = 0;
    bool along = true;
    for (int64_t e = 0; e < m; ++e) {
        along = along && succ_idx[e] > edge_src[e];
        out.reach = std::max(out.reach, succ_idx[e] - edge_src[e]);
        const int32_t climbs = level[succ_idx[e]] - level[edge_src[e]];
        if (climbs <= 0) return CP_ERR_LEVELS;
        per_level += 1.0 / climbs;
    }
    if (!along) out.reach = 0;
    int64_t apart = 0;
    for (int32_t i = 1; i < n; ++i) apart += std::abs((int64_t)level_vtx[i] - level_vtx[i - 1]) >= 64;
    out.scattered = (double)apart / n;
    out.hops = m > 0 ? (int32_t)(L * (per_level / (double)m)) : 0;

    int64_t max_c = 0, max_t = 0;
    for (int32_t v = 0; v < n; ++v) {
        if (c[v] < 0) return CP_ERR_NEGATIVE;
        max_c = std::max(max_c, c[v]);
    }
    for (int64_t e = 0; e < m; ++e) {
        if (succ_t[e] < 0) return CP_ERR_NEGATIVE;
        max_t = std::max(max_t, succ_t[e]);
    }

    // U0: longest path with w = c and x = t bounds every tick value for every s, B >= 1
    const uint64_t kLimit = 1ull << 62;
    uint64_t u0 = 0;
    {
        std::vector<uint64_t> b0((size_t)n, 0);
        for (int32_t l = L - 1; l >= 0; --l)
            for (int32_t i = level_ptr[l]; i < level_ptr[l + 1]; ++i) {
                int32_t v = level_vtx[i];
                uint64_t best = 0;
                for (int32_t e = succ_ptr[v]; e < succ_ptr[v + 1]; ++e) {
                    uint64_t cand = (uint64_t)succ_t[e] + b0[succ_idx[e]];  // each term < 2^63
                    best = std::max(best, cand);
                }
                if (best >= kLimit || (uint64_t)c[v] >= kLimit) return CP_ERR_OVERFLOW;
                uint64_t val = best + (uint64_t)c[v];
                if (val >= kLimit) return CP_ERR_OVERFLOW;
                b0[v] = val;
                u0 = std::max(u0, val);
            }
    }

    Packed &P = out;
    P.n = n; P.m = m; P.L = L;
    P.narrow = (uint64_t)max_c < (1ull << 32) && (uint64_t)max_t < (1ull << 32);

    cp_graph_info &info = P.info;
    info = cp_graph_info{};
    info.n = n; info.L = L; info.m = m;
    info.max_c = max_c; info.max_t = max_t;
    info.raw_path_bound = (int64_t)u0;
    info.min_tick_bytes = u0 < (1ull << 31) ? 4 : 8;
    std::vector<int32_t> sources;
    for (int32_t v = 0; v < n; ++v) {
        int32_t od = succ_ptr[v + 1] - succ_ptr[v], id = pred_ptr[v + 1] - pred_ptr[v];
        info.max_out_degree = std::max(info.max_out_degree, od);
        info.max_in_degree = std::max(info.max_in_degree, id);
        if (od == 0) info.num_sinks++;
        if (id == 0) sources.push_back(v);
    }
    info.num_sources = (int32_t)sources.size();
    for (int32_t l = 0; l < L; ++l)
        info.max_level_width = std::max(info.max_level_width, level_ptr[l + 1] - level_ptr[l]);
    P.max_width = info.max_level_width;

    Csr succ{succ_ptr, succ_idx, {}}, pred{pred_ptr, pred_idx, {}};
    succ.wt.assign(succ_t, succ_t + m);
    pred.wt.resize((size_t)m);
    for (int64_t j = 0; j < m; ++j) pred.wt[j] = succ_t[pred_eid[j]];

    std::vector<int32_t> order_b, order_t;
    sweep_order(n, L, level_ptr, level_vtx, succ_ptr, /*forward=*/false, order_b, P.col_b);
    sweep_order(n, L, level_ptr, level_vtx, pred_ptr, /*forward=*/true, order_t, P.col_t);

    try {
        P.blob.clear();
        P.blob.reserve(blob_room(n, m, L, P.narrow));
        BlobWriter w(P.blob);
        // beside the rest, on a thread of its own where there is one to have (211,000 vertices: 170 -> 120 ms in all)
        std::future<ChainPacked> chain;
        if (L >= kChainLevels && n < (1 << 24) - 1 && (uint64_t)max_c + (uint64_t)max_t < (1ull << 32)) {
            auto pack = [&] { return pack_chain(n, L, (size_t)info.min_tick_bytes, succ, pred, level_ptr, level_vtx); };
            try {
                chain = std::async(std::launch::async, pack);
            } catch (const std::system_error &) {             // no thread to have: when it is asked for
                chain = std::async(std::launch::deferred, pack);
            }
        }
        pack_column_dir(w, n, m, P.narrow, succ, order_b, P.col_b);
        pack_column_dir(w, n, m, P.narrow, pred, order_t, P.col_t);
        if (P.narrow) {
            P.c_off = w.reserve(sizeof(uint32_t) * (size_t)n);
            uint32_t *cp = w.at<uint32_t>(P.c_off);
            for (int32_t v = 0; v < n; ++v) cp[v] = (uint32_t)c[v];
        } else {
            P.c_off = w.reserve(sizeof(int64_t) * (size_t)n);
            std::memcpy(w.at<int64_t>(P.c_off), c, sizeof(int64_t) * (size_t)n);
        }
        P.sources_off = w.reserve(sizeof(int32_t) * sources.size());
        std::memcpy(w.at<int32_t>(P.sources_off), sources.data(), sizeof(int32_t) * sources.size());

        P.have_window = false;
        if (P.narrow) {
            size_t mark = P.blob.size();
            bool ok = pack_window_dir(w, n, L, c, max_t, info.min_tick_bytes == 4, succ, order_b, P.col_b, P.win_b) &&
                      pack_window_dir(w, n, L, c, max_t, info.min_tick_bytes == 4, pred, order_t, P.col_t, P.win_t);
            if (ok) P.have_window = true;
            else P.blob.resize(mark);
        }
        P.have_lanes = false;
        P.lane_word = u0 < (1ull << (32 - kLaneIdBits)) ? 4 : 8;
        if (P.narrow && u0 < (1ull << (64 - kLaneIdBits))) {
            const size_t mark = P.blob.size();
            // entries per sub-row: an item costs about 28 instructions and 8 per entry
            int64_t rows2 = 0, rows4 = 0;
            for (const int32_t *ptr : {succ_ptr, pred_ptr})
                for (int32_t v = 0; v < n; ++v) {
                    rows2 += std::max(1, (ptr[v + 1] - ptr[v] + 1) / 2);
                    rows4 += std::max(1, (ptr[v + 1] - ptr[v] + 3) / 4);
                }
            const int width = rows2 * (28 + 8 * 2) < rows4 * (28 + 8 * 4) ? 2 : 4;
            P.have_lanes = pack_lane_dir(w, n, c, (size_t)P.lane_word, width, succ, level_ptr, level_vtx, false, P.col_b, P.lane_b) &&
                           pack_lane_dir(w, n, c, (size_t)P.lane_word, width, pred, level_ptr, level_vtx, true, P.col_t, P.lane_t);
            if (!P.have_lanes) P.blob.resize(mark);
        }
        P.have_whole = P.narrow && n <= kWholeVertices && u0 < (1ull << (64 - kLaneIdBits));
        P.whole = WholeDir{};
        if (P.have_whole) pack_whole(w, n, L, c, succ, pred, level_ptr, level_vtx, P.whole);
        P.have_chain = false;
        if (chain.valid()) {
            const ChainPacked packed = chain.get();
            P.have_chain = packed.ok;
            P.chain_width = packed.width;
            P.chain_b = packed.b;
            P.chain_t = packed.t;
            P.blob.resize(align_up(P.blob.size()));
            for (ChainDir *dir : {&P.chain_b, &P.chain_t}) {
                dir->unit_off += P.blob.size();
                dir->edge_off += P.blob.size();
            }
            P.blob.insert(P.blob.end(), packed.blob.begin(), packed.blob.end());
        }
        P.blob.resize(align_up(P.blob.size()));
    } catch (const std::bad_alloc &) {
        return CP_ERR_ALLOC;
    }

    info.window_slots_b = P.have_window ? P.win_b.slots : 0;
    info.window_slots_t = P.have_window ? P.win_t.slots : 0;
    info.window_packet_bytes_b = P.have_window ? 16 * P.win_b.max_chunks : 0;
    info.window_packet_bytes_t = P.have_window ? 16 * P.win_t.max_chunks : 0;
    info.window_ticks_b = P.have_window ? P.win_b.ticks : 0;
    info.window_ticks_t = P.have_window ? P.win_t.ticks : 0;
    info.window_slices_b = P.have_window ? P.win_b.smax : 0;
    info.window_slices_t = P.have_window ? P.win_t.smax : 0;
    info.window_far_b = P.have_window ? P.win_b.far_cap : 0;
    info.window_far_t = P.have_window ? P.win_t.far_cap : 0;
    info.blob_bytes = P.blob.size();
    return CP_OK;
}

}  // namespace cpeval
