// Host-only driver of the launch rules and tables that the GPU entry points build on the host.
// argv[1] names the check; exit status 0 = it holds, 1 = it does not (with a line that says where).
#include <cfenv>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../paper_1711_01912_amd/csrc/launch.hpp"

using namespace cpeval;

// The launch that clears CP leaves no thread more than its share of the batch.
static int prepare() {
    for (int32_t words : {1, 6, 300, 448})
        for (int64_t cells : {0ll, 1ll, 256ll, 257ll, 65536ll, 500000ll, 2000000ll, 0x7fffffffll}) {
            const int64_t threads = 256 * (int64_t)prepare_blocks(words, (int32_t)cells);
            const int64_t each = (cells + threads - 1) / threads;
            if (threads < words || each > std::max<int64_t>(1, (cells + 256 * 2048 - 1) / (256 * 2048))) {
                std::printf("words %d cells %lld: %lld threads\n", words, (long long)cells, (long long)threads);
                return 1;
            }
        }
    return 0;
}

// Every row of every slice is taken once, in either order; by runs, the XCDs (block number modulo 8) get even shares of
// the rows, which are alike where that order is taken for any number of slices.
static int column_rows(int32_t rows, int32_t slices, int per_block, bool by_runs) {
    const ColumnDeal d = column_deal(rows, slices, per_block, by_runs);
    const int64_t blocks = column_blocks(d, rows, slices, per_block);
    std::vector<int> taken((size_t)rows * slices, 0);
    int64_t share[8] = {};
    for (int32_t b = 0; b < blocks; ++b)
        for (int wave = 0; wave < per_block; ++wave) {
            int32_t r, slice;
            column_place(b, wave, d, slices, per_block, r, slice);
            if (r < 0 || slice < 0) return std::printf("below 0\n"), 1;
            if (r >= rows || slice >= slices) continue;
            ++taken[(size_t)r * slices + slice];
            ++share[b % 8];
        }
    for (int x : taken)
        if (x != 1) return std::printf("slices %d rows %d: a row %d times\n", slices, rows, x), 1;
    if (!by_runs) return 0;
    const int64_t units = ((int64_t)slices * d.parts + 7) / 8, row_blocks = (rows + per_block - 1) / per_block;
    const int64_t most = *std::max_element(share, share + 8);
    if (most > units * d.part_blocks * per_block)
        return std::printf("slices %d rows %d: an XCD has %lld rows\n", slices, rows, (long long)most), 1;
    // no more than the blocks of the rows, rounded up per part and per round of the XCDs
    if (blocks > slices * row_blocks + (int64_t)slices * d.parts + 8 * d.part_blocks)
        return std::printf("slices %d rows %d: %lld blocks\n", slices, rows, (long long)blocks), 1;
    return 0;
}

static int column() {
    for (int per_block : {1, 4})
        for (int32_t slices : {1, 2, 3, 4, 7, 8, 10, 17, 24})
            for (int32_t rows : {1, 3, 4, 5, 31, 32, 33, 1000, 4001})
                for (bool by_runs : {false, true})
                    if (column_rows(rows, slices, per_block, by_runs)) return 1;
    // rows of very different lengths stay in order where runs would give one XCD the long ones of many slices
    if (!column_by_runs(kHubDegree, 17) || column_by_runs(255, 17) || column_by_runs(255, 5) || !column_by_runs(255, 1) ||
        !column_by_runs(64, 8) || column_by_runs(63, 1))
        return std::printf("the rule\n"), 1;
    return 0;
}

// Where calls with 64-bit ring words end: at divisors, and volumes and divisors together, of 32 bits.
static int wide_words() {
    const int32_t k = 3;
    const int64_t top = (int64_t)1 << 32;
    for (int64_t amax : {(int64_t)0, (int64_t)1, (int64_t)1000, top / 2, top - 1000}) {
        const int64_t most = std::min(top - 1, top - amax);              // the largest divisor that fits
        const int64_t speeds[3] = {1, std::min<int64_t>(3, most), std::max<int64_t>(1, most / 2)};
        const int64_t bw[9] = {7, 1, most, std::max<int64_t>(1, most - 1), 7, std::min<int64_t>(2, most),
                               std::max<int64_t>(1, most / 3), std::min<int64_t>(10, most), 7};
        if (!wide_words_fit(k, speeds, bw, amax, amax)) return std::printf("refused at %lld\n", (long long)amax), 1;
        for (int at : {1, 5, 7}) {
            int64_t over[9];
            std::copy(bw, bw + 9, over);
            over[at] = most + 1;
            if (wide_words_fit(k, speeds, over, amax, amax)) return std::printf("a divisor too large fits\n"), 1;
        }
        const int64_t fast[3] = {1, most + 1, 1};
        if (wide_words_fit(k, fast, bw, amax, amax)) return std::printf("a speed too large fits\n"), 1;
    }
    return 0;
}

// Quotients by the tables of inverses, as the kernels take them: one multiply-add rounded up to whole numbers (or to units of
// 2^-6, for floats, which 2^17 makes the last bit of).
static uint32_t by_double(uint32_t a, double inverse) {
    volatile double x = (double)a, y = inverse, base = 4503599627370496.0;
    volatile double sum = std::fma(x, y, base);
    const double got = sum;
    uint64_t bits;
    std::memcpy(&bits, &got, 8);
    return (uint32_t)bits;
}
static uint32_t by_float(uint32_t a, float inverse) {
    volatile float x = (float)a, y = inverse, base = kFloatUnit * 8388608.0f;
    volatile float sum = std::fmaf(x, y, base);
    const float got = sum;
    uint32_t bits;
    std::memcpy(&bits, &got, 4);
    return bits & 0x7fffffu;
}

static int inverses() {
    std::vector<int64_t> divisors;
    for (int64_t d = 1; d <= 1200; ++d) divisors.push_back(d);
    for (int bit = 10; bit < 63; ++bit)
        for (int64_t off : {-1, 0, 1}) divisors.push_back(((int64_t)1 << bit) + off);
    for (int64_t d : std::vector<int64_t>{3000017, 8388593, 8388607, 12345678, 2147483647, 4294967295, INT64_MAX}) divisors.push_back(d);
    std::vector<int64_t> dividends;
    const int32_t k = 2;
    std::vector<double> wide(table_entries(k));
    std::vector<float> narrow(table_entries(k));
    for (size_t at = 0; at < divisors.size(); ++at) {
        const int64_t d = divisors[at], e = divisors[(at * 7 + 3) % divisors.size()];
        const int64_t speeds[2] = {d, e}, bw[4] = {5, d, e, 5};
        build_inverse_table(k, speeds, bw, wide.data());
        build_float_table(k, speeds, bw, narrow.data());
        // b sweep (own, neighbour), t sweep transposed, vertices
        const int64_t of[10] = {0, d, e, 0, 0, e, d, 0, d, e};
        dividends = {0, 1, 2, kFloatMost - 1, kFloatMost - 2, 4294967295ll, 4294967294ll, 2147483648ll, 65535, 65536};
        for (int64_t x : {d, e})
            for (int64_t times : std::vector<int64_t>{1, 2, 3, 1000, kFloatMost / x, 4294967295 / x})
                for (int64_t off : {-1, 0, 1})
                    if (times <= 4294967296ll / x) dividends.push_back(x * times + off);
        std::fesetround(FE_UPWARD);
        int64_t wrong = -1;
        size_t entry = 0;
        for (size_t i = 0; i < 10 && wrong < 0; ++i)
            for (int64_t a : dividends) {
                if (a < 0 || a >= (int64_t)1 << 32) continue;
                const uint32_t want = of[i] ? (uint32_t)(a / of[i] + (a % of[i] != 0)) : 0;
                if (by_double((uint32_t)a, wide[i]) != want || (a < kFloatMost && by_float((uint32_t)a, narrow[i]) != want)) {
                    wrong = a;
                    entry = i;
                    break;
                }
            }
        std::fesetround(FE_TONEAREST);
        if (wrong >= 0) return std::printf("%lld / %lld, entry %zu\n", (long long)wrong, (long long)of[entry], entry), 1;
    }
    return 0;
}

// Buckets that are left to be ranked: each is looked at once, by as many workgroups as there are buckets or by thousands,
// and a run of digits that all partitions use falls to the XCDs in even shares.
static int left_over() {
    for (int32_t partitions : {1, 2, 3, 7, 31, 32, 33, 64, 100, 129, 257, 512}) {
        const int32_t buckets = 512 * partitions, each = left_over_each(buckets);
        if (each < 1 || each > 16 || 512 % each || (each > 1 && buckets / each < 8192))
            return std::printf("%d buckets, %d each\n", buckets, each), 1;
        std::vector<int> taken((size_t)buckets, 0);
        int64_t share[8] = {};
        for (int32_t b = 0; b < buckets / each; ++b)
            for (int32_t t = 0; t < each; ++t) {
                const uint32_t d = left_over_bucket<512>((uint32_t)b, (uint32_t)t, each);
                if (d >= 512) return std::printf("digit %u\n", d), 1;
                ++taken[(size_t)(b / (512 / each)) * 512 + d];
                share[b % 8] += d % 32 < 19;
            }
        for (int x : taken)
            if (x != 1) return std::printf("%d buckets: one %d times\n", buckets, x), 1;
        if (partitions >= 8 && *std::max_element(share, share + 8) > 1.1 * (buckets * 19 / 32 / 8))
            return std::printf("%d buckets: an XCD has too many\n", buckets), 1;
        const int32_t dealt = bins_each(buckets);
        if (dealt < 1 || dealt > 4 || 512 % dealt || (dealt > 1 && buckets / dealt < 8192) ||
            (dealt < 4 && buckets / dealt > 16384))
            return std::printf("%d buckets, %d dealt\n", buckets, dealt), 1;
    }
    return 0;
}

// The workgroups that take the buckets of a partition's keys hold 1.4 times the average of those in use, up to 4,096 items.
static int bucket_sizes() {
    for (int32_t n : {65536, 70000, 211000, 250000, 262143, 480000, 1048576})
        for (int32_t k : {1, 2, 3, 5, 9, 16, 17, 33, 50, 64, 100, 255})
            for (int64_t max_b : {131072ll, 262143ll, 1000000ll, 1048576ll, 2100000ll, 4194303ll, 5000000ll, 16777215ll}) {
                const int bb = 64 - __builtin_clzll((uint64_t)max_b), kb = k > 1 ? 32 - __builtin_clz((unsigned)k - 1) : 0;
                const int rem = bb + kb - 9;
                if (bb + kb > 32 || bb + kb <= 17) continue;
                std::vector<char> in(512, 0);
                for (int64_t dev = 0; dev < k; ++dev)
                    for (int64_t x = 0; x <= max_b; x = x < max_b && x + (1ll << rem) > max_b ? max_b : x + (1ll << rem))
                        in[(size_t)((dev << bb | x) >> rem)] = 1;
                const int64_t used = std::count(in.begin(), in.end(), 1), threads = bucket_threads(n, k, bb, rem, max_b);
                if (8 * threads < std::min<int64_t>(4096, n / used * 7 / 5) || (threads > 128 && 4 * threads >= n / used * 7 / 5 + 7) || (threads != 128 && threads != 256 && threads != 512))
                    return std::printf("n %d k %d max_b %lld: %lld digits, %lld threads\n", n, k, (long long)max_b,
                                       (long long)used, (long long)threads), 1;
            }
    return 0;
}

// A graph's blob is allocated once.  argv[2]: the directory with the caller-side arrays.
template <typename T>
static std::vector<T> read_all(const std::string &name) {
    std::vector<T> v;
    FILE *f = std::fopen(name.c_str(), "rb");
    if (!f) return v;
    std::fseek(f, 0, SEEK_END);
    v.resize((size_t)std::ftell(f) / sizeof(T));
    std::fseek(f, 0, SEEK_SET);
    if (!v.empty() && std::fread(v.data(), sizeof(T), v.size(), f) != v.size()) v.clear();
    std::fclose(f);
    return v;
}

static int room(const std::string &dir) {
    auto i32 = [&](const char *name) { return read_all<int32_t>(dir + "/" + name + ".bin"); };
    auto i64 = [&](const char *name) { return read_all<int64_t>(dir + "/" + name + ".bin"); };
    const auto hdr = i64("hdr");
    if (hdr.size() != 3) return 2;
    const auto sp = i32("succ_ptr"), si = i32("succ_idx"), pp = i32("pred_ptr"), pi = i32("pred_idx"), pe = i32("pred_eid"),
               lp = i32("level_ptr"), lv = i32("level_vtx");
    const auto st = i64("succ_t"), c = i64("c");
    Packed p;
    if (pack_graph((int32_t)hdr[0], hdr[1], (int32_t)hdr[2], sp.data(), si.data(), st.data(), pp.data(), pi.data(),
                   pe.data(), c.data(), lp.data(), lv.data(), p) != CP_OK)
        return 2;
    const size_t made = blob_room(p.n, p.m, p.L, p.narrow);
    std::printf("blob %zu, room %zu, held %zu\n", p.blob.size(), made, p.blob.capacity());
    return p.blob.size() > made || p.blob.capacity() != made;
}

// A path by records or jumps only where it can be long: `wanted` says which of the two the packed graph of argv[2] gets.
static int paths(const std::string &dir, const std::string &wanted) {
    auto i32 = [&](const char *name) { return read_all<int32_t>(dir + "/" + name + ".bin"); };
    auto i64 = [&](const char *name) { return read_all<int64_t>(dir + "/" + name + ".bin"); };
    const auto hdr = i64("hdr");
    if (hdr.size() != 3) return 2;
    const auto sp = i32("succ_ptr"), si = i32("succ_idx"), pp = i32("pred_ptr"), pi = i32("pred_idx"), pe = i32("pred_eid"),
               lp = i32("level_ptr"), lv = i32("level_vtx");
    const auto st = i64("succ_t"), c = i64("c");
    Packed p;
    if (pack_graph((int32_t)hdr[0], hdr[1], (int32_t)hdr[2], sp.data(), si.data(), st.data(), pp.data(), pi.data(),
                   pe.data(), c.data(), lp.data(), lv.data(), p) != CP_OK)
        return 2;
    std::string got = path_by_records(p.n, p.m, p.L, p.hops) ? "records" : "csr";
    if (path_by_jumps(p.n, 1, p.L, p.hops)) got += "+jumps";
    if (path_by_jumps(p.n, 2, p.L, p.hops)) got += "+jumps of a batch";
    std::printf("%s, hops %d of %d\n", got.c_str(), p.hops, p.L);
    return got != wanted;
}

// Where b and the device ids are streamed past a walk.
static int streams() {
    auto tables = [](size_t k) { return (k * k + k) * 8; };
    const int32_t n = 121000, hops = 300, reach = 1000;
    auto ring = [&](int32_t P, size_t k) { return path_ring(n, 3 * n, P, hops, reach, tables(k)); };
    // 64 devices' tables and a ring take 53,760 bytes, 55,040 in granules: two workgroups a compute unit
    if (ring(512, 64) != 4096 || ring(513, 64) != 0) return std::printf("rounds of 64 devices\n"), 1;
    if (ring(777, 11) != 4096 || ring(63, 11) != 0 || ring(1025, 11) != 0) return std::printf("partitions\n"), 1;
    if (path_ring(n, 3 * n, 512, hops, 2049, tables(50)) != 8192 || path_ring(n, 3 * n, 513, hops, 2049, tables(50)) != 0)
        return std::printf("rounds of the larger ring\n"), 1;
    if (path_ring(n, 3 * n, 100, n / 700 - 1, reach, tables(8)) != 0 || path_ring(n, n / 2, 100, hops, reach, tables(8)) != 0)
        return std::printf("short paths\n"), 1;
    return 0;
}

// Where a few partitions take records at all.
static int few_records() {
    const int32_t n = 121000, hops = 300;
    if (!records_for(n, 3 * n, 1, hops) || records_for(n, 4 * n, 7, hops) || !records_for(n, 4 * n, 8, hops) ||
        records_for(n, 5 * n, 31, hops) || !records_for(n, 5 * n, 32, hops))
        return std::printf("records by edges\n"), 1;
    if (!records_for(7999, 5 * 7999 - 1, 4, hops) || records_for(7999, 5 * 7999, 4, hops) || records_for(8000, 4 * 8000, 4, hops) ||
        !records_for(11999, 6 * 11999 - 1, 31, hops) || records_for(12000, 5 * 12000, 31, hops))
        return std::printf("records of few vertices\n"), 1;
    if (records_for(n, 3 * n, 31, n / 700 - 1) || records_for(n, 3 * n, 7, n / 500 - 1) || !records_for(n, 3 * n, 32, 64) || records_for(n, n / 2, 5, hops))
        return std::printf("records by paths\n"), 1;
    return 0;
}

int main(int argc, char **argv) {
    if (argc < 2) return 2;
    if (argc > 2 && !std::strcmp(argv[1], "room")) return room(argv[2]);
    if (argc > 3 && !std::strcmp(argv[1], "paths")) return paths(argv[2], argv[3]);
    if (!std::strcmp(argv[1], "prepare")) return prepare();
    if (!std::strcmp(argv[1], "wide words")) return wide_words();
    if (!std::strcmp(argv[1], "inverses")) return inverses();
    if (!std::strcmp(argv[1], "column")) return column();
    if (!std::strcmp(argv[1], "few records")) return few_records();
    if (!std::strcmp(argv[1], "streams")) return streams();
    if (!std::strcmp(argv[1], "left-over")) return left_over();
    if (!std::strcmp(argv[1], "bucket-sizes")) return bucket_sizes();
    return 2;
}
