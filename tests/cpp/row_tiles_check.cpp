// CPU check of the row tiles' planning (row_tiles.h): tiles of random and of
// edge-case row lengths, and the ranges that a launch's workgroups allow.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "row_tiles.h"

using namespace spk;

#define CHECK(c, ...)                                            \
    do {                                                         \
        if (!(c)) {                                              \
            printf("FAIL %s:%d: %s: ", __FILE__, __LINE__, #c);  \
            printf(__VA_ARGS__);                                 \
            printf("\n");                                        \
            exit(1);                                             \
        }                                                        \
    } while (0)

// Ranges cover all tiles, none needs more workgroups than a launch has, and
// none could be longer.
static void check_ranges(int64_t ntiles, const std::vector<int32_t> &longs, int64_t unit, int64_t cap)
{
    const auto groups = [&](int64_t lo, int64_t end) {
        int64_t n = (end - lo + unit - 1) / unit;
        for (int32_t t : longs) n += t >= lo && t < end;
        return n;
    };
    int64_t lo = 0;
    while (lo < ntiles) {
        const int64_t end = row_tile_range(longs, lo, ntiles, unit, cap);
        CHECK(end > lo && end <= ntiles, "%lld: range [%lld, %lld)", (long long)ntiles, (long long)lo, (long long)end);
        CHECK(groups(lo, end) <= cap, "range [%lld, %lld) takes %lld workgroups", (long long)lo, (long long)end,
              (long long)groups(lo, end));
        CHECK(end == ntiles || groups(lo, end + 1) > cap, "range [%lld, %lld) is short", (long long)lo, (long long)end);
        lo = end;
    }
}

static void ranges(std::mt19937_64 &g)
{
    for (int rep = 0; rep < 300; ++rep) {
        const int64_t ntiles = 1 + (int64_t)(g() % 400);
        std::vector<int32_t> longs;
        const int density = (int)(g() % 5);   // none to all tiles long
        for (int64_t t = 0; t < ntiles; ++t)
            if ((int)(g() % 4) < density) longs.push_back((int32_t)t);
        for (int64_t unit : {1, 2, 4, 8})
            for (int64_t cap : {2, 3, 7, 64, 100000}) check_ranges(ntiles, longs, unit, cap);
    }
    // rows of 513 entries only, as many as 2^31 entries hold: 256 threads
    std::vector<int32_t> longs((size_t)((int64_t(1) << 31) / 513));
    for (size_t t = 0; t < longs.size(); ++t) longs[t] = (int32_t)t;
    const int64_t end = row_tile_range(longs, 0, (int64_t)longs.size(), 4, (int64_t(1) << 30) / 256);
    CHECK((end + (end + 3) / 4) * 256 <= (int64_t(1) << 30), "range of %lld long rows", (long long)end);
}

// Every row is in one tile of its kind: streams of at most E entries and 128
// rows, runs of rows over the stream's, and rows over the line alone.
static std::vector<int32_t> check_tiles(const std::vector<int64_t> &len, int E, int BS, bool f64, int64_t line)
{
    std::vector<int32_t> rp{0}, k, longs;
    for (int64_t l : len) rp.push_back((int32_t)(rp.back() + l));
    const int64_t m = (int64_t)len.size();
    const int64_t top = m > 0 ? *std::max_element(len.begin(), len.end()) : 0;
    std::vector<uint32_t> t;
    for (int64_t max_len : {top, (int64_t)INT32_MAX})
        CHECK(long_row_line(rp.data(), m, E, BS, f64, max_len) == line, "line %lld, not %lld",
              (long long)long_row_line(rp.data(), m, E, BS, f64, max_len), (long long)line);
    make_row_tiles(rp.data(), m, E, BS, f64, top, t, k, longs);
    const int64_t short_max = E < 512 ? E : 512;
    std::vector<int32_t> found;
    CHECK(t.size() == k.size() && (t.back() & kBlkRowMask) == (uint32_t)m && (t[0] & kBlkRowMask) == 0, "ends");
    for (size_t i = 0; i + 1 < t.size(); ++i) {
        const int64_t r0 = t[i] & kBlkRowMask, r1 = t[i + 1] & kBlkRowMask, n = rp[r1] - rp[r0];
        CHECK(r1 > r0 && k[i] == rp[r0], "tile %zu", i);
        const uint32_t mode = t[i] >> 30;
        if (mode == kBlkLong) {
            CHECK(r1 == r0 + 1 && n > line, "tile %zu of %lld entries", i, (long long)n);
            found.push_back((int32_t)i);
        } else if (mode == kBlkWave) {
            CHECK(n <= kMediumRun || r1 == r0 + 1, "tile %zu of %lld entries", i, (long long)n);
            for (int64_t r = r0; r < r1; ++r) CHECK(len[r] > short_max && len[r] <= line, "row %lld", (long long)r);
        } else {
            CHECK(mode == kBlkStream && n <= E && r1 - r0 <= 128, "tile %zu", i);
        }
    }
    CHECK(found == longs, "long rows");
    return longs;
}

static void tiles(std::mt19937_64 &g)
{
    const auto rows = [](int64_t n, int64_t l) { return std::vector<int64_t>((size_t)n, l); };
    // one length throughout: a wavefront each once they are many, in FP64
    for (int64_t l : {513, 600, 1024, 4096}) {
        CHECK(check_tiles(rows(2048, l), 512, 256, true, 4096).empty(), "%lld", (long long)l);
        CHECK(check_tiles(rows(2047, l), 512, 256, true, 512).size() == 2047, "%lld", (long long)l);
        CHECK(check_tiles(rows(2048, l), 512, 256, false, 512).size() == 2048, "%lld", (long long)l);
    }
    check_tiles(rows(5000, 512), 512, 256, true, 512);
    check_tiles(rows(5000, 1024), 512, 512, true, 1024);
    check_tiles(rows(5000, 1025), 512, 512, true, 4096);
    CHECK(check_tiles(rows(2048, 4097), 512, 256, true, 4096).size() == 2048, "over the upper line");
    // as many among more tiles of short rows, and just fewer
    auto mixed = rows(3000, 600);
    mixed.resize(3000 + 4000 * 32, 16);
    check_tiles(mixed, 512, 256, true, 512);
    mixed.resize(3000 + 1000 * 32);
    check_tiles(mixed, 512, 256, true, 4096);
    check_tiles({}, 512, 256, true, 512);
    check_tiles(rows(300, 0), 512, 256, true, 512);
    for (int rep = 0; rep < 200; ++rep) {
        std::vector<int64_t> len((size_t)(g() % 4000));
        const uint64_t top = 1 + g() % (rep % 3 == 0 ? 5000 : 200);
        for (auto &l : len) l = g() % 50 == 0 ? (int64_t)(g() % 6000) : (int64_t)(g() % top);
        std::vector<int32_t> rp{0};
        for (int64_t l : len) rp.push_back((int32_t)(rp.back() + l));
        for (int E : {256, 512, 1024})
            for (int BS : {64, 256, 512})
                for (bool f64 : {false, true})
                    check_tiles(len, E, BS, f64, long_row_line(rp.data(), (int64_t)len.size(), E, BS, f64, INT32_MAX));
    }
}

int main()
{
    std::mt19937_64 g(4242);
    ranges(g);
    tiles(g);
    printf("ok\n");
    return 0;
}
