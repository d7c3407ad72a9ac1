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

int main()
{
    std::mt19937_64 g(4242);
    ranges(g);
    printf("ok\n");
    return 0;
}
