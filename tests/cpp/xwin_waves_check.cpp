// CPU check of the x-window form's wavefront ranges (xwin_waves): the walk of
// the first pass replayed over the marked column words, tile by tile, as the
// kernel does it.  Every pair gets exactly one sum, the sum of its entries, and
// no tile reads past the slack.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "xwin_layout.h"

using namespace spk;

static int failures = 0;
#define CHECK(c, ...)                                            \
    do {                                                         \
        if (!(c)) {                                              \
            ++failures;                                          \
            printf("FAIL %s:%d: %s: ", __FILE__, __LINE__, #c);  \
            printf(__VA_ARGS__);                                 \
            printf("\n");                                        \
            return;                                              \
        }                                                        \
    } while (0)

constexpr int64_t kSlack = 512;

static void check_one(int64_t m, int64_t n, const std::vector<int32_t> &rp, const std::vector<int32_t> &ci, int64_t wc,
                      int E, int nw, int64_t target, const char *name)
{
    const int64_t nnz = (int64_t)ci.size();
    std::vector<double> val((size_t)nnz);
    for (int64_t k = 0; k < nnz; ++k) val[k] = 1.0 + (double)(k % 29);
    XwinHost d;
    CHECK(xwin_layout(m, n, nnz, rp.data(), ci.data(), val.data(), 8, wc, d) == kXwinOk, "%s", name);
    std::vector<uint32_t> tiles;
    std::vector<int32_t> tile_k, chunk_t, chunk_w, wp, wk, wcnt;
    xwin_plan(d, E, target, tiles, tile_k, chunk_t, chunk_w);
    xwin_waves(d, nw, tiles, chunk_t, wp, wk, wcnt);
    const size_t nr = chunk_w.size() * nw;
    CHECK(wp.size() == nr + 1 && wk.size() == nr + 1 && wcnt.size() == nr, "%s sizes", name);
    CHECK(wp[nr] == d.npairs && wk[nr] == nnz, "%s end", name);
    std::vector<uint16_t> word(d.ci.begin(), d.ci.end());
    for (int64_t p = 0; p < d.npairs; ++p) {
        CHECK(!(word[d.ent[p]] & kXwinMark), "%s column takes the mark's bit", name);
        word[d.ent[p]] |= kXwinMark;
    }
    word.resize((size_t)(nnz + kSlack), kXwinMark);
    std::vector<double> v((size_t)(nnz + kSlack), 0.0), part((size_t)d.npairs, NAN);
    if (nnz > 0) memcpy(v.data(), d.val.data(), (size_t)nnz * 8);
    for (size_t i = 0; i < nr; ++i) {
        const int64_t p0 = wp[i], p1 = wp[i + 1];
        CHECK(p0 <= p1 && wk[i] == d.ent[p0], "%s range %zu", name, i);
        const size_t c = i / nw;
        CHECK(p0 >= d.pair_off[chunk_w[c]] && p1 <= d.pair_off[chunk_w[c] + 1], "%s range %zu leaves its window", name, i);
        const int64_t k0 = wk[i] & ~3, k1 = wk[i + 1];
        const int64_t nt = p0 < p1 ? (k1 - k0 + E - 1) / E : 0;
        CHECK(k0 + std::max<int64_t>(nt, 1) * E <= nnz + kSlack, "%s range %zu reads past the slack", name, i);
        int64_t held = 0, from = p0, skip = p0 - wcnt[i] + 1;
        double carry = 0.0;
        std::vector<double> slice;
        for (int64_t t = 0; t < nt; ++t) {
            int64_t closed = 0;
            for (int64_t k = k0 + t * E; k < k0 + (t + 1) * E; ++k) {
                if (word[k] & kXwinMark) {
                    if (closed++ >= skip) slice.push_back(carry);
                    carry = 0.0;
                }
                carry += v[k];
            }
            CHECK(closed >= skip, "%s range %zu: the first tile does not reach its first pair", name, i);
            held = std::min<int64_t>(held + closed - skip, p1 - from);
            slice.resize((size_t)held);
            skip = 0;
            const int64_t end = (from + held) & ~(int64_t)63;
            if (end > from) {
                const int64_t cnt = end - from;
                CHECK(cnt <= E + 64, "%s slice", name);
                for (int64_t q = 0; q < cnt; ++q) {
                    CHECK(std::isnan(part[from + q]), "%s pair twice", name);
                    part[from + q] = slice[q];
                }
                slice.erase(slice.begin(), slice.begin() + cnt);
                held -= cnt;
                from = end;
            }
            CHECK(held < 64, "%s held %lld", name, (long long)held);
        }
        if (nt == 0) continue;
        if (from + held < p1) {
            slice.push_back(carry);
            ++held;
        }
        CHECK(from + held == p1, "%s range %zu leaves pairs out", name, i);
        for (int64_t q = 0; q < held; ++q) {
            CHECK(std::isnan(part[from + q]), "%s pair twice", name);
            part[from + q] = slice[q];
        }
    }
    for (int64_t p = 0; p < d.npairs; ++p) {
        double ref = 0.0;
        for (int32_t k = d.ent[p]; k < d.ent[p + 1]; ++k) ref += v[k];
        CHECK(part[p] == ref, "%s pair %lld: %g, not %g", name, (long long)p, part[p], ref);   // whole numbers: exact
    }
}

int main()
{
    std::mt19937_64 g(777);
    check_one(0, 5, {0}, {}, 16384, 256, 12, 256, "m0");
    check_one(3, 5, {0, 0, 0, 0}, {}, 16384, 256, 12, 256, "empty");
    check_one(1, 1, {0, 1}, {0}, 16384, 256, 12, 256, "1x1");
    for (int rep = 0; rep < 30; ++rep) {
        const int64_t m = 1 + (int64_t)(g() % 3000), n = 1 + (int64_t)(g() % 120000);
        const int64_t maxlen = rep % 3 == 0 ? 3 : 1 + (int64_t)(g() % 120);
        std::vector<int32_t> rp{0}, ci;
        for (int64_t i = 0; i < m; ++i) {
            int64_t len = (int64_t)(g() % (uint64_t)(maxlen + 1));
            if (rep % 5 == 4 && g() % 200 == 0) len = 3000 + (int64_t)(g() % 9000);
            for (int64_t k = 0; k < len; ++k) ci.push_back((int32_t)(g() % (uint64_t)n));
            rp.push_back((int32_t)ci.size());
        }
        for (int64_t wc : {8192, 16384, 32768})
            for (int nw : {4, 12, 16})
                for (int64_t target : {1, 256}) {
                    char name[96];
                    snprintf(name, sizeof name, "rep %d m %lld n %lld wc %lld nw %d target %lld", rep, (long long)m,
                             (long long)n, (long long)wc, nw, (long long)target);
                    check_one(m, n, rp, ci, wc, nw == 16 ? 128 : 256, nw, target, name);
                    if (failures) return 1;
                }
    }
    printf("ok\n");
    return failures != 0;
}
