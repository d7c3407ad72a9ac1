// CPU check of the marks that xwin_layout writes into the column words: every
// pair's first entry has the bit and no other entry, the columns below it are
// those of the layout without marks, the slack is room that adding entries does
// not move, and a window that does not fit the word is refused.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "xwin_layout.h"

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

int main()
{
    std::mt19937_64 g(99);
    for (int rep = 0; rep < 60; ++rep) {
        const int64_t m = (int64_t)(g() % 500), n = 1 + (int64_t)(g() % 150000);
        std::vector<int32_t> rp{0}, ci;
        for (int64_t i = 0; i < m; ++i) {
            for (int64_t k = (int64_t)(g() % 40); k > 0; --k) ci.push_back((int32_t)(g() % (uint64_t)n));
            rp.push_back((int32_t)ci.size());
        }
        const int64_t nnz = (int64_t)ci.size();
        std::vector<double> val((size_t)nnz);
        for (auto &v : val) v = (double)(g() % 1000);
        for (int64_t wc : {1, 8192, 16384, 32767, 32768}) {
            if (wc == 1 && n > 30) continue;   // (thousands of windows)
            XwinHost a, b;
            CHECK(xwin_layout(m, n, nnz, rp.data(), ci.data(), val.data(), 8, wc, a) == kXwinOk, "rep %d", rep);
            CHECK(xwin_layout(m, n, nnz, rp.data(), ci.data(), val.data(), 8, wc, b, kXwinMark, 512) == kXwinOk,
                  "rep %d", rep);
            CHECK(a.ent == b.ent && a.val == b.val && a.pair_off == b.pair_off && a.rowpos == b.rowpos, "rep %d", rep);
            std::vector<char> first((size_t)nnz, 0);
            for (int64_t p = 0; p < a.npairs; ++p) first[a.ent[p]] = 1;
            for (int64_t k = 0; k < nnz; ++k) {
                CHECK((b.ci[k] & 0x7fff) == a.ci[k], "rep %d entry %lld", rep, (long long)k);
                CHECK(((b.ci[k] & kXwinMark) != 0) == (first[k] != 0), "rep %d entry %lld", rep, (long long)k);
            }
            CHECK((int64_t)b.ci.capacity() >= nnz + 512 && (int64_t)b.val.capacity() >= (nnz + 512) * 8, "rep %d", rep);
        }
        XwinHost d;
        CHECK(xwin_layout(m, n, nnz, rp.data(), ci.data(), val.data(), 8, 32769, d, kXwinMark) == kXwinTooWide, "mark");
        CHECK(xwin_layout(m, n, nnz, rp.data(), ci.data(), val.data(), 8, 65536, d) == kXwinOk, "65536");
        CHECK(xwin_layout(m, n, nnz, rp.data(), ci.data(), val.data(), 8, 65537, d) == kXwinTooWide, "word");
    }
    printf("ok\n");
    return 0;
}
