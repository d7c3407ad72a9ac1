// row_tiles.h -- tiles over the rows of a CSR matrix (host planning of the
// row-block and CG kernels, and, over (row, window) pairs, of the x-window
// form; plain C++, no GPU headers).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

namespace spk {

// A tile is recorded as its start row | mode << 30 and its first entry.
constexpr uint32_t kBlkRowMask = 0x3FFFFFFFu;
constexpr uint32_t kBlkStream = 0u;     // short rows streamed through the wavefront's LDS slice
constexpr uint32_t kBlkWave = 1u;       // medium rows, one after another, 64 lanes per row
constexpr uint32_t kBlkLong = 2u;       // one long row, a workgroup

// Tiles of the x-window form's pairs, of which only the cuts are used (chunks
// end at them): runs of short rows (at most 96 entries each) whose entries fit
// E and that number at most 128; runs of medium rows, up to 4E entries in all;
// single long rows (over 8E entries).
inline void make_blocks(const int32_t *rp, int64_t m, int E, std::vector<uint32_t> &out, std::vector<int32_t> &out_k)
{
    const int64_t kShort = std::min<int64_t>(96, E);
    const int64_t kLong = 8 * (int64_t)E;
    const int64_t kRows = 2 * 64;
    out.clear();
    out_k.clear();
    int64_t r = 0;
    while (r < m) {
        const int64_t len = rp[r + 1] - rp[r];
        out_k.push_back(rp[r]);
        if (len > kLong) {
            out.push_back((uint32_t)r | (kBlkLong << 30));
            ++r;
        } else if (len > kShort) {
            out.push_back((uint32_t)r | (kBlkWave << 30));
            int64_t nz = 0;
            while (r < m) {
                const int64_t l = rp[r + 1] - rp[r];
                if (l <= kShort || l > kLong || (nz > 0 && nz + l > 4 * (int64_t)E)) break;
                nz += l;
                ++r;
            }
        } else {
            out.push_back((uint32_t)r | (kBlkStream << 30));
            int64_t nz = 0, c = 0;
            while (r < m && c < kRows) {
                const int64_t l = rp[r + 1] - rp[r];
                if (l > kShort || nz + l > E) break;
                nz += l;
                ++r;
                ++c;
            }
        }
    }
    out.push_back((uint32_t)m);
    out_k.push_back(rp[m]);
}

// Tiles of the single-matrix row-block and CG kernels, E = row-stream
// capacity, BS = threads per workgroup: runs of short rows (at most
// min(E, 512) entries each, at most 128 rows, at most E entries); runs of
// medium rows of up to kMediumRun entries (or one row), 64 lanes per row;
// rows over long_row_line entries stand alone, and are named in `longs` (tile
// indices): a whole workgroup runs each.  The aim is that no wavefront
// has much more to do than a full row-stream tile: gathers are bound by rate,
// so a wavefront with four times the entries outlives the others and ends
// alone, bound by latency.  300,001 rows of truncated-Zipf length (mean 16),
// FP32, 256 threads: 69 us with rows over 96 entries ending a tile and a
// wavefront for every longer row up to any length; 48 us with the line at
// 2,048, 39 us at 1,024, 37 us at 512.  With 512 threads (CG) a row of 513
// to 1,024 gives each lane two entries at most: 20,000-row solves take
// 162 us with the line at 512, 153 us at 1,024, 155 us at 2,048.
constexpr int64_t kStreamRowMax = 512;
constexpr int64_t kMediumRun = 1024;
inline int64_t long_row_min(int BS) { return BS > 256 ? 1024 : 512; }

// Where most wavefronts would run such rows, none outlives the others, and a
// workgroup per row mostly waits (a row of 600 is one pass of its loads): FP64
// rows over long_row_min get a wavefront each, up to kManyLongRowMax entries,
// when they are at least kManyLongRows (eight wavefronts per compute unit) and
// outnumber the other tiles.  One length throughout, FP64, a workgroup and a
// wavefront per row: 10,000 rows of 520 21.1 us and 14.7, 8,000 of 800 31.9 and
// 26.7, 5,000 of 1,100 23.2 and 17.9, 3,000 of 2,000 15.4 and 15.5, 1,500 of
// 700 5.7 and 6.0, 300 of 2,000 5.7 and 7.7; CG's 512 threads, five iterations:
// 8,000 of 1,100 274 and 172, 3,000 of 3,000 198 and 195.  In FP32 the
// workgroup is the faster one at all of these (10,000 of 520 16.4 and 19.7,
// 3,000 of 2,000 11.9 and 29.7).  (`max_len`: the longest row, or more; it
// spares matrices without long rows the count.)
constexpr int64_t kManyLongRows = 2048, kManyLongRowMax = 4096;
inline int64_t long_row_line(const int32_t *rp, int64_t m, int E, int BS, bool f64, int64_t max_len)
{
    const int64_t line = long_row_min(BS);
    if (!f64 || max_len <= line) return line;
    int64_t rows = 0, entries = 0;
    for (int64_t r = 0; r < m; ++r) {
        const int64_t l = rp[r + 1] - rp[r];
        if (l > line) {
            ++rows;
            entries += l;
        }
    }
    const int64_t others = (rp[m] - rp[0] - entries) / E + (m - rows) / (2 * 64);   // at least so many tiles
    return rows >= kManyLongRows && rows > others ? kManyLongRowMax : line;
}

inline void make_row_tiles(const int32_t *rp, int64_t m, int E, int BS, bool f64, int64_t max_len,
                           std::vector<uint32_t> &out, std::vector<int32_t> &out_k, std::vector<int32_t> &longs)
{
    const int64_t short_max = std::min<int64_t>(kStreamRowMax, E);
    const int64_t long_min = long_row_line(rp, m, E, BS, f64, max_len);
    const int64_t row_cap = 2 * 64;
    out.clear();
    out_k.clear();
    longs.clear();
    int64_t r = 0;
    while (r < m) {
        const int64_t len = rp[r + 1] - rp[r];
        out_k.push_back(rp[r]);
        if (len > long_min) {
            longs.push_back((int32_t)out.size());
            out.push_back((uint32_t)r | (kBlkLong << 30));
            ++r;
        } else if (len > short_max) {
            out.push_back((uint32_t)r | (kBlkWave << 30));
            int64_t nz = 0;
            while (r < m) {
                const int64_t l = rp[r + 1] - rp[r];
                if (l <= short_max || l > long_min || (nz > 0 && nz + l > kMediumRun)) break;
                nz += l;
                ++r;
            }
        } else {
            out.push_back((uint32_t)r | (kBlkStream << 30));
            int64_t nz = 0, c = 0;
            while (r < m && c < row_cap) {
                const int64_t l = rp[r + 1] - rp[r];
                if (l > short_max || nz + l > E) break;
                nz += l;
                ++r;
                ++c;
            }
        }
    }
    out.push_back((uint32_t)m);
    out_k.push_back(rp[m]);
}

// End of the longest range of tiles from `lo` on that one launch of at most
// `cap` (two or more) workgroups runs: a workgroup per `unit` tiles, and one
// for each long tile of the range (`longs`, ascending).
inline int64_t row_tile_range(const std::vector<int32_t> &longs, int64_t lo, int64_t hi, int64_t unit, int64_t cap)
{
    const auto l0 = std::lower_bound(longs.begin(), longs.end(), (int32_t)lo);
    const auto groups = [&](int64_t end) {
        return (end - lo + unit - 1) / unit + (std::lower_bound(l0, longs.end(), (int32_t)end) - l0);
    };
    if (groups(hi) <= cap) return hi;
    int64_t fits = lo + 1, over = hi;
    while (over - fits > 1) {
        const int64_t mid = fits + (over - fits) / 2;
        if (groups(mid) <= cap) fits = mid;
        else over = mid;
    }
    return fits;
}

}  // namespace spk
