// kernels_xwin.hip -- CSR SpMV with x staged in LDS by column window
// (SPK_FMT_XWIN).
//
// A random-column matrix gathers x from all over the vector; once x is
// larger than an XCD's L2, most gathers miss it and each miss moves a whole
// 128-byte line for 8 useful bytes.  Here the columns are cut into windows
// of at most 128 KiB of x (64 KiB for the smaller variants), small enough to
// live in a compute unit's LDS.  At conversion the entries are regrouped
// window by window: a (row, window) pair holds the row's entries whose
// columns fall in the window, in their original order, with 16-bit column
// words: 15 bits of column inside the window and the top bit on a pair's
// first entry.  The first pass runs one workgroup per chunk of one window's
// pairs: it copies that window of x into LDS once, then its wavefronts
// stream the chunk's values and column words with coalesced loads, take x
// from LDS, sum between the marks and write one FP64 partial per pair.  A
// second pass adds each row's partials in window order (and forms
// w = alpha*y + x when fused).  Every byte of the first pass is a coalesced
// stream; the gathers never leave the compute unit.
#include "device_common.h"
#include "device_rows.h"
#include "kernels.h"
#include "xwin_layout.h"

namespace spk {

namespace {

// A tile is 64*ITEMS consecutive entries of a wavefront's range, lane l
// holding ITEMS consecutive ones: its values in 16-byte loads, its column
// words in one load.
template <typename T, int ITEMS>
struct WinTile {
    T v[ITEMS];
    uint32_t c[ITEMS / 2];   // two column words each
};

template <typename T, int ITEMS>
__device__ __forceinline__ void window_load(const XwinArgs &a, int64_t k, WinTile<T, ITEMS> &tl)
{
    constexpr int VN = 16 / (int)sizeof(T) < ITEMS ? 16 / (int)sizeof(T) : ITEMS;   // values per load
    typedef T vv __attribute__((ext_vector_type(VN)));
    typedef uint32_t vc __attribute__((ext_vector_type(ITEMS / 2)));
    const vc c = __builtin_nontemporal_load((gptr<vc>)(as_global(a.ci) + k));
#pragma unroll
    for (int j = 0; j < ITEMS; j += VN) {
        const vv t = *(gptr<vv>)(as_global((const T *)a.val) + k + j);
#pragma unroll
        for (int u = 0; u < VN; ++u) tl.v[j + u] = t[u];
    }
    if constexpr (ITEMS == 2) {
        tl.c[0] = *(const uint32_t *)&c;
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS / 2; ++j) tl.c[j] = c[j];
    }
}

// Inclusive sums over lanes back to the nearest marked lane: lane l gets
// v(m) + ... + v(l), m the last lane <= l with a mark, dist = l - m (or
// anything over l if there is none, for the sum from lane 0).  Shifts inside
// rows of 16 lanes, then the rows' last lanes to the rows above.
constexpr int kDppRowShr = 0x110;       // + distance: lane l reads lane l - distance of its row
constexpr int kDppRowBcast15 = 0x142;   // the last lane of each row to the next row
constexpr int kDppRowBcast31 = 0x143;   // lane 31 to the rows above
constexpr int kDppWaveShr1 = 0x138;     // lane l reads lane l - 1

__device__ __forceinline__ double marked_scan(double v, int dist, int l)
{
    double t;
    t = dpp_f64<kDppRowShr + 1>(v);
    v += dist >= 1 ? t : 0.0;
    t = dpp_f64<kDppRowShr + 2>(v);
    v += dist >= 2 ? t : 0.0;
    t = dpp_f64<kDppRowShr + 4>(v);
    v += dist >= 4 ? t : 0.0;
    t = dpp_f64<kDppRowShr + 8>(v);
    v += dist >= 8 ? t : 0.0;
    t = dpp_f64<kDppRowBcast15>(v);
    v += (l & 16) && dist > (l & 15) ? t : 0.0;
    t = dpp_f64<kDppRowBcast31>(v);
    v += (l & 32) && dist > (l & 31) ? t : 0.0;
    return v;
}

// One wavefront's walk over its entries: the pair open where the next tile
// begins has the sum `carry` so far; the slice holds `held` closed sums, of the
// pairs from `from` on; the next tile first closes `skip` pairs that are not
// the wavefront's (only a range's first tile does).
struct WinWalk {
    double carry;
    int held, from, skip;
};

// Writes the held sums of the pairs before `end` and moves the rest to the
// slice's front.
template <int ITEMS>
__device__ __forceinline__ void window_flush(const XwinArgs &a, double *sp, int end, WinWalk &wk)
{
    const int l = threadIdx.x & (kWave - 1);
    const int count = end - wk.from;
    if (count <= 0) return;
    const gptr_mut<double> part = as_global_mut(a.part) + wk.from;
#pragma unroll
    for (int q = 0; q <= ITEMS; ++q)
        if (q * kWave < count && l + q * kWave < count) part[l + q * kWave] = sp[l + q * kWave];
    const double rest = sp[min(count + l, kWave * (ITEMS + 1) - 1)];
    wave_lds_sync();
    sp[l] = rest;
    wave_lds_sync();
    wk.held -= count;
    wk.from = end;
}

// Sums one tile between its marks.  A pair that ends in the tile is closed by
// the lane that holds the next mark: its own entries before the mark plus
// what the lanes below hold of the pair (one scan over the lanes), so pairs
// may be of any length and start anywhere.  The closed sums collect in the
// wavefront's LDS slice sp and leave in whole aligned groups of 64, so that
// every line of partials is written once; those of pairs past p1 (entries of
// the next range in the last tile) are dropped.
template <typename T, int ITEMS>
__device__ __forceinline__ void window_tile(const XwinArgs &a, const T *win, const WinTile<T, ITEMS> &tl, double *sp,
                                            int p1, WinWalk &wk)
{
    const int l = threadIdx.x & (kWave - 1);
    double run[ITEMS];      // sums since the last mark inside the lane
    bool mark[ITEMS];
    unsigned long long any = 0;
    int below = 0, total = 0;   // marks in lower lanes, in the tile
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t c = tl.c[j / 2] >> (16 * (j & 1));
        mark[j] = (c & 0x8000u) != 0;
        const double x = (double)win[c & 0x7fffu];
        run[j] = fma_t((double)tl.v[j], x, mark[j] || j == 0 ? 0.0 : run[j > 0 ? j - 1 : 0]);
        const unsigned long long m = __ballot(mark[j]);
        any |= m;
        total += __builtin_popcountll(m);
        below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, below));
    }
    // the nearest lane at or below this one that holds a mark
    const unsigned long long upto = any & (~0ull >> (kWave - 1 - l));
    const int dist = upto ? l - (kWave - 1 - __builtin_clzll(upto)) : kWave;
    const double s = marked_scan(run[ITEMS - 1], dist, l);
    double open = dpp_f64<kDppWaveShr1>(s);   // of the pair open where the lane begins
    if (below == 0) open += wk.carry;
    const double end = readlane_f64(s, kWave - 1);
    wk.carry = any ? end : wk.carry + end;
    int at = wk.held + below - wk.skip;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        if (mark[j]) {
            if (at >= 0) sp[at] = open + (j > 0 ? run[j > 0 ? j - 1 : 0] : 0.0);
            open = 0.0;
            ++at;
        }
    }
    wave_lds_sync();
    wk.held = min(wk.held + total - wk.skip, p1 - wk.from);
    wk.skip = 0;
    window_flush<ITEMS>(a, sp, (wk.from + wk.held) & ~(kWave - 1), wk);
}

}  // namespace

// First pass: workgroup c runs chunk c, pairs of window chunk_w[c]; its
// wavefront v runs pairs [wave_p[i], wave_p[i+1]), i = c*NW + v, whose entries
// start at wave_k[i] (the next wavefront's start ends them).  Tiles lie on
// multiples of ITEMS entries from the range's start rounded down, so a range's
// first tile may begin with up to three entries before it: wave_c[i] counts
// the pairs that start before the tile.  The window's x values (WB bytes at
// most) are copied to LDS once, eight loads in flight per lane, while the
// first tiles are on their way.
// What bounds it is the memory system, not the sums: without its stores it
// takes 39 us, without the gathers or the scan the same as with them.  On the
// 1,000,000-row Zipf matrix (16.2 M entries, 5.4 M pairs, 768 threads) it takes
// 46 us where one lane per pair, walking products staged in LDS between pair
// starts read from memory, took 63 us: 16.2 us of the difference are the
// partials (written as each tile's run they cost 16 us, in whole aligned
// groups 7) and the pair starts no longer read; values loaded without the
// non-temporal hint (a lane's 32 bytes are two loads of the same lines) give
// 3 us, two tiles in flight rather than four 4 us, and an XCD taking
// neighbouring chunks 2 us.
constexpr int kRing = 2;   // tiles in flight per wavefront

template <typename T, int BS, int WB, int E>
__global__ __launch_bounds__(BS) void k_xwin(XwinArgs a)
{
    constexpr int NW = BS / kWave;
    constexpr int WC = WB / (int)sizeof(T);
    constexpr int ITEMS = E / kWave;
    static_assert(WC <= 0x8000, "a column word has 15 bits of column");
    __shared__ T win[WC];
    __shared__ double sp[NW * (E + kWave)];
    // XCD k runs the k-th eighth of the chunks, so that a window's chunks, which
    // copy the same x, share an L2
    const int b = (int)blockIdx.x, xcd = b % kXcds, each = a.nchunk / kXcds, rest = a.nchunk % kXcds;
    const int c = xcd * each + min(xcd, rest) + b / kXcds;
    const int l = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int i = c * NW + wv;
    const int p0 = a.wave_p[i], p1 = a.wave_p[i + 1];
    const int64_t k0 = a.wave_k[i] & ~3, k1 = a.wave_k[i + 1];
    const int nt = p0 < p1 ? (int)((k1 - k0 + E - 1) / E) : 0;
    using Tile = WinTile<T, ITEMS>;
    // tile t of the range (clamped to the last: the ring's loads are issued
    // unconditionally)
    auto load = [&](int t, Tile &tl) {
        window_load<T, ITEMS>(a, k0 + (int64_t)max(min(t, nt - 1), 0) * E + l * ITEMS, tl);
    };
    Tile ring[kRing];
#pragma unroll
    for (int r = 0; r < kRing - 1; ++r) load(r, ring[r]);
    const int wnd = a.chunk_w[c];
    const int64_t col0 = (int64_t)wnd * WC;
    const int ncw = (int)min<int64_t>((int64_t)WC, a.n - col0);
    const T *xs = (const T *)a.x + col0;
    constexpr int BATCH = 8;
    for (int i0 = 0; i0 < ncw; i0 += BS * BATCH) {
        T t[BATCH];
        // clamped, so the loads are issued unconditionally (a chunk's window
        // holds at least one column)
#pragma unroll
        for (int j = 0; j < BATCH; ++j) t[j] = xs[min(i0 + j * BS + (int)threadIdx.x, ncw - 1)];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int at = i0 + j * BS + (int)threadIdx.x;
            if (at < ncw) win[at] = t[j];
        }
    }
    __syncthreads();
    double *my_sp = sp + wv * (E + kWave);
    WinWalk wk{0.0, 0, p0, p0 - a.wave_c[i] + 1};
    // ring slots are indexed by constants once the inner loop is unrolled, so
    // the ring stays in registers
    for (int t = 0; t < nt; t += kRing) {
#pragma unroll
        for (int r = 0; r < kRing; ++r) {
            load(t + r + kRing - 1, ring[(r + kRing - 1) % kRing]);
            if (r == 0 || t + r < nt) window_tile<T, ITEMS>(a, win, ring[r], my_sp, p1, wk);
        }
    }
    if (nt == 0) return;
    // the last pair, when no mark followed it in the last tile
    if (wk.from + wk.held < p1) {
        if (l == 0) my_sp[wk.held] = wk.carry;
        ++wk.held;
        wave_lds_sync();
    }
    window_flush<ITEMS>(a, my_sp, p1, wk);
}

// Second pass: workgroup b reads block b's partials run by run (window w's
// run of pairs from first[b][w] fills slots pre[b][w]..pre[b][w+1]; the
// window of a slot comes from a map built in LDS; all of a lane's loads in
// one round) and places each in LDS in row order, so that each of the block's
// rows then adds its own contiguous partials (its windows in order, four
// interleaved sums; 0 for a row with no entries), rounds once and, fused,
// forms w = alpha*y + x.
// Threads per workgroup of the adding pass: one per row of a 1,024-row
// block, sixteen wavefronts (two workgroups per compute unit fit the LDS,
// so eight wavefronts per SIMD hide the pass's three dependent rounds of
// loads: 22.7 us on the 1M-row Zipf matrix against 23.7 us with 512
// threads and 27.1 us with 256).
constexpr int kXsumBS = 1024;

template <typename T, bool FUSED>
__global__ __launch_bounds__(kXsumBS) void k_xwin_sum(XsumArgs a)
{
    constexpr int RPT = (int)(kXwinMaxRb / kXsumBS);   // rows per thread at most
    __shared__ double stage[kXwinStage];     // the block's partials in row order
    __shared__ uint16_t wof[kXwinStage];     // window of each slot
    __shared__ int pre[kXwinMaxWin + 1];
    __shared__ int first[kXwinMaxWin];
    const int b = (int)blockIdx.x;
    const int t = (int)threadIdx.x;
    const int S = a.nwin;
    const int64_t r0 = (int64_t)b * a.rb;
    // the pair ranges of the thread's rows r0 + t + kXsumBS*q (clamped rows for
    // threads without one: no load here sits in a branch, so none is waited
    // for early), in flight during the staging
    int s[RPT], e[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int64_t ic = min(r0 + t + kXsumBS * q, a.m - 1);
        s[q] = a.pos_ptr[ic];
        e[q] = a.pos_ptr[ic + 1];
    }
    const int base = a.pos_ptr[r0];
    const int *bpre = a.pre + (int64_t)b * (S + 1);
    const int *bfirst = a.first + (int64_t)b * S;
    for (int w = t; w <= S; w += kXsumBS) {
        pre[w] = bpre[w];
        if (w < S) first[w] = bfirst[w];
    }
    __syncthreads();
    const int total = pre[S];
    // every slot of the block in one round of loads (U per lane; slots
    // clamped to the last one, so the loads are issued unconditionally):
    // first the slots' places in row order, which need nothing else, then,
    // once the map of windows is built, the partials
    constexpr int U = (int)(kXwinStage / kXsumBS);
    static_assert(U * kXsumBS == kXwinStage, "staging area is a whole number of rounds");
    uint16_t place[U];
    if (total > 0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            place[u] = __builtin_nontemporal_load(a.rowpos + base + min(u * kXsumBS + t, total - 1));
    }
    for (int w = t; w < S; w += kXsumBS)
        for (int j = pre[w]; j < pre[w + 1]; ++j) wof[j] = (uint16_t)w;
    __syncthreads();
    if (total > 0) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int jj = min(u * kXsumBS + t, total - 1);
            const int w = wof[jj];
            v[u] = __builtin_nontemporal_load(a.part + first[w] + (jj - pre[w]));
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u * kXsumBS + t < total) stage[place[u]] = v[u];
    }
    __syncthreads();
    // each row's partials are contiguous: four interleaved sums (a fixed
    // order, so the result is reproducible)
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int64_t i = r0 + t + kXsumBS * q;
        if (t + kXsumBS * q >= a.rb || i >= a.m) break;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        int k = s[q] - base;
        const int ke = e[q] - base;
        for (; k + 4 <= ke; k += 4) {
            a0 += stage[k];
            a1 += stage[k + 1];
            a2 += stage[k + 2];
            a3 += stage[k + 3];
        }
        if (k < ke) a0 += stage[k];
        if (k + 1 < ke) a1 += stage[k + 1];
        if (k + 2 < ke) a2 += stage[k + 2];
        const double acc = (a0 + a1) + (a2 + a3);
        const T yt = (T)acc;
        ((T *)a.y)[i] = yt;
        if constexpr (FUSED) ((T *)a.w)[i] = fma_t((T)a.alpha, yt, ((const T *)a.x)[i]);
    }
}

namespace {

template <typename T, int BS, int WB, int E>
hipError_t L_xwin(const XwinArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL((k_xwin<T, BS, WB, E>), dim3((unsigned)a.nchunk), dim3(BS), 0, s, a);
    return hipGetLastError();
}

#define XENTRY(BS, KIB, E) {BS, KIB, E, {L_xwin<float, BS, KIB * 1024, E>, L_xwin<double, BS, KIB * 1024, E>}}

// (threads per workgroup, window KiB, row-stream entries per wavefront):
// 128 KiB windows leave room for one workgroup per compute unit, 64 KiB
// windows for two.
const XwinEntry kXwin[] = {
    XENTRY(512, 128, 256),
    XENTRY(1024, 128, 128),
    XENTRY(768, 128, 256),   // 161,792 bytes of LDS: twelve wavefronts of 256-entry tiles
    XENTRY(256, 64, 256),
    XENTRY(512, 64, 256),
};

}  // namespace

const XwinEntry *xwin_table(int *count)
{
    *count = (int)(sizeof(kXwin) / sizeof(kXwin[0]));
    return kXwin;
}

hipError_t launch_xwin_sum(int dtype, bool fused, const XsumArgs &a, hipStream_t s)
{
    if (a.m <= 0) return hipSuccess;
    const unsigned g = (unsigned)((a.m + a.rb - 1) / a.rb);
    if (dtype == 1) {
        if (fused) hipLaunchKernelGGL((k_xwin_sum<double, true>), dim3(g), dim3(kXsumBS), 0, s, a);
        else hipLaunchKernelGGL((k_xwin_sum<double, false>), dim3(g), dim3(kXsumBS), 0, s, a);
    } else {
        if (fused) hipLaunchKernelGGL((k_xwin_sum<float, true>), dim3(g), dim3(kXsumBS), 0, s, a);
        else hipLaunchKernelGGL((k_xwin_sum<float, false>), dim3(g), dim3(kXsumBS), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace spk
