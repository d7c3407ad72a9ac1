// kernels_batch.hip -- one launch over many independent CSR instances.
//
// The host planner cuts every instance into tiles (row ranges) and gives
// each tile the kernel chosen for the instance's shape class: an LDS-staged
// row stream (mode 0) or G lanes per row (mode G).  The kernel either runs
// one workgroup per group of tiles (one tile per wavefront), or is
// persistent: a grid sized to fill the GPU whose workgroups walk the groups
// in fixed strides.  Neither keeps state between launches, so a launch can
// be captured in a hipGraph and replayed.
//
// Each row is always reduced by the same code in the same order, so a
// row's result depends only on (matrix, tile mode): an instance gives the
// same bits alone, in a batch, or in any other mix.
#include "device_common.h"
#include "device_rows.h"
#include "kernels.h"

namespace spk {

// Tiles per run when tile groups are dealt to the XCDs (measured on the
// 4096-instance banded batch: runs of 32 to 128 tiles stream 5% faster than
// contiguous eighths, and 2-3% faster than dealing single groups).
constexpr int kXcdRunTiles = 64;

// Tiles are wavefront-sized: every wavefront of a workgroup runs its own
// tile, with its own slice of the workgroup's LDS (TILE/(BS/64) products and
// 129 row offsets), and no workgroup barrier.
template <typename T, int BS, int TILE>
struct WaveTiles {
    static constexpr int NW = BS / kWave;        // wavefronts per workgroup
    static constexpr int ENTRIES = TILE / NW;    // row-stream capacity of one wavefront
    static constexpr int ITEMS = ENTRIES / kWave;
    static_assert(ITEMS * kWave * NW == TILE, "tile must split evenly over the wavefronts");
};

// An address every lane holds, as a scalar.
__device__ __forceinline__ uint64_t uniform_addr(const void *p)
{
    const uint64_t a = (uint64_t)p;
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
}

// Reads the record of launch tile `tile`, and where its y and w go.  The
// record stays wavefront-uniform: with a request table the 16-bit map entry
// arrives through a vector load and is made uniform again, and the record is
// read through the constant address space (scalar loads).
template <typename T, bool REQ>
__device__ __forceinline__ BatchTile load_tile(const BatchArgs<T> &a, int tile, T **y, T **w)
{
    const BatchTile *tp = a.tiles + tile;
    int64_t voff = 0;
    if constexpr (REQ) {
        const int r = __builtin_amdgcn_readfirstlane((int)a.req_of_tile[tile]);
        const BatchReq *q = a.reqs + r;
        tp = q->tiles + (tile - q->first);
        voff = q->vec_off;
        *y = (T *)uniform_addr(q->y);
        *w = (T *)uniform_addr(q->w);
    }
    const uint64_t tu = uniform_addr(tp);
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const __attribute__((address_space(4))) u32x4 *src = (const __attribute__((address_space(4))) u32x4 *)tu;
    u32x4 parts[sizeof(BatchTile) / sizeof(u32x4)];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(BatchTile) / sizeof(u32x4)); ++i) parts[i] = src[i];
    BatchTile td;
    __builtin_memcpy(&td, parts, sizeof td);
    if constexpr (REQ) {
        td.vec_off = voff;
    } else {
        *y = a.y + td.vec_off;
        *w = a.w ? a.w + td.vec_off : nullptr;
    }
    return td;
}

template <typename T, int BS, int TILE, int XW, bool REQ, bool NTC>
__device__ __forceinline__ void run_wave_tile(const BatchArgs<T> &a, int tile, double *sp, int *srp, T *xs)
{
    T *y, *w;
    const BatchTile td = load_tile<T, REQ>(a, tile, &y, &w);
    const int32_t *rp = td.rp;
    const int32_t *ci = td.ci;
    const T *val = (const T *)td.val;
    const T *x = a.x + td.vec_off;
    constexpr int ITEMS = WaveTiles<T, BS, TILE>::ITEMS;
    switch (td.mode) {
    case 0:  // entries and rows fit the wavefront's LDS slice (guaranteed by the planner)
        wave_stream<T, ITEMS, false, 0, 4, false, NTC>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1, td.k0, td.k1, sp,
                                                       srp);
        break;
    case 1:  // the same, x from the tile's window in LDS when it fits the kernel's room
        wave_stream<T, ITEMS, false, XW, 4, false, NTC>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1, td.k0, td.k1, sp,
                                                        srp, td.xlo, XW > 0 && td.xn <= XW ? td.xn : 0, xs);
        break;
    case 3:  // mode 1 with compact columns: ci holds each entry's byte offset in the window (which fits)
        if constexpr (XW > 0 && XW <= 256)
            wave_stream<T, ITEMS, false, XW, 1, false, NTC>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1, td.k0, td.k1,
                                                            sp, srp, td.xlo, td.xn, xs);
        break;
    case 5:  // compact columns of a wider tile: two-byte offsets from xlo, x gathered from memory
        wave_stream<T, ITEMS, false, XW, 2, false, NTC>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1, td.k0, td.k1, sp,
                                                        srp, td.xlo, 0, xs);
        break;
    case 2: wave_group_rows<T, 2>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1); break;
    case 4: wave_group_rows<T, 4>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1); break;
    case 8: wave_group_rows<T, 8>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1); break;
    case 16: wave_group_rows<T, 16>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1); break;
    case 32: wave_group_rows<T, 32>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1); break;
    default: wave_group_rows<T, 64>(rp, ci, val, x, y, w, a.alpha, td.r0, td.r1); break;
    }
}

template <typename T, int BS, int TILE, int XW, bool REQ, bool NTC>
__global__ __launch_bounds__(BS) void k_batch_grid(BatchArgs<T> a)
{
    using WT = WaveTiles<T, BS, TILE>;
    __shared__ double sp[TILE];
    __shared__ int srp[WT::NW * (kWaveTileRows + 1)];
    __shared__ T xs[WT::NW * (XW > 0 ? XW : 1)];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ngroups = (a.ntiles + WT::NW - 1) / WT::NW;
    // runs of kXcdRunTiles tiles dealt to the XCDs in turn
    const int tile = xcd_chunk((int)blockIdx.x, ngroups, kXcdRunTiles / WT::NW) * WT::NW + wv;
    if (tile >= a.ntiles) return;
    run_wave_tile<T, BS, TILE, XW, REQ, NTC>(a, tile, sp + wv * WT::ENTRIES, srp + wv * (kWaveTileRows + 1),
                                             xs + wv * (XW > 0 ? XW : 1));
}

// Persistent form: a grid of bounded size (the host's persistent_cap), each
// workgroup walking the tile groups b, b + gridDim, ... (dealt to the XCDs as
// in the grid form: the grid is a multiple of 8 when a workgroup has more
// than one group).  A batch with no more groups than the cap runs as in the
// grid form.  The walk is fixed, so there is no queue: with one queue head
// per XCD every wavefront claimed at least once and counted itself out, and
// those device-scope atomics on nine addresses set the launch's length.
// 96 banded FP32 instances (8,390 tiles, 37 MB): 104.3 us with the queues,
// 12.0 us without.
template <typename T, int BS, int TILE, int XW, bool NTC>
__global__ __launch_bounds__(BS) void k_batch_persistent(BatchArgs<T> a)
{
    using WT = WaveTiles<T, BS, TILE>;
    __shared__ double sp[TILE];
    __shared__ int srp[WT::NW * (kWaveTileRows + 1)];
    __shared__ T xs[WT::NW * (XW > 0 ? XW : 1)];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int ngroups = (a.ntiles + WT::NW - 1) / WT::NW;
    for (int g = (int)blockIdx.x; g < ngroups; g += (int)gridDim.x) {
        const int tile = xcd_chunk(g, ngroups, kXcdRunTiles / WT::NW) * WT::NW + wv;
        if (tile < a.ntiles)
            run_wave_tile<T, BS, TILE, XW, false, NTC>(a, tile, sp + wv * WT::ENTRIES, srp + wv * (kWaveTileRows + 1),
                                                       xs + wv * (XW > 0 ? XW : 1));
    }
}

// The x windows of mode-1 and mode-3 tiles (see launch_tile_windows), one
// wavefront per tile.  A mode-3 tile whose window fits writes its entries'
// offsets in the window to c8 (at the entries' own positions: instance
// arrays at ci + d map to c8 + d) and takes c8 as its column array; one
// whose columns span at most 65,536 does the same with two-byte offsets
// from its first column in c16 and becomes a mode-5 tile (x gathered from
// memory), or, while c16 is NULL, counts itself in *need16 and becomes a
// mode-1 tile; any other becomes a mode-1 tile.
__global__ __launch_bounds__(256) void k_tile_windows(BatchTile *tiles, int64_t ntiles, int cap, const int32_t *ci0,
                                                      uint8_t *c8, uint16_t *c16, int *need16)
{
    const int64_t t = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave;
    if (t >= ntiles) return;
    const int l = threadIdx.x & (kWave - 1);
    BatchTile &td = tiles[t];
    const int mode = td.mode;
    if (mode != 1 && mode != 3) return;
    const int32_t *ci = td.ci;
    const int k0 = td.k0, k1 = td.k1;
    int lo = INT32_MAX, hi = -1;
    for (int k = k0 + l; k < k1; k += kWave) {
        const int c = ci[k];
        lo = min(lo, c);
        hi = max(hi, c);
    }
#pragma unroll
    for (int d = 1; d < kWave; d *= 2) {
        lo = min(lo, __shfl_xor(lo, d));
        hi = max(hi, __shfl_xor(hi, d));
    }
    const bool fits = hi >= lo && (int64_t)hi - lo + 1 <= cap;
    const bool span16 = hi >= lo && (int64_t)hi - lo < 65536;
    const bool one = mode == 3 && fits && cap <= 256 && c8 != nullptr;
    const bool two = mode == 3 && !one && span16 && c16 != nullptr;
    uint8_t *cb = one ? c8 + (ci - ci0) : nullptr;
    uint16_t *cw = two ? c16 + (ci - ci0) : nullptr;
    if (one)
        for (int k = k0 + l; k < k1; k += kWave) cb[k] = (uint8_t)(ci[k] - lo);
    if (two)
        for (int k = k0 + l; k < k1; k += kWave) cw[k] = (uint16_t)(ci[k] - lo);
    if (l == 0) {
        td.xlo = fits || two ? lo : 0;
        td.xn = fits && !two ? hi - lo + 1 : 0;
        if (mode == 3) {
            td.mode = one ? 3 : two ? 5 : 1;
            if (one) td.ci = reinterpret_cast<const int32_t *>(cb);
            if (two) td.ci = reinterpret_cast<const int32_t *>(cw);
            if (!one && !two && span16 && c16 == nullptr && need16 != nullptr) atomicAdd(need16, 1);
        }
    }
}

namespace {

template <typename T, int BS, int TILE, int XW>
int occ_batch()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(&k_batch_persistent<T, BS, TILE, XW, false>),
                                                     BS, 0) != hipSuccess)
        n = 1;
    return n > 0 ? n : 1;
}

template <typename T, int BS, int TILE, int XW, int KIND, bool NTC>
hipError_t L_batch(const void *p, dim3 g, hipStream_t s)
{
    const BatchArgs<T> &a = *(const BatchArgs<T> *)p;
    if constexpr (KIND == kBatchPersistent)
        hipLaunchKernelGGL((k_batch_persistent<T, BS, TILE, XW, NTC>), g, dim3(BS), 0, s, a);
    else
        hipLaunchKernelGGL((k_batch_grid<T, BS, TILE, XW, KIND == kBatchRequests, NTC>), g, dim3(BS), 0, s, a);
    return hipGetLastError();
}

#define BFN(T, BS, TILE, XW, REQ)                                                                        \
    {{L_batch<T, BS, TILE, XW, kBatchGrid, false>, L_batch<T, BS, TILE, XW, kBatchPersistent, false>, REQ}, \
     {L_batch<T, BS, TILE, XW, kBatchGrid, true>, L_batch<T, BS, TILE, XW, kBatchPersistent, true>, nullptr}}
#define BOCC(BS, TILE, XW) {occ_batch<float, BS, TILE, XW>, occ_batch<double, BS, TILE, XW>}
#define BENTRY(BS, TILE, XW) \
    {BS, TILE, XW, {BFN(float, BS, TILE, XW, nullptr), BFN(double, BS, TILE, XW, nullptr)}, BOCC(BS, TILE, XW)}
// with the request-table form too (serving's shape)
#define BENTRY_REQ(BS, TILE, XW)                                                       \
    {BS, TILE, XW,                                                                     \
     {BFN(float, BS, TILE, XW, (L_batch<float, BS, TILE, XW, kBatchRequests, false>)),   \
      BFN(double, BS, TILE, XW, (L_batch<double, BS, TILE, XW, kBatchRequests, false>))}, \
     BOCC(BS, TILE, XW)}

// (threads per workgroup, LDS products per workgroup, LDS room for x per
// wavefront): a wavefront's row stream holds TILE/(BS/64) entries: 256
// to 2048; the kernels with room for x run mode-1 tiles from LDS
const BatchEntry kBatch[] = {
    BENTRY(256, 2048, 0), BENTRY(256, 1024, 0), BENTRY(256, 4096, 0),
    BENTRY(128, 1024, 0), BENTRY(128, 2048, 0),
    BENTRY(512, 2048, 0), BENTRY(512, 4096, 0),
    BENTRY_REQ(256, 2048, 256), BENTRY(256, 4096, 256), BENTRY(128, 2048, 256),
    BENTRY(128, 1024, 256), BENTRY(64, 1024, 256), BENTRY(64, 512, 256), BENTRY(64, 2048, 256),
};

}  // namespace

const BatchEntry *batch_table(int *count)
{
    *count = (int)(sizeof(kBatch) / sizeof(kBatch[0]));
    return kBatch;
}

hipError_t launch_tile_windows(BatchTile *tiles, int64_t ntiles, int cap, hipStream_t s, const int32_t *ci0,
                               uint8_t *c8, uint16_t *c16, int *need16)
{
    if (ntiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tile_windows, dim3((unsigned)((ntiles + 3) / 4)), dim3(256), 0, s, tiles, ntiles, cap, ci0,
                       c8, c16, need16);
    return hipGetLastError();
}

}  // namespace spk
