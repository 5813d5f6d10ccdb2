// Kernels and launches of the direct-to-LDS engine, included once per storage type.
#pragma once
#include "igemm_dma_tile.h"

namespace dlk {

template <class T, int BM, int BN, int WM, int WN, int KB, int STAGES, bool PP, bool CMAJOR, bool BT = false, bool RES = false>
__global__ __launch_bounds__(WM *WN * 64) void igemm_dma_kernel(const IgemmArgs p)
{
    // Split reduction into 2, 4 or 8 ranges: range s runs on the XCDs s, s + ranges, ... (workgroups are dealt to the
    // eight XCDs in turn, x fastest), so that an XCD's L2 holds one range of the channels of both operands
    // instead of all of them (ASPP 3x3 forward: 4.7 MB per XCD instead of 37 MB).
    if (gridDim.y > 1 && 8 % gridDim.y == 0) {
        const unsigned id = blockIdx.y * gridDim.x + blockIdx.x;
        igemm_dma_tile<T, BM, BN, WM, WN, CMAJOR, BT, KB, STAGES, false, RES, PP>(p, (int)(id / gridDim.y), (int)(id % gridDim.y));
        return;
    }
    igemm_dma_tile<T, BM, BN, WM, WN, CMAJOR, BT, KB, STAGES, false, RES, PP>(p, xcd_remap(blockIdx.x, gridDim.x), blockIdx.y);
}

// Several GEMMs of one tile shape in one launch, the longest reduction first: the stride-parity classes of a strided data
// gradient, which read the same tensor.  Channel-major order only.  One after the other each class ends in a round of
// workgroups that is partly empty, and starts with one that waits for its first loads; here an XCD (hardware deals workgroups to
// the eight in turn) has a range of every class's tiles and takes the classes in order, so that what is left for the end is
// short.  3x3, stride 2, batch 2, four launches / workgroups dealt to the classes in turn / in this order: 384 x 576 x 256 ->
// 256 183 / 200 / 162 us; 229 x 361, 160 -> 256 69 / 61 / 54; 145 x 351, 512 -> 64 38 / 36 / 28; 112 x 183, 64 -> 64 20 / 11 / 11.
template <class T, int BM, int BN, int WM, int WN, int KB, int STAGES, bool PP, bool BT>
__global__ __launch_bounds__(WM *WN * 64) void igemm_dma_batch_kernel(const IgemmBatch b)
{
    const int per = (int)gridDim.x / (8 * b.n), xcd = blockIdx.x % 8, slot = blockIdx.x / 8;   // per: ceil(b.tiles / 8)
    const int tile = (int)((int64_t)b.tiles * xcd / 8) + slot % per;
    if (tile >= (int)((int64_t)b.tiles * (xcd + 1) / 8)) return;
    const IgemmArgs &p = b.a[slot / per];
    const int64_t M = (int64_t)p.NB * p.OH * p.OW;
    const int64_t tiles = ((M + BM - 1) / BM) * ((p.Nout + BN - 1) / BN);
    if (tile >= tiles) return;                           // this GEMM has fewer tiles than the largest
    igemm_dma_tile<T, BM, BN, WM, WN, true, BT, KB, STAGES, false, false, PP>(p, tile, 0);
}

static std::string dma_label(const char *base, int bm, int bn, int kb) { return kname((std::string(base) + (kb == 64 ? ".k64" : "")).c_str(), {bm, bn}); }

template <class T, int BM, int BN, int WM, int WN, int KB, int STAGES, bool PP = false>
static hipError_t launch_dma_cfg(const IgemmArgs &a, hipStream_t stream)
{
    const int64_t M = (int64_t)a.NB * a.OH * a.OW;
    const int64_t tiles = ((M + BM - 1) / BM) * ((a.Nout + BN - 1) / BN);
    if (tiles <= 0 || tiles > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles, (unsigned)(a.c_outer && a.ksplits > 1 ? a.ksplits : 1)), block(WM * WN * 64);
    if (a.b_transposed) {
        if (!a.c_outer || a.Nout % 8 != 0) return hipErrorInvalidValue;
        DLK_LAUNCH(dma_label("igemm_dma_kernel.bt", BM, BN, KB), (igemm_dma_kernel<T, BM, BN, WM, WN, KB, STAGES, PP, true, true>), grid, block, 0, stream, a);
    } else if (a.c_outer && BN <= 128 && BM * BN >= 4096 && grid.y == 1 && resid_prefetchable(a)) {
        if constexpr (BN <= 128 && BM * BN >= 4096)
            DLK_LAUNCH(dma_label("igemm_dma_kernel.cmajor.res", BM, BN, KB), (igemm_dma_kernel<T, BM, BN, WM, WN, KB, STAGES, PP, true, false, true>), grid, block, 0, stream, a);
    } else if (a.c_outer)
        DLK_LAUNCH(dma_label("igemm_dma_kernel.cmajor", BM, BN, KB), (igemm_dma_kernel<T, BM, BN, WM, WN, KB, STAGES, PP, true>), grid, block, 0, stream, a);
    else return hipErrorInvalidValue;
    return dlk::launch_status();
}

template <class T, int BM, int BN, int WM, int WN>
static hipError_t launch_dma_tap_major(const IgemmArgs &a, hipStream_t stream)
{
    const int64_t M = (int64_t)a.NB * a.OH * a.OW;
    const int64_t tiles = ((M + BM - 1) / BM) * ((a.Nout + BN - 1) / BN);
    if (tiles <= 0 || tiles > 0x7fffffff || a.b_transposed) return hipErrorInvalidValue;
    DLK_LAUNCH(dma_label("igemm_dma_kernel.tapmajor", BM, BN, 32), (igemm_dma_kernel<T, BM, BN, WM, WN, 32, 4, false, false>), dim3((unsigned)tiles),
               dim3(WM * WN * 64), 0, stream, a);
    return dlk::launch_status();
}

template <class T, int BM, int BN, int WM, int WN, int KB, int STAGES, bool PP = false>
static hipError_t launch_dma_batch_cfg(const IgemmBatch &b, hipStream_t stream)
{
    int64_t tiles_max = 0;
    for (int i = 0; i < b.n; ++i) {
        const IgemmArgs &a = b.a[i];
        if (!a.c_outer || a.ksplits > 1 || a.b_transposed != b.a[0].b_transposed) return hipErrorInvalidValue;
        if (a.b_transposed && a.Nout % 8 != 0) return hipErrorInvalidValue;
        const int64_t M = (int64_t)a.NB * a.OH * a.OW;
        const int64_t tiles = ((M + BM - 1) / BM) * ((a.Nout + BN - 1) / BN);
        if (tiles > tiles_max) tiles_max = tiles;
    }
    if (tiles_max <= 0 || (tiles_max + 7) * b.n > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((tiles_max + 7) / 8 * 8 * b.n)), block(WM * WN * 64);
    IgemmBatch c = b;
    c.tiles = (int32_t)tiles_max;
    if (b.a[0].b_transposed) DLK_LAUNCH(dma_label("igemm_dma_batch_kernel.bt", BM, BN, KB), (igemm_dma_batch_kernel<T, BM, BN, WM, WN, KB, STAGES, PP, true>), grid, block, 0, stream, c);
    else DLK_LAUNCH(dma_label("igemm_dma_batch_kernel", BM, BN, KB), (igemm_dma_batch_kernel<T, BM, BN, WM, WN, KB, STAGES, PP, false>), grid, block, 0, stream, c);
    return dlk::launch_status();
}

// The tiles.  Eight waves (four for 64 x 64) with small wave tiles: what a step costs beyond its loads and products is
// a chain of instructions per wave (barrier, LDS reads, loads, products that wait for each other), which more waves of the
// same tile walk side by side: 6912 pixels, 256 -> 256, 3x3: 128 x 64 tiles of four waves 14.1 us, of eight waves 12.7 us.
// A step of 64 channels reads whole 128-byte lines: with 32 the other half of a line comes into the 32 KB L1
// again some taps later (64-byte pieces at 70 bytes per ns and compute unit, whole lines at 130).
template <class T>
static hipError_t dispatch_dma(const IgemmArgs &a, int cfg, hipStream_t stream)
{
    if (!a.c_outer) {
        switch (cfg) {
            case TILE_64x32: return launch_dma_tap_major<T, 64, 32, 2, 1>(a, stream);
            case TILE_64x64: return launch_dma_tap_major<T, 64, 64, 2, 2>(a, stream);
            case TILE_128x64: return launch_dma_tap_major<T, 128, 64, 4, 1>(a, stream);
            case TILE_128x128: return launch_dma_tap_major<T, 128, 128, 4, 2>(a, stream);
            case TILE_256x256: return launch_dma_tap_major<T, 256, 256, 2, 4>(a, stream);
            default: return hipErrorInvalidValue;
        }
    }
    switch (cfg) {
        case TILE_64x32: return launch_dma_cfg<T, 64, 32, 2, 1, 32, 4>(a, stream);
        case TILE_64x64: return launch_dma_cfg<T, 64, 64, 2, 2, 32, 4>(a, stream);
        case TILE_64x64_K64: return launch_dma_cfg<T, 64, 64, 2, 2, 64, 4>(a, stream);
        case TILE_128x64_K64: return launch_dma_cfg<T, 128, 64, 4, 2, 64, 3>(a, stream);
        case TILE_128x128: return launch_dma_cfg<T, 128, 128, 4, 2, 32, 4>(a, stream);
        case TILE_128x128_K64: return launch_dma_cfg<T, 128, 128, 4, 2, 64, 4, true>(a, stream);
        case TILE_256x128_K64: return launch_dma_cfg<T, 256, 128, 4, 2, 64, 3, true>(a, stream);
        case TILE_256x256: return launch_dma_cfg<T, 256, 256, 2, 4, 32, 4, true>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

template <class T>
static hipError_t dispatch_dma_batch(const IgemmBatch &b, int cfg, hipStream_t stream)
{
    switch (cfg) {
        case TILE_64x32: return launch_dma_batch_cfg<T, 64, 32, 2, 1, 32, 4>(b, stream);
        case TILE_64x64: return launch_dma_batch_cfg<T, 64, 64, 2, 2, 32, 4>(b, stream);
        case TILE_128x64_K64: return launch_dma_batch_cfg<T, 128, 64, 4, 2, 64, 3>(b, stream);
        case TILE_128x128: return launch_dma_batch_cfg<T, 128, 128, 4, 2, 32, 4>(b, stream);
        case TILE_256x256: return launch_dma_batch_cfg<T, 256, 256, 2, 4, 32, 4, true>(b, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace dlk
