// Implicit-GEMM convolution engine, direct-to-LDS variant: kernels with the four-slot ring and their launches.
#include "igemm_dma_tile.h"

namespace dlk {

template <class T, int BM, int BN, int WM, int WN, bool CMAJOR, bool BT = false, bool RES = false>
__global__ __launch_bounds__(WM *WN * 64) void igemm_dma_kernel(const IgemmArgs p)
{
    // Split reduction into 2, 4 or 8 ranges: range s runs on the XCDs s, s + ranges, ... (workgroups are dealt to the
    // eight XCDs in turn, x fastest), so that an XCD's L2 holds one range of the channels of both operands
    // instead of all of them (ASPP 3x3 forward: 4.7 MB per XCD instead of 37 MB).
    if (gridDim.y > 1 && 8 % gridDim.y == 0) {
        const unsigned id = blockIdx.y * gridDim.x + blockIdx.x;
        igemm_dma_tile<T, BM, BN, WM, WN, CMAJOR, BT, 32, 4, false, RES>(p, (int)(id / gridDim.y), (int)(id % gridDim.y));
        return;
    }
    igemm_dma_tile<T, BM, BN, WM, WN, CMAJOR, BT, 32, 4, false, RES>(p, xcd_remap(blockIdx.x, gridDim.x), blockIdx.y);
}

// Several small GEMMs of one tile shape in one launch (the stride-parity classes of a strided
// data gradient on a small image, each of which alone is a ~10 us kernel): workgroup ids are
// dealt to the GEMMs in turn.  Channel-major order only.
template <class T, int BM, int BN, int WM, int WN, bool BT>
__global__ __launch_bounds__(WM *WN * 64) void igemm_dma_batch_kernel(const IgemmBatch b)
{
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int which = id % b.n, tile = id / b.n;
    const IgemmArgs &p = b.a[which];
    const int64_t M = (int64_t)p.NB * p.OH * p.OW;
    const int64_t tiles = ((M + BM - 1) / BM) * ((p.Nout + BN - 1) / BN);
    if (tile >= tiles) return;                           // this GEMM has fewer tiles than the largest
    igemm_dma_tile<T, BM, BN, WM, WN, true, BT>(p, tile, 0);
}

template <class T, int BM, int BN, int WM, int WN>
static hipError_t launch_dma_cfg(const IgemmArgs &a, hipStream_t stream)
{
    const int64_t M = (int64_t)a.NB * a.OH * a.OW;
    const int64_t tiles = ((M + BM - 1) / BM) * ((a.Nout + BN - 1) / BN);
    if (tiles <= 0 || tiles > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles, (unsigned)(a.c_outer && a.ksplits > 1 ? a.ksplits : 1)), block(WM * WN * 64);
    if (a.b_transposed) {
        if (!a.c_outer || a.Nout % 8 != 0) return hipErrorInvalidValue;
        DLK_LAUNCH(kname("igemm_dma_kernel.bt", {BM, BN}), (igemm_dma_kernel<T, BM, BN, WM, WN, true, true>), grid, block, 0, stream, a);
    } else if (a.c_outer && BN <= 128 && BM * BN >= 4096 && grid.y == 1 && resid_prefetchable(a)) {
        if constexpr (BN <= 128 && BM * BN >= 4096)
            DLK_LAUNCH(kname("igemm_dma_kernel.cmajor.res", {BM, BN}), (igemm_dma_kernel<T, BM, BN, WM, WN, true, false, true>), grid, block, 0, stream, a);
    } else if (a.c_outer)
        DLK_LAUNCH(kname("igemm_dma_kernel.cmajor", {BM, BN}), (igemm_dma_kernel<T, BM, BN, WM, WN, true>), grid, block, 0, stream, a);
    else
        DLK_LAUNCH(kname("igemm_dma_kernel.tapmajor", {BM, BN}), (igemm_dma_kernel<T, BM, BN, WM, WN, false>), grid, block, 0, stream, a);
    return dlk::launch_status();
}

template <class T>
static hipError_t dispatch_dma(const IgemmArgs &a, int cfg, hipStream_t stream)
{
    switch (cfg) {
        case 0: return launch_dma_cfg<T, 256, 256, 2, 4>(a, stream);   // 8 waves, wave tile 128x64
        case 2: return launch_dma_cfg<T, 128, 128, 2, 2>(a, stream);   // 4 waves, wave tile 64x64
        case 3: return launch_dma_cfg<T, 128, 64, 2, 2>(a, stream);    // 4 waves, wave tile 64x32
        case 4: return launch_dma_cfg<T, 64, 32, 2, 1>(a, stream);     // 2 waves, wave tile 32x32
        case 8: return launch_dma_cfg<T, 64, 64, 2, 1>(a, stream);     // 2 waves, wave tile 32x64
        default: return hipErrorInvalidValue;
    }
}

template <class T, int BM, int BN, int WM, int WN>
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
    if (tiles_max <= 0 || tiles_max * b.n > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(tiles_max * b.n)), block(WM * WN * 64);
    if (b.a[0].b_transposed) DLK_LAUNCH(kname("igemm_dma_batch_kernel.bt", {BM, BN}), (igemm_dma_batch_kernel<T, BM, BN, WM, WN, true>), grid, block, 0, stream, b);
    else DLK_LAUNCH(kname("igemm_dma_batch_kernel", {BM, BN}), (igemm_dma_batch_kernel<T, BM, BN, WM, WN, false>), grid, block, 0, stream, b);
    return dlk::launch_status();
}

template <class T>
static hipError_t dispatch_dma_batch(const IgemmBatch &b, int cfg, hipStream_t stream)
{
    switch (cfg) {
        case 0: return launch_dma_batch_cfg<T, 256, 256, 2, 4>(b, stream);
        case 2: return launch_dma_batch_cfg<T, 128, 128, 2, 2>(b, stream);
        case 3: return launch_dma_batch_cfg<T, 128, 64, 2, 2>(b, stream);
        case 4: return launch_dma_batch_cfg<T, 64, 32, 2, 1>(b, stream);
        case 8: return launch_dma_batch_cfg<T, 64, 64, 2, 1>(b, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_igemm_dma_batch(const IgemmBatch &b, bool is_bf16, int cfg, hipStream_t stream)
{
    if (b.n < 1 || b.n > IgemmBatch::MAX) return hipErrorInvalidValue;
    return is_bf16 ? dispatch_dma_batch<BF16>(b, cfg, stream) : dispatch_dma_batch<F16>(b, cfg, stream);
}

hipError_t launch_igemm_dma(const IgemmArgs &a, bool is_bf16, int cfg, hipStream_t stream)
{
    return is_bf16 ? dispatch_dma<BF16>(a, cfg, stream) : dispatch_dma<F16>(a, cfg, stream);
}

}  // namespace dlk
