// 1x1 layers with 32 or 64 input channels and many output pixels (the expanding layers of a residual block on a wide
// map, the data gradient of its contracting layer): the whole reduction is one 64-channel step of the direct-to-LDS
// engine's tile code, fetched at once.
//
// Bound by memory: a 128 x 128 tile moves 32 KB in, 32 KB out (and 32 KB of residual) for 16 MFMAs (32x32x16) per wave.  What
// counts is how many workgroups a CU holds at different stages of that: 32 KB of LDS and 122 registers leave room for
// four, where the ring kernel's 256 x 256 tile (128 KB, and two of its four steps multiply zeros) leaves one.
// Measured (fp16, plain / with bias, residual and ReLU, before -> after): 110592 pixels, 64 -> 256 23.3 -> 18.1 us /
// 49.2 -> 32.7 us (3.9 TB/s), 64 -> 128 15.6 -> 11.3 / 27.0 -> 19.7 us; 442368 pixels, 32 -> 96 40.9 -> 27.7 /
// 70.9 -> 52.5 us, 64 -> 304 105 -> 90 / 282 -> 162 us; data gradient with 64 output channels 23.2 -> 17.9 us.
#include "igemm_dma_tile.h"

namespace dlk {

template <class T, bool BT, bool RES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void igemm_short_kernel(const IgemmArgs p)
{
    igemm_dma_tile<T, 128, 128, 2, 2, true, BT, 64, 1, true, RES>(p, xcd_remap(blockIdx.x, gridDim.x), 0);
}

static int64_t short_tiles(const IgemmArgs &a)
{
    return (((int64_t)a.NB * a.OH * a.OW + 127) / 128) * ((a.Nout + 127) / 128);
}

// Two tiles per CU and more: with 48 tiles (3015 pixels, 64 -> 256) the ring kernel's smaller tiles take 5.1 us, this
// kernel 5.6.  Two such steps for up to 128 channels (64 KB of LDS, two workgroups per CU) gained 2-5 % on 442368 pixels
// and lost 11 % on 27648 (128 -> 512), so those layers stay with the ring.
bool igemm_short_applicable(const IgemmArgs &a)
{
    return a.TR * a.TS == 1 && a.Cin % 32 == 0 && a.Cin <= 64 && a.Nout > 64 && a.Nout % 8 == 0 && a.ksplits <= 1 &&
           short_tiles(a) >= 512;
}

template <class T>
static hipError_t launch_short(const IgemmArgs &a, hipStream_t stream)
{
    const int64_t tiles = short_tiles(a);
    if (tiles > 0x7fffffff || !igemm_short_applicable(a)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(256);
    if (a.b_transposed) {
        if (a.resid) return hipErrorInvalidValue;
        DLK_LAUNCH("igemm_short_kernel.bt", (igemm_short_kernel<T, true, false>), grid, block, 0, stream, a);
    } else if (resid_prefetchable(a))
        DLK_LAUNCH("igemm_short_kernel.res", (igemm_short_kernel<T, false, true>), grid, block, 0, stream, a);
    else
        DLK_LAUNCH("igemm_short_kernel", (igemm_short_kernel<T, false, false>), grid, block, 0, stream, a);
    return dlk::launch_status();
}

hipError_t launch_igemm_short(const IgemmArgs &a, bool is_bf16, hipStream_t stream)
{
    return is_bf16 ? launch_short<BF16>(a, stream) : launch_short<F16>(a, stream);
}

}  // namespace dlk
