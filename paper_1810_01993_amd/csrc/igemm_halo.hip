// Halo-tile kernels for stride-1 filters with several taps (gfx950): which layers they take, and the filter copy they read.
//
// A workgroup of such a kernel deposits the input patch of its output pixels, with its halo, in LDS once per 32-channel chunk and
// visits all taps on it.  There is one for dense 3x3 filters (igemm_halo3x3.hip) and two for dense 5x5 ones with few channels on
// one side (igemm_narrow5x5.hip).  Other filters stay with the ring kernels: a general halo-tile kernel (16 x 16 pixels x 256
// channels) lost to them on every one of 4703 dilated and 5x5 layers of 200..256 patches, 1.9x on average (forward and data gradient,
// fp16; least 1.04x: 2 x 147 x 160, 256 -> 304, 5x5, 244 against 236 us; 230 x 250, 32 -> 192, dilation 2: 1.8x).
//
// The filter is read from a re-laid-out copy [chunk][tap][output channel][32] (ragged chunk zero-filled), so that the filter
// tile of a step is one contiguous run spread evenly over the L2 channels.
#include "device_common.h"
#include "kernels.h"

namespace dlk {

// ---- eligibility (shared by the workspace query and the launch) ---------------
// tuning override: 0 = never
static bool halo_mode() { return tuning_knob("DLCONV_HALO", 1) != 0; }

static bool takes_3x3(const IgemmArgs &a)
{
    // 48..64 columns and a short reduction of whole chunks, or of half a chunk: one column tile, mostly set-up (and the filter
    // copy ahead of it), where the ring kernels take 0.6-0.98x the time (110592 pixels, 64 -> 64: 21.6 -> 15.3 us; 162936, 16 -> 64:
    // 23.8 -> 14.7).  With other channel counts either may be ahead (48..304 input channels and 64 columns: this kernel 0.7-1.5x as
    // fast), with how far the last chunk is filled and with the number of patches.
    if (a.Nout >= 48 && a.Nout <= 64 && (a.Cin <= 16 || a.Cin == 32 || a.Cin == 64)) return false;
    return igemm_halo3x3_applicable(a) && igemm_halo3x3_tiles(a) >= 200;
}

bool igemm_halo_takes(const IgemmArgs &a)
{
    return halo_mode() && a.Nout > 0 && (igemm_narrow5x5_applicable(a) || igemm_wide5x5_applicable(a) || takes_3x3(a));
}

size_t igemm_blocked_filter_bytes(const IgemmArgs &a)
{
    return (size_t)((a.Cin + BK - 1) / BK) * a.TR * a.TS * a.Nout * BK * sizeof(uint16_t);
}

hipError_t launch_igemm_halo(const IgemmArgs &a, bool is_bf16, hipStream_t stream)
{
    if (igemm_narrow5x5_applicable(a)) return launch_igemm_narrow5x5(a, is_bf16, stream);
    if (igemm_wide5x5_applicable(a)) return launch_igemm_wide5x5(a, is_bf16, stream);
    return launch_igemm_halo3x3(a, is_bf16, stream);
}

// ---- filter re-layout into [chunk][tap][row][32] --------------------------------
// dst[((chunk*NT + jr*TS + js)*Nrows + j)*32 + e] = src[base + j*sj + jr*sr + js*ss + (chunk*32+e)*sc],
// zero where chunk*32 + e >= Cin.
__global__ void filter_block_kernel(const FilterBlockArgs p)
{
    const int64_t total = (int64_t)((p.Cin + BK - 1) / BK) * p.TR * p.TS * p.Nrows * BK;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        int64_t r = i;
        const int e = (int)(r % BK); r /= BK;
        const int j = (int)(r % p.Nrows); r /= p.Nrows;
        const int js = (int)(r % p.TS); r /= p.TS;
        const int jr = (int)(r % p.TR); r /= p.TR;
        const int c = (int)r * BK + e;
        p.dst[i] = c < p.Cin ? p.src[p.base + (int64_t)j * p.sj + (int64_t)jr * p.sr + (int64_t)js * p.ss + (int64_t)c * p.sc]
                             : (uint16_t)0;
    }
}

hipError_t launch_filter_block(const FilterBlockArgs &a, hipStream_t stream)
{
    const int64_t total = (int64_t)((a.Cin + BK - 1) / BK) * a.TR * a.TS * a.Nrows * BK;
    if (total <= 0) return hipSuccess;
    const int blocks = (int)((total + 255) / 256 < 8192 ? (total + 255) / 256 : 8192);
    DLK_LAUNCH("filter_block_kernel", filter_block_kernel, dim3(blocks), dim3(256), 0, stream, a);
    return dlk::launch_status();
}

}  // namespace dlk
