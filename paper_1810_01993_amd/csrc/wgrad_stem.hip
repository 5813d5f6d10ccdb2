// Filter gradient of a 7x7, stride-2, padding-3 convolution with 8 or 16 input channels (or a copy padded to that) and at most
// 64 output channels (gfx950): the network's stem.
//
// In the general kernel every tap is columns of its own, so each pixel of x is fetched up to 13 times in pieces of 16 channels,
// and transposed LDS reads feed tiles that are mostly one operand: 88 us for 768 x 1152 x 16 -> 64, batch 2 (products 28 us).
// Here a workgroup stays for a run of 16 x 16 patches of output pixels and keeps the sums of all 49 taps x 32 output channels
// in registers: 8 waves, each with up to 7 blocks of 16 columns (a tap of 16 channels, or two of 8) times two of 16 output
// channels.  Per patch it fetches x with its halo (37 x 38 pixels) and its 32 channels of dy into one of two LDS buffers while the
// other is multiplied.  Two workgroups share a patch (the two halves of the output channels), which halves the fp32
// partial sums that one workgroup per compute unit leaves for the ordered reduce (25 MB instead of 51).  With that reduce the
// pass takes 69 us where it took 94.
//
// The reduction index of an MFMA (16x16x32) is two rows of 16 output pixels.  x lies in planes [column parity][8-channel half]
// [row][column / 2] of 16-byte slots, so the pixels of a row that a tap meets are neighbouring slots; a tap is a constant
// offset.  Both operands are read with ds_read_b64_tr_b16; the plane pitch (4 slots more than a multiple of 16) and the
// exchange of dy's 32-byte blocks keep the eight pieces of a half-wave on different banks.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace dlk {

namespace {
constexpr int SW_R = 7, SW_PAD = 3, SW_T = 16;           // filter, padding, patch edge
constexpr int SW_ROWS = 2 * SW_T + SW_R - 2;             // 37 input rows
constexpr int SW_COLS2 = SW_T + 3;                       // column pairs: 38 input columns
constexpr int SW_PLANE = 708;                            // slots from plane to plane: 37 * 19 = 703, and 708 % 16 == 4
static_assert(SW_ROWS * SW_COLS2 <= SW_PLANE && SW_PLANE % 16 == 4, "plane pitch");
typedef short sw_s16x4_t __attribute__((ext_vector_type(4)));
// which 32-byte block of its 64-byte row holds logical block b of output pixel px (0 .. 255 of the patch)
__device__ __forceinline__ int sw_block(int b, int px) { return b ^ ((px >> 3) & 1); }
}  // namespace

// CP: input channels (8 or 16)
template <class T, int CP>
__global__ __launch_bounds__(512) void wgrad_stem_kernel(const WgradStemArgs p)
{
    constexpr int NW = 8, PLANES = CP / 4;               // parities x halves
    constexpr int NB = CP == 16 ? 49 : 28;               // blocks of 16 columns: a tap, or two neighbouring taps (the last of a row alone)
    constexpr int NBW = (NB + NW - 1) / NW;              // per wave: 7 or 4
    constexpr int XP = (PLANES * SW_PLANE + 63) / 64;    // 1 KB pieces
    constexpr int XI = (XP + NW - 1) / NW, DI = 16 / NW; // per wave; dy: 256 pixels x 64 bytes
    constexpr int X_ELEMS = XI * NW * 512, D_ELEMS = 256 * 32, BUF = X_ELEMS + D_ELEMS;
    __shared__ __align__(16) uint16_t lds[2 * BUF];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_x = (p.Q + SW_T - 1) / SW_T, tiles_y = (p.P + SW_T - 1) / SW_T;
    const int64_t tiles = (int64_t)p.N * tiles_x * tiles_y;
    const int halves = (p.K + 31) / 32;
    const int id = xcd_remap(blockIdx.x, gridDim.x);
    const int run = id / halves, k0 = (id - run * halves) * 32;
    const int first = (int)(tiles * run / p.splits), last = (int)(tiles * (run + 1) / p.splits);

    const i32x4_t rsX = make_rsrc_words(p.x, (uint32_t)p.N * p.H * p.W * CP * 2u);
    const i32x4_t rsD = make_rsrc_words(p.dy, (uint32_t)p.N * p.P * p.Q * p.K * 2u);

    // ---- what this lane fetches ---------------------------------------------------
    uint32_t at[XI];                                     // row << 16 | column << 8 | half of a slot of x, or all ones
#pragma unroll
    for (int i = 0; i < XI; ++i) {
        const int s = (wave + i * NW) * 64 + lane, plane = s / SW_PLANE, rem = s - plane * SW_PLANE;
        const int row = rem / SW_COLS2, c2 = rem - row * SW_COLS2;
        const int parity = CP == 16 ? plane >> 1 : plane, h = CP == 16 ? plane & 1 : 0;
        at[i] = plane < PLANES && row < SW_ROWS ? (uint32_t)(row << 16 | (2 * c2 + parity) << 8 | h) : ~0u;
    }
    auto place = [&](int tile, int &img, int &y0, int &x0) {
        const int tx = tile % tiles_x, rest = tile / tiles_x, ty = rest % tiles_y;
        img = rest / tiles_y;
        y0 = ty * SW_T;
        x0 = tx * SW_T;
    };
    auto fetch = [&](int tile, int buf) __attribute__((always_inline)) {
        int img, y0, x0;
        place(tile, img, y0, x0);
        const int iy0 = 2 * y0 - SW_PAD, ix0 = 2 * x0 - SW_PAD;
        const uint32_t dst = lds_addr(lds) + (uint32_t)buf * BUF * 2 + (uint32_t)wave * 1024;
#pragma unroll
        for (int i = 0; i < XI; ++i) {
            const int iy = iy0 + (int)(at[i] >> 16), ix = ix0 + (int)(at[i] >> 8 & 255);
            const bool in = ((unsigned)iy < (unsigned)p.H) & ((unsigned)ix < (unsigned)p.W) & (at[i] != ~0u);
            const uint32_t off = (uint32_t)(((img * p.H + iy) * p.W + ix) * CP + 8 * (int)(at[i] & 255)) * 2u;
            dma_load_16B(rsX, dst + i * NW * 1024, in ? off : OOB_OFFSET);
        }
#pragma unroll
        for (int i = 0; i < DI; ++i) {                   // a piece: 16 pixels of one patch row
            const int row = wave + i * NW, px = row * SW_T + (lane >> 2), oy = y0 + row, ox = x0 + (lane >> 2);
            const int k = k0 + sw_block((lane & 3) >> 1, px) * 16 + (lane & 1) * 8;
            const bool in = (oy < p.P) & (ox < p.Q) & (k < p.K);
            const uint32_t off = (uint32_t)(((img * p.P + oy) * p.Q + ox) * p.K + k) * 2u;
            dma_load_16B(rsD, dst + X_ELEMS * 2 + i * NW * 1024, in ? off : OOB_OFFSET);
        }
    };

    // ---- fragment addresses (elements) ------------------------------------------------
    // lane = 16 g + 4 j + m points at pixel 8 (g & 1) + j (+ 4) of row g >> 1 of the step and at quad m of 16 channels
    const int g = lane >> 4, j = lane >> 2 & 3, m = lane & 3;
    const int xlane = ((m >> 1) * SW_PLANE + 2 * (g >> 1) * SW_COLS2 + 8 * (g & 1) + j) * 8 + (m & 1) * 4;
    int xoff[NBW];
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
        const int blk = min(wave * NBW + b, NB - 1);
        const int r = CP == 16 ? blk / 7 : blk >> 2, s = CP == 16 ? blk % 7 : 2 * (blk & 3);
        xoff[b] = xlane + ((CP == 16 ? (s & 1) * 2 * SW_PLANE : 0) + r * SW_COLS2 + (s >> 1)) * 8;
    }
    const int dpx = (g >> 1) * SW_T + 8 * (g & 1) + j;   // pixel of the step (and + 4)
    int doff[2][2];                                      // [16-channel block][pixels + 0, + 4]
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int t = 0; t < 2; ++t) doff[b][t] = X_ELEMS + (dpx + 4 * t) * 32 + sw_block(b, dpx + 4 * t) * 16 + m * 4;
    auto tr = [&](const uint16_t *q) __attribute__((always_inline)) {
        return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((sw_s16x4_t __attribute__((address_space(3))) *)q));
    };

    floatx4_t acc[NBW][2];
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[b][h] = floatx4_t{0.f, 0.f, 0.f, 0.f};

    if (first < last) fetch(first, 0);
    for (int tile = first, buf = 0; tile < last; ++tile, buf ^= 1) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");     // this patch is there, nobody reads the other buffer
        if (tile + 1 < last) fetch(tile + 1, buf ^ 1);
        const uint16_t *const at_buf = lds + buf * BUF;
        int img, y0, x0;
        place(tile, img, y0, x0);
        // Pixels behind the image's edge: dy is zero there, but x need not be (a neighbour's window reaches it), and an infinity
        // times zero is not.  In such patches x is cleared too.
        const bool ragged = x0 + SW_T > p.Q || y0 + SW_T > p.P;
        const int cols = p.Q - x0 - 8 * (g & 1);             // of this lane's eight pixels of a row
        u32x4_t fx[2][NBW], fd[2][2];
        auto read = [&](int step) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const u32x2_t lo = tr(at_buf + doff[b][0] + step * 2 * SW_T * 32), hi = tr(at_buf + doff[b][1] + step * 2 * SW_T * 32);
                fd[step & 1][b] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
            }
#pragma unroll
            for (int b = 0; b < NBW; ++b) {
                const uint16_t *const q = at_buf + xoff[b] + step * 4 * SW_COLS2 * 8;
                const u32x2_t lo = tr(q), hi = tr(q + 4 * 8);
                fx[step & 1][b] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
            }
        };
        read(0);
#pragma unroll
        for (int step = 0; step < SW_T / 2; ++step) {
            if (step + 1 < SW_T / 2) read(step + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (ragged) {                                // uniform
                const int n = y0 + 2 * step + (g >> 1) < p.P ? cols : 0;
#pragma unroll
                for (int b = 0; b < NBW; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) fx[step & 1][b][e] &= n >= 2 * e + 2 ? ~0u : n == 2 * e + 1 ? 0xffffu : 0u;
            }
            asm volatile("s_nop 3" ::: "memory");        // vector writes ahead of MFMAs that the compiler does not see
#pragma unroll
            for (int b = 0; b < NBW; ++b)
#pragma unroll
                for (int h = 0; h < 2; ++h) T::mfma16_acc(acc[b][h], fd[step & 1][h], fx[step & 1][b]);       // rows = output channels
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    mfma_acc_settle();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    float *const out = p.partial + (size_t)run * p.K * SW_R * SW_R * CP;
#pragma unroll
    for (int b = 0; b < NBW; ++b) {
        const int blk = wave * NBW + b;
        if (blk >= NB) continue;
        const int r = CP == 16 ? blk / 7 : blk >> 2, s = CP == 16 ? blk % 7 : 2 * (blk & 3) + ((lane & 15) >> 3), c = lane & (CP - 1);
        if (s >= SW_R) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + 16 * h + 4 * g + e;
                if (k < p.K) out[((size_t)k * SW_R * SW_R + r * SW_R + s) * CP + c] = acc[b][h][e];
            }
    }
}

bool wgrad_stem_applicable(int C, int K, int R, int S, int sh, int sw, int ph, int pw, int dh, int dw)
{
    return R == SW_R && S == SW_R && sh == 2 && sw == 2 && ph == SW_PAD && pw == SW_PAD && dh == 1 && dw == 1 && (C == 8 || C == 16) && K % 8 == 0 && K <= 64;
}

// Runs of patches (slices of partial sums): one workgroup per compute unit and half of the output channels.
int wgrad_stem_splits(int N, int K, int P, int Q)
{
    const int64_t tiles = (int64_t)N * ((P + SW_T - 1) / SW_T) * ((Q + SW_T - 1) / SW_T);
    return (int)std::min<int64_t>(tiles, 256 / ((K + 31) / 32));
}

hipError_t launch_wgrad_stem(const WgradStemArgs &a, bool is_bf16, hipStream_t stream)
{
    if ((a.C != 8 && a.C != 16) || a.K > 64 || a.K % 8 != 0 || a.splits < 1) return hipErrorInvalidValue;
    if (a.P != (a.H - 1) / 2 + 1 || a.Q != (a.W - 1) / 2 + 1) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(a.splits * ((a.K + 31) / 32))), block(512);
    if (a.C == 16) {
        if (is_bf16) DLK_LAUNCH("wgrad_stem_kernel<16>", (wgrad_stem_kernel<BF16, 16>), grid, block, 0, stream, a);
        else DLK_LAUNCH("wgrad_stem_kernel<16>", (wgrad_stem_kernel<F16, 16>), grid, block, 0, stream, a);
    } else {
        if (is_bf16) DLK_LAUNCH("wgrad_stem_kernel<8>", (wgrad_stem_kernel<BF16, 8>), grid, block, 0, stream, a);
        else DLK_LAUNCH("wgrad_stem_kernel<8>", (wgrad_stem_kernel<F16, 8>), grid, block, 0, stream, a);
    }
    return dlk::launch_status();
}

}  // namespace dlk
