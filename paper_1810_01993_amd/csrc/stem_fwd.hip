// Forward pass of a 7x7, stride-2, padding-3 convolution with 8 or 16 input channels (or a copy padded to that) and at most 64
// output channels (gfx950): the network's stem.
//
// In the general engine every tap fetches its own 32 or 16 bytes per pixel: 89 us for 768 x 1152 x 16 -> 64, batch 2, where
// the bytes take 20 us and the products 28.  Here a workgroup stays for all its 16 x 16 patches of output pixels.  The
// filter is laid out once, as MFMA fragments in registers (what does not fit, in LDS); the input patch with its halo (37 x 38
// pixels) is fetched into one of two LDS images while the other is multiplied.  51 us (0.87 PFLOP/s); of the 6 us a patch
// takes, 3 are products, the rest is the store and the wait of both waves of a SIMD for it.  With 8 channels 361 x 577 -> 64,
// batch 2: 24 -> 16 us.
//
// LDS image: planes [column parity][8-channel half][row][column / 2] of 16-byte slots.  The 16 output pixels of an MFMA
// operand read every other column, i.e. neighbouring slots of one plane: no bank conflicts, and every tap is a constant
// offset from the lane's first slot.  A 32-deep step covers, with 16 channels, two taps (columns s and s + 1 of a row, or
// column 6 of two rows): 25 steps; with 8 channels, four: 14 steps.  Lanes whose tap does not exist have their input cleared
// as well as their filter, so that an infinity next to the window does not reach the sum.
//
// Wave w multiplies 32 output channels (half w % HALVES) and some rows of the patch.  The filter rides in the first MFMA
// operand: a lane ends up with four consecutive channels of a pixel.
#include "device_common.h"
#include "kernels.h"

namespace dlk {

namespace {
constexpr int SF_R = 7, SF_PAD = 3, SF_T = 16;           // filter, padding, patch edge
constexpr int SF_ROWS = 2 * SF_T + SF_R - 2;             // 37 input rows
constexpr int SF_COLS2 = SF_T + 3;                       // column pairs: 38 input columns
constexpr int SF_PLANE = SF_ROWS * SF_COLS2;             // slots of a plane
}  // namespace

// CP: input channels (8 or 16).  HALVES: 32-channel halves of the output.
template <class T, int CP, int HALVES>
__global__ __launch_bounds__(512) void stem_fwd_kernel(const StemFwdArgs p)
{
    constexpr int NW = 8, NH = CP / 8, PLANES = 2 * NH;
    constexpr int NK = CP == 16 ? 25 : 14;               // steps
    constexpr int NREG = CP == 16 ? 13 : 14;             // of which the filter is in registers
    constexpr int RB = HALVES == 2 ? 4 : 2;              // patch rows per wave
    constexpr int PPW = (PLANES * SF_PLANE + NW * 64 - 1) / (NW * 64);         // 1 KB pieces of an image per wave
    constexpr int PIECES = PPW * NW, IMAGE = PIECES * 64 * 8;                  // elements
    constexpr int TAPS = SF_R * SF_R;
    constexpr int RAW = 32 * HALVES * TAPS * CP;         // the filter as [channel][tap][CP], before it is dealt out
    constexpr int FRAGS = (NK - NREG) * 2 * HALVES * 64 * 8;
    constexpr int EP = 40;                               // staging pitch of an output pixel: 32 channels and 16 bytes
    constexpr int STAGE = NW * RB * 16 * EP;
    constexpr bool OWN_STAGE = STAGE > IMAGE;            // else the output passes through the image just read
    // two images, filter fragments, staging area; at first the filter lies behind the first image
    constexpr int USED = 2 * IMAGE + FRAGS + (OWN_STAGE ? STAGE : 0);
    __shared__ __align__(16) uint16_t lds[USED > IMAGE + RAW ? USED : IMAGE + RAW];
    uint16_t *const sF = lds + 2 * IMAGE, *const raw = lds + IMAGE;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = HALVES == 2 ? wave & 1 : 0, rg = HALVES == 2 ? wave >> 1 : wave;
    const int ox = lane & 15, v = lane >> 4;

    const int tiles_x = (p.Q + SF_T - 1) / SF_T, tiles_y = (p.P + SF_T - 1) / SF_T;
    const int64_t tiles = (int64_t)p.N * tiles_x * tiles_y;
    const int wg = xcd_remap(blockIdx.x, gridDim.x);
    const int first = (int)(tiles * wg / gridDim.x), last = (int)(tiles * (wg + 1) / gridDim.x);

    // ---- the input patch ---------------------------------------------------------------
    const i32x4_t rsX = make_rsrc_words(p.x, (uint32_t)p.N * p.H * p.W * CP * 2u);
    // row, column and half of slot s
    auto slot_at = [&](int s, int &row, int &col, int &h) {
        const int plane = s / SF_PLANE, rem = s - plane * SF_PLANE;
        row = rem / SF_COLS2;
        col = 2 * (rem - row * SF_COLS2) + plane / NH;
        h = plane % NH;
        return plane < PLANES;
    };
    uint32_t at[PPW];                                    // row << 16 | column << 8 | half, or all ones
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
        int row, col, h;
        at[i] = slot_at((wave + i * NW) * 64 + lane, row, col, h) ? (uint32_t)(row << 16 | col << 8 | h) : ~0u;
    }
    auto place = [&](int tile, int &img, int &y0, int &x0) {
        const int tx = tile % tiles_x, rest = tile / tiles_x, ty = rest % tiles_y;
        img = rest / tiles_y;
        y0 = ty * SF_T;
        x0 = tx * SF_T;
    };
    auto fetch = [&](int tile, int buf) {
        int img, y0, x0;
        place(tile, img, y0, x0);
        const int iy0 = 2 * y0 - SF_PAD, ix0 = 2 * x0 - SF_PAD;
        const uint32_t dst = lds_addr(lds) + (uint32_t)buf * IMAGE * 2 + (uint32_t)wave * 1024;
#pragma unroll
        for (int i = 0; i < PPW; ++i) {
            const int iy = iy0 + (int)(at[i] >> 16), ix = ix0 + (int)(at[i] >> 8 & 255);
            const bool in = ((unsigned)iy < (unsigned)p.H) & ((unsigned)ix < (unsigned)p.W) & (at[i] != ~0u);
            const uint32_t off = (uint32_t)(((img * p.H + iy) * p.W + ix) * CP + 8 * (int)(at[i] & 255)) * 2u;
            dma_load_16B(rsX, dst + i * NW * 1024, in ? off : OOB_OFFSET);
        }
    };

    int buf = 0;
    if (first < last) fetch(first, 0);

    // ---- the filter: as it lies in LDS, zero rows behind the last channel, then as fragments --------------
    for (int i = tid; i < 32 * HALVES * TAPS; i += 512) {
        const int k = i / TAPS;
#pragma unroll
        for (int h = 0; h < NH; ++h)
            *reinterpret_cast<u32x4_t *>(raw + i * CP + 8 * h) = k < p.K ? *reinterpret_cast<const u32x4_t *>(p.w + (size_t)i * CP + 8 * h) : u32x4_t{0, 0, 0, 0};
    }
    __syncthreads();
    // tap of step q in this lane's slice, or -1
    auto tap_of = [&](int q) -> int {
        if constexpr (CP == 16) {
            if (q < 21) return q / 3 * SF_R + 2 * (q % 3) + (v >> 1);
            const int r = 2 * (q - 21) + (v >> 1);
            return r < SF_R ? r * SF_R + 6 : -1;
        } else {
            const int s = 4 * (q & 1) + v;
            return s < SF_R ? (q >> 1) * SF_R + s : -1;
        }
    };
    u32x4_t fw[NREG][2];
    {
        u32x4_t rest[NK > NREG ? NK - NREG : 1][2];
#pragma unroll
        for (int q = 0; q < NK; ++q)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int tap = tap_of(q), k = half * 32 + b * 16 + ox;
                u32x4_t f{0, 0, 0, 0};
                if (tap >= 0) f = *reinterpret_cast<const u32x4_t *>(raw + (k * TAPS + tap) * CP + (CP == 16 ? 8 * (v & 1) : 0));
                if (q < NREG) fw[q < NREG ? q : 0][b] = f;
                else rest[q < NREG ? 0 : q - NREG][b] = f;
            }
        __syncthreads();                                 // the filter has been read
        if (rg == 0) {
#pragma unroll
            for (int q = NREG; q < NK; ++q)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    *reinterpret_cast<u32x4_t *>(sF + (((q - NREG) * HALVES + half) * 2 + b) * 512 + lane * 8) = rest[q < NREG ? 0 : q - NREG][b];
        }
    }

    // this lane's first slot in an image (elements): column pairs of a row, and (16 channels) column 6 of row pairs
    int base1, base2;
    if constexpr (CP == 16) {
        base1 = (((v >> 1) * NH + (v & 1)) * SF_PLANE + ox) * 8;
        base2 = ((v & 1) * SF_PLANE + (v >> 1) * SF_COLS2 + ox + 3) * 8;
    } else {
        base1 = ((v & 1) * SF_PLANE + (v >> 1) + ox) * 8;
        base2 = 0;
    }
    const int base3 = ((v & 1) * SF_PLANE + ox + 3) * 8;                       // step 24: row 6 alone
    const uint32_t keep = (CP == 16 ? v < 2 : v < 3) ? ~0u : 0u;               // lanes of a step's last, missing tap

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    for (int tile = first; tile < last; ++tile, buf ^= 1) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");             // this patch is there, nobody reads the other image
        if (tile + 1 < last) fetch(tile + 1, buf ^ 1);
        const uint16_t *const image = lds + buf * IMAGE;
        floatx4_t acc[RB][2];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[i][b] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        const uint16_t *const rows = image + 2 * rg * RB * SF_COLS2 * 8;
        // fragments of step q: the lanes' input of RB patch rows, and the filter where it is not in registers
        u32x4_t fa[2][RB], fl[2][2];
        auto read = [&](int q) __attribute__((always_inline)) {
            int off;                                     // constant but for the lane's base
            if constexpr (CP == 16)
                off = q < 21 ? base1 + (q / 3 * SF_COLS2 + q % 3) * 8 : q < 24 ? base2 + 2 * (q - 21) * SF_COLS2 * 8 : base3 + 6 * SF_COLS2 * 8;
            else
                off = base1 + ((q >> 1) * SF_COLS2 + 2 * (q & 1)) * 8;
#pragma unroll
            for (int i = 0; i < RB; ++i) fa[q & 1][i] = *reinterpret_cast<const u32x4_t *>(rows + off + 2 * i * SF_COLS2 * 8);
            if (q >= NREG) {
#pragma unroll
                for (int b = 0; b < 2; ++b) fl[q & 1][b] = *reinterpret_cast<const u32x4_t *>(sF + (((q - NREG) * HALVES + half) * 2 + b) * 512 + lane * 8);
            }
        };
        read(0);
        // The products are issued in this order (mfma16_acc), each step's fragments requested one step ahead: left to the
        // compiler's scheduler the reads came just before their use.
#pragma unroll
        for (int q = 0; q < NK; ++q) {
            if (q + 1 < NK) read(q + 1);
            __builtin_amdgcn_sched_barrier(0);
            if (CP == 16 ? q == 24 : q & 1) {            // a tap is missing
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) fa[q & 1][i][e] &= keep;
            }
            if (q == 0 || (CP == 16 ? q == 24 : q & 1)) asm volatile("s_nop 3" ::: "memory");      // vector writes ahead of an MFMA that the compiler does not see
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b) T::mfma16_acc(acc[i][b], q < NREG ? fw[q < NREG ? q : 0][b] : fl[q & 1][b], fa[q & 1][i]);      // rows = output channels
            __builtin_amdgcn_sched_barrier(0);
        }
        mfma_acc_settle();
        // the next patch has landed before the stores are issued, so that nothing waits for these until then
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // ---- store: rounded, rows of 16 pixels x 32 channels at a time, through an area of the wave's own -------
        int img, y0, x0;
        place(tile, img, y0, x0);
        if constexpr (!OWN_STAGE) __syncthreads();       // everyone has read this image
        uint16_t *const stg = (OWN_STAGE ? lds + 2 * IMAGE + FRAGS : lds + buf * IMAGE) + wave * RB * 16 * EP;
        const bool tail = p.bias != nullptr || p.relu != 0;
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                floatx4_t c = acc[i][b];
                const int ch = b * 16 + 4 * v;
                if (tail && half * 32 + ch < p.K) c = apply_tail4(c, p.bias, p.relu, half * 32 + ch, p.K);
                *reinterpret_cast<u32x2_t *>(stg + (i * 16 + ox) * EP + ch) = u32x2_t{T::pack2(c[0], c[1]), T::pack2(c[2], c[3])};
            }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int px = lane >> 2, c8 = (lane & 3) * 8, y = y0 + rg * RB + i, x = x0 + px, k = half * 32 + c8;
            const u32x4_t d = *reinterpret_cast<const u32x4_t *>(stg + (i * 16 + px) * EP + c8);
            if (y < p.P && x < p.Q && k < p.K) *reinterpret_cast<u32x4_t *>(p.y + ((size_t)(img * p.P + y) * p.Q + x) * p.K + k) = d;
        }
    }
}

bool stem_fwd_applicable(int C, int K, int R, int S, int sh, int sw, int ph, int pw, int dh, int dw)
{
    return R == SF_R && S == SF_R && sh == 2 && sw == 2 && ph == SF_PAD && pw == SF_PAD && dh == 1 && dw == 1 && (C == 8 || C == 16) && K % 8 == 0 && K <= 64;
}

template <class T>
static hipError_t launch_stem(const StemFwdArgs &a, hipStream_t stream)
{
    const int64_t tiles = (int64_t)a.N * ((a.P + SF_T - 1) / SF_T) * ((a.Q + SF_T - 1) / SF_T);
    if (tiles <= 0 || tiles > 0x7fffffff || (a.C != 8 && a.C != 16) || a.K > 64 || a.K % 8 != 0) return hipErrorInvalidValue;
    if (a.P != (a.H - 1) / 2 + 1 || a.Q != (a.W - 1) / 2 + 1) return hipErrorInvalidValue;
    // one workgroup per compute unit, each with as many patches as any other or one fewer
    const dim3 grid((unsigned)(tiles < 256 ? tiles : 256)), block(512);
    if (a.C == 16) {
        if (a.K > 32) DLK_LAUNCH("stem_fwd_kernel<16>", (stem_fwd_kernel<T, 16, 2>), grid, block, 0, stream, a);
        else DLK_LAUNCH("stem_fwd_kernel<16>", (stem_fwd_kernel<T, 16, 1>), grid, block, 0, stream, a);
    } else {
        if (a.K > 32) DLK_LAUNCH("stem_fwd_kernel<8>", (stem_fwd_kernel<T, 8, 2>), grid, block, 0, stream, a);
        else DLK_LAUNCH("stem_fwd_kernel<8>", (stem_fwd_kernel<T, 8, 1>), grid, block, 0, stream, a);
    }
    return dlk::launch_status();
}

hipError_t launch_stem_fwd(const StemFwdArgs &a, bool is_bf16, hipStream_t stream)
{
    return is_bf16 ? launch_stem<BF16>(a, stream) : launch_stem<F16>(a, stream);
}

}  // namespace dlk
