// Filter-gradient kernel, direct-to-LDS variant (gfx950).
//
// GEMM view: rows = output channel k, columns j = (r*S + s)*C + c, reduction
// over the N*P*Q output pixels.  Both operands are channel-contiguous in
// memory (NHWC), i.e. the reduction index is their slow axis.  Tiles are
// therefore deposited in LDS as they lie in memory, [pixel][channel], by
// `buffer_load_dwordx4 ... lds` (zero for padding pixels, ragged edges and
// pixels past the end of the slice), and the MFMA fragments -- 8 consecutive
// pixels of one channel per lane -- are produced by the LDS transpose read
// ds_read_b64_tr_b16: within a group of 16 lanes, lane i receives element
// (i % 4) of the 64-bit words addressed by lanes 4j + i/4, j = 0..3.  Pointing
// lane s at pixel s/4, channels 4*(s%4)..+3 of a 4-pixel x 16-channel block
// hands lane i the 4 pixels of channel i.
//
// The pixel range is cut into `splits` slices; every slice writes an fp32
// partial tile and a second kernel adds the slices in a fixed order.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "kernels.h"

namespace dlk {

typedef short s16x4_t __attribute__((ext_vector_type(4)));

// LDS image of a tile: row = pixel (BX channels = 2*BX bytes), and within a
// row the 32-byte block b (16 channels) sits at block b ^ (2 * (pixel & 3))
// (b ^ (pixel & 3) for rows of only four blocks).  Half a wave (the unit a
// 64-bit LDS read serves per cycle) touches four pixel rows x two adjacent
// blocks; rows are a multiple of the 256-byte bank width apart, and the rule
// puts those eight 32-byte pieces on eight different bank ranges.
__device__ __host__ constexpr int swz_shift(int BX) { return BX >= 128 ? 1 : 0; }
// KB: pixels of a step.  LINEAR: 1x1, unit stride, no padding, so x is read like dy.  PP: two groups of waves half a step apart.
template <class T, int BM, int BN, int WM, int WN, int KB, int STAGES, bool PP, bool LINEAR>
__global__ __launch_bounds__(WM *WN * 64) void wgrad_dma_kernel(const WgradArgs p)
{
    constexpr int NW = WM * WN;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int LPR_A = BM / 8, LPR_B = BN / 8;          // lanes (16-byte chunks) per pixel row
    constexpr int PPI_A = 64 / LPR_A, PPI_B = 64 / LPR_B;  // pixel rows per load instruction
    constexpr int AIW = KB / PPI_A / NW, BIW = KB / PPI_B / NW;   // load instructions per wave per step
    static_assert(BM >= 64 && BN >= 64 && BM <= 512 && BN <= 512, "a row must be 4..32 chunks of 32 bytes");
    static_assert((KB / PPI_A) % NW == 0 && (KB / PPI_B) % NW == 0, "every wave must issue the same number of loads");
    static_assert(AIW >= 1 && BIW >= 1 && TM >= 1 && TN >= 1, "tile too small for this many waves");
    static_assert(STAGES == 3 || STAGES == 4, "ring of 3 or 4 LDS buffers");
    static_assert(!PP || NW == 8, "one wave of each group per SIMD");
    constexpr int IN_FLIGHT = (STAGES - 2) * (AIW + BIW);

    __shared__ __align__(16) uint16_t lds[STAGES * KB * (BM + BN)];
    auto slot_a = [&](int s) { return lds + s * KB * BM; };
    auto slot_b = [&](int s) { return lds + STAGES * KB * BM + s * KB * BN; };

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    const int RSC = p.R * p.S * p.C;
    const int npix = p.N * p.P * p.Q;
    const int tiles_n = (RSC + BN - 1) / BN;
    const int tiles = tiles_n * ((p.K + BM - 1) / BM);
    // Workgroups are dealt to the 8 XCDs round-robin by id.  All tiles of one
    // pixel slice are given to the same XCD, back to back, so that the slice of
    // dy and x they all read is fetched into that XCD's L2 once.
    // With few slices (small images with large filters) that would leave XCDs idle: then
    // consecutive ids take consecutive tiles of a slice, i.e. every slice runs on all XCDs.
    const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int tile = p.spread ? (int)(blockIdx.x % tiles) : slot % tiles;
    const int split = p.spread ? (int)(blockIdx.x / tiles) : (slot / tiles) * 8 + xcd;
    if (split >= p.splits) return;                         // uniform for the whole workgroup
    const int k0 = (tile / tiles_n) * BM, j0 = (tile % tiles_n) * BN;
    const int pix_begin = split * p.chunk;
    const int pix_end = min(npix, pix_begin + p.chunk);

    const i32x4_t rsA = make_rsrc_words(p.dy, (uint32_t)npix * p.K * 2u);
    const i32x4_t rsB = make_rsrc_words(p.x, (uint32_t)p.N * p.H * p.W * p.C * 2u);

    // ---- what this lane fetches --------------------------------------------
    // A (dy): instruction `inst` covers pixel rows inst*PPI_A .. +PPI_A-1 of the step
    const int a_prow = lane / LPR_A;                        // pixel row within an instruction
    const int a_pchunk = lane % LPR_A;                      // physical 16-byte chunk within the row
    // pixel & 3 is the same for all of this lane's instructions (see static_asserts on NW / PPI)
    const int a_pix3 = ((wave * PPI_A) + a_prow) & 3;
    const int a_ch = k0 + ((((a_pchunk >> 1) ^ (a_pix3 << swz_shift(BM))) << 1) | (a_pchunk & 1)) * 8;

    const int b_prow = lane / LPR_B, b_pchunk = lane % LPR_B;
    const int b_pix3 = ((wave * PPI_B) + b_prow) & 3;
    const int b_col = j0 + ((((b_pchunk >> 1) ^ (b_pix3 << swz_shift(BN))) << 1) | (b_pchunk & 1)) * 8;
    const int b_tap = LINEAR ? 0 : b_col / p.C, b_c = b_col - b_tap * p.C;
    const int b_r = b_tap / p.S, b_s = b_tap - b_r * p.S;
    const int b_dh = b_r * p.dh - p.ph, b_dw = b_s * p.dw - p.pw;
    static_assert((NW * PPI_A) % 4 == 0 && (NW * PPI_B) % 4 == 0, "swizzle must not depend on the instruction index");

    // Byte offsets and the pixels they stand for run along with the steps: what lies outside is or-ed with OOB_OFFSET, the
    // pixel's place in x moves by additions and masks; decoding it from the pixel number, or carrying row by row, is a chain that
    // a wave walks between two barriers.  Against a walk with a loop of carries 8507 random layers ran 1.12x as fast on average
    // (6912 pixels, 2048 -> 256, 3x3: 83 -> 75 us; 2 x 192 x 288 outputs, 256 -> 256, stride 2: 161 -> 148).
    const uint32_t a_bad = a_ch < p.K ? 0u : OOB_OFFSET, b_bad = b_col < RSC ? 0u : OOB_OFFSET;
    uint32_t a_off[AIW], b_off[BIW];
    // (load i of a lane is pixel tid / LPR + i * NW * PPI of the step)
#pragma unroll
    for (int i = 0; i < AIW; ++i) {
        const int pix = pix_begin + tid / LPR_A + i * NW * PPI_A;
        a_off[i] = (uint32_t)(pix * p.K + a_ch) * 2u;
    }
    int b_ih[BIW], b_iw[BIW];                               // input pixel of the tap
#pragma unroll
    for (int i = 0; i < BIW; ++i) {
        const int pix = pix_begin + tid / LPR_B + i * NW * PPI_B;
        if constexpr (LINEAR) b_off[i] = (uint32_t)(pix * p.C + b_c) * 2u;
        else {
            const int n = pix / (p.P * p.Q), rem = pix - n * (p.P * p.Q), oh = rem / p.Q;
            b_ih[i] = oh * p.sh + b_dh;
            b_iw[i] = (rem - oh * p.Q) * p.sw + b_dw;
            b_off[i] = (uint32_t)(((n * p.H + b_ih[i]) * p.W + b_iw[i]) * p.C + b_c) * 2u;
        }
    }
    // The pixels of a step as whole images, rows of an image and columns of a row: rows and columns each carry at most once, and
    // nothing grows with the step times the stride.  The offsets are sums modulo 2^32 whose last value fits; coordinates stay
    // below 2^31 (launch_cfg).
    const int step_rows = __builtin_amdgcn_readfirstlane(KB / p.Q), step_n = __builtin_amdgcn_readfirstlane(step_rows / p.P);
    const int step_ih = (step_rows - step_n * p.P) * p.sh, step_iw = (KB - step_rows * p.Q) * p.sw;
    const uint32_t a_step = (uint32_t)(KB * p.K) * 2u;
    const uint32_t b_step = LINEAR ? (uint32_t)(KB * p.C) * 2u : (((uint32_t)step_n * p.H + step_ih) * p.W + step_iw) * p.C * 2u;
    const int row_iw = p.Q * p.sw, col_ih = p.P * p.sh;     // extents of the walk in x
    const int iw_end = row_iw + b_dw, ih_end = col_ih + b_dh;
    const uint32_t wrap_w = ((uint32_t)p.sh * p.W - row_iw) * p.C * 2u, wrap_h = ((uint32_t)p.H - col_ih) * p.W * p.C * 2u;
    int pix_left = pix_end - pix_begin;                     // pixels from the first of the step to be issued (uniform)

    const uint32_t dst0 = lds_addr(lds) + (uint32_t)wave * 1024;
    auto issue = [&](int s) __attribute__((always_inline)) {
        const uint32_t sa = dst0 + s * KB * BM * 2, sb = dst0 + (STAGES * KB * BM + s * KB * BN) * 2;
        const bool whole = pix_left >= KB;                  // else some pixels of the step lie behind the slice
#pragma unroll
        for (int i = 0; i < AIW; ++i) {
            uint32_t off = a_off[i] | a_bad;
            if (!whole && tid >= (pix_left - i * NW * PPI_A) * LPR_A) off = OOB_OFFSET;
            dma_load_16B(rsA, sa + i * NW * 1024, off);
            a_off[i] += a_step;
        }
#pragma unroll
        for (int i = 0; i < BIW; ++i) {
            uint32_t off = b_off[i] | b_bad;
            if (!whole && tid >= (pix_left - i * NW * PPI_B) * LPR_B) off = OOB_OFFSET;
            if constexpr (!LINEAR)
                if ((unsigned)b_ih[i] >= (unsigned)p.H || (unsigned)b_iw[i] >= (unsigned)p.W) off = OOB_OFFSET;
            dma_load_16B(rsB, sb + i * NW * 1024, off);
            if constexpr (LINEAR) b_off[i] += b_step;
            else {
                b_iw[i] += step_iw;
                b_ih[i] += step_ih;
                b_off[i] += b_step;
                // (all ones or zero, kept as such: as selects the six uniform values would each hold a register of every lane)
                uint32_t carry = b_iw[i] >= iw_end ? ~0u : 0u;
                asm("" : "+v"(carry));
                b_iw[i] -= carry & row_iw;
                b_off[i] += carry & wrap_w;
                b_ih[i] += carry & p.sh;
                uint32_t next = b_ih[i] >= ih_end ? ~0u : 0u;
                asm("" : "+v"(next));
                b_ih[i] -= next & col_ih;
                b_off[i] += next & wrap_h;
            }
        }
        pix_left -= KB;
    };

    floatx16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // ---- fragment addressing for the transpose reads ------------------------
    // lane = 16*g + s.  As a source it points at pixel 8*(g>>1) + 4*t + s/4 (t = 0, 1: the two
    // halves of its 8-pixel slice) and channels 16*(g&1) + 4*(s%4)..+3 of a 32-channel MFMA tile.
    const int g = lane >> 4, s16 = lane & 15;
    const int f_pix = 8 * (g >> 1) + (s16 >> 2);            // + 4*t + 16*ks
    const int f_ch = 16 * (g & 1);                          // block-aligned part of the channel
    const int f_sub = 4 * (s16 & 3);                        // channel within the 16-channel block
    // element offset of (pixel, 32-channel tile `ct`, this lane) in a [KB][BX] tile
    auto frag_off = [&](int BX, int pix, int ch_tile0) {
        const int ch = ch_tile0 + f_ch;
        const int blk = (ch >> 4) ^ ((pix & 3) << swz_shift(BX));
        return pix * BX + blk * 16 + f_sub;
    };
    auto read_frag = [&](const uint16_t *tile, int BX, int ks, int ch_tile0) {
        const int p0 = 16 * ks + f_pix;
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (s16x4_t __attribute__((address_space(3))) *)(tile + frag_off(BX, p0, ch_tile0)));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (s16x4_t __attribute__((address_space(3))) *)(tile + frag_off(BX, p0 + 4, ch_tile0)));
        u32x4_t r;
        const u32x2_t l2 = __builtin_bit_cast(u32x2_t, lo), h2 = __builtin_bit_cast(u32x2_t, hi);
        r[0] = l2[0]; r[1] = l2[1]; r[2] = h2[0]; r[3] = h2[1];
        return r;
    };
    constexpr int KS = KB / 16;
    auto wait_and_sync = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(IN_FLIGHT) : "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // fragments of slot u, loads of a later step into slot `next`, products; PP: the hand-over to the other group of waves in
    // between (the ring's guarantees are those of igemm_dma_tile.h)
    auto step = [&](int u, int next) __attribute__((always_inline)) {
        u32x4_t a[KS][TM], b[KS][TN];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int i = 0; i < TM; ++i) a[ks][i] = read_frag(slot_a(u), BM, ks, (wm * TM + i) * 32);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[ks][j] = read_frag(slot_b(u), BN, ks, (wn * TN + j) * 32);
        }
        __builtin_amdgcn_sched_barrier(0);
        issue(next);
        if constexpr (PP) wait_and_sync();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = T::mfma(a[ks][i], b[ks][j], acc[i][j]);
    };

    // The step count is rounded up to a whole turn of the ring (the extra
    // steps load and multiply zeros) so that the unrolled loop has one exit.
    const int nk = pix_end > pix_begin ? (pix_end - pix_begin + KB - 1) / KB : 0;
    const int nturns = (nk + STAGES - 1) / STAGES;
    if (nk > 0) {
#pragma unroll
        for (int u = 0; u < STAGES - 1; ++u) issue(u);
        const bool late = PP && wave >= NW / 2;
        if (late) wait_and_sync();
        for (int turn = 0; turn < nturns; ++turn) {
#pragma unroll
            for (int u = 0; u < STAGES; ++u) {
                wait_and_sync();
                step(u, (u + STAGES - 1) % STAGES);
            }
        }
        if (PP && !late) wait_and_sync();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }

    float *out = p.partial + (size_t)split * p.K * RSC;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int k = k0 + (wm * TM + i) * 32 + acc_row(v, lane);
            if (k >= p.K) continue;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = j0 + (wn * TN + j) * 32 + (lane & 31);
                if (col < RSC) out[(size_t)k * RSC + col] = acc[i][j][v];
            }
        }
}

template <class T, int BM, int BN, int WM, int WN, int KB, int STAGES, bool PP = false>
static hipError_t launch_cfg(const WgradArgs &args, hipStream_t stream)
{
    WgradArgs a = args;
    // the stride of an axis with one output position moves nothing, and may be too large to calculate with
    if (a.P == 1) a.sh = 1;
    if (a.Q == 1) a.sw = 1;
    const int RSC = a.R * a.S * a.C;
    const int64_t tiles = (int64_t)((a.K + BM - 1) / BM) * ((RSC + BN - 1) / BN);
    const int64_t split_groups = (a.splits + 7) / 8;        // each XCD takes every 8th slice
    const int64_t blocks = a.spread ? tiles * a.splits : tiles * split_groups * 8;
    if (blocks <= 0 || blocks > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(WM * WN * 64);
    const bool linear = a.R * a.S == 1 && args.sh == 1 && args.sw == 1 && a.ph == 0 && a.pw == 0;
    const auto label = [&]() { return kname("wgrad_dma_kernel", {BM, BN}) + (KB == 64 ? ".k64" : "") + (linear ? ".linear" : ""); };
    if (linear) DLK_LAUNCH(label(), (wgrad_dma_kernel<T, BM, BN, WM, WN, KB, STAGES, PP, true>), grid, block, 0, stream, a);
    else DLK_LAUNCH(label(), (wgrad_dma_kernel<T, BM, BN, WM, WN, KB, STAGES, PP, false>), grid, block, 0, stream, a);
    return dlk::launch_status();
}

// Tiles of the direct-to-LDS kernel (output channels x columns, pixels of a step, workgroups a compute unit holds) and the
// constants of their cost (wgrad_make_plan).
struct WgradTile {
    int bm, bn, kb, per_cu;
    double t0, step, fix;
};
static const WgradTile WGRAD_TILES[] = {
    {256, 256, 32, 1, 6.25, 0.757, 6.98}, {128, 128, 32, 2, 10.70, 0.251, 0.05}, {64, 64, 32, 4, 10.59, 0.111, 0.05}, {64, 128, 64, 2, 10.74, 0.347, 0.05},
    {128, 64, 64, 1, 6.70, 0.353, 3.03},  {64, 64, 64, 3, 10.86, 0.224, 0.05},   {128, 128, 64, 1, 6.47, 0.493, 3.69}, {128, 256, 64, 1, 5.71, 0.846, 5.60}};

WgradPlan wgrad_make_plan(int64_t npix, int64_t x_elems, int K, int C, int RSC, bool thin_ok, bool fetch_term, int64_t max_splits)
{
    static const int forced = tuning_knob("DLCONV_WGRAD_CFG", -2); // tuning override, unset in normal use
    WgradPlan pl{-1, 1, 32, 0, 0};
    if (thin_ok && forced != -1) {
        // streaming kernel: one workgroup per slice of pixels, about eight slices per CU
        int64_t s = (npix + 255) / 256;
        if (s > 2048) s = 2048;
        if (s < 1) s = 1;
        pl.cfg = -2;
        pl.chunk = (int)((npix + s - 1) / s);
        pl.splits = (int)((npix + pl.chunk - 1) / pl.chunk);
        return pl;
    }
    constexpr int NTILES = sizeof(WGRAD_TILES) / sizeof(WGRAD_TILES[0]);
    const bool dma_ok = K % 8 == 0 && C % 8 == 0 && K >= 32 && RSC >= 64;
    if (!dma_ok || forced == -1 || forced >= NTILES) {
        // register-transposing fallback kernel (128 x 128 tiles): about 1024 workgroups
        const int64_t tiles = (int64_t)((K + 127) / 128) * ((RSC + 127) / 128);
        int64_t s = (1024 + tiles - 1) / tiles;
        const int64_t max_by_len = (npix + 127) / 128;       // at least four 32-pixel steps per slice
        if (s > max_by_len) s = max_by_len;
        if (s > 512) s = 512;
        if (s < 1) s = 1;
        int64_t chunk = (npix + s - 1) / s;
        chunk = (chunk + 31) / 32 * 32;
        pl.chunk = (int)chunk;
        pl.splits = (int)((npix + chunk - 1) / chunk);
        return pl;
    }
    // Direct-to-LDS kernel: tile and number of pixel slices by their estimated time in us,
    //   t0 + (steps * step + fix) * (tiles a compute unit works through) + 8 bytes per output and slice at 8.2 TB/s.
    // All tiles of a slice go to one XCD (32 compute units) or, with few slices, to all of them in turn; either way what counts
    // is the compute unit with the most, and where each holds one workgroup, whole rounds of them.  The last term is the
    // partial sums, written and read once: with as many slices as keep every compute unit busy with 128 x 128 tiles they are
    // half the time of a 1x1 filter (6912 pixels, 1024 x 256: 24 slices 22 us, 8 slices of 128 x 64 tiles 15 us).  The constants
    // are fitted to 3600 timings of 104 layers (fp16, 400..460000 pixels, 16..2048 x 32..1024 channels, 1x1 to 7x7); the
    // choice is 5 % behind the best of each on average.
    const double outputs = (double)K * RSC;
    // Tiles of one slice that run on different XCDs share no L2.  With up to nine taps and operands beyond what the L2s hold
    // (32 MB together) every operand tile of a dealt slice may come from the last-level cache or HBM, at about 9 TB/s
    // (fetch_us below).  `pl` is the best plan without that term, `local` the best with it.
    const bool large = fetch_term && RSC / C <= 9 && 2 * (x_elems + npix * K) >= 40000000;
    // Numbers of slices looked at, with the pixels of each: 8, 16, ... 512, the same number on every XCD, each slice on one XCD,
    // or 1 .. 15 whose tiles are dealt over all XCDs.  (Worked out once for all tiles: this runs on every call.)
    struct Slices { int splits, chunk; bool spread; };
    Slices cands[20 + 15];
    int n_cands = 0;
    for (int i = 0; i < 20 + 15; ++i) {
        const bool spread = i >= 20;
        const int s = spread ? i - 19 : i < 8 ? 8 * (i + 1) : i < 12 ? 64 + 16 * (i - 7) : i < 16 ? 128 + 32 * (i - 11) : 256 + 64 * (i - 15);
        if (s > 1 && (int64_t)s * 128 > npix) continue;      // at least four 32-pixel steps per slice
        const uint32_t chunk = (((uint32_t)npix + s - 1) / s + 31) / 32 * 32;
        const int splits = (int)(((uint32_t)npix + chunk - 1) / chunk);
        if (splits == 1 || splits <= max_splits) cands[n_cands++] = Slices{splits, (int)chunk, spread};
    }
    double best = 1e300, best_local = 1e300, pl_steps = 0;
    WgradPlan local = pl;
    for (int cfg = 0; cfg < NTILES; ++cfg) {
        if (forced >= 0 && cfg != forced) continue;
        const WgradTile &sh = WGRAD_TILES[cfg];
        // tiles of 64 only for filters of few outputs or output channels, of 128 x 256 only with more than one row of them:
        // elsewhere the estimates favour them by less than they err
        if (forced < 0 && (sh.bm == 64 || sh.bn == 64) && K > 64 && outputs > 3e5) continue;
        if (forced < 0 && sh.bm < sh.bn && sh.bn == 256 && K <= 128) continue;
        const int64_t tiles = (int64_t)((K + sh.bm - 1) / sh.bm) * ((RSC + sh.bn - 1) / sh.bn);
        const double fetch_us = 2.0 * tiles * (sh.bm + sh.bn) * (double)npix / 9e6;
        for (int i = 0; i < n_cands; ++i) {
            const Slices &c = cands[i];
            const double n = c.spread ? tiles * c.splits / 256.0 : tiles * ((c.splits + 7) / 8) / 32.0;
            const double load = n > 2 * sh.per_cu ? n + 0.3 * sh.per_cu : n > sh.per_cu ? 2 * sh.per_cu : std::ceil(n);
            const double reduce_us = c.splits * outputs * (8.0 / 8.2e6);
            const double steps_us = (((unsigned)(c.chunk + sh.kb - 1) >> (sh.kb == 64 ? 6 : 5)) * sh.step + sh.fix) * load;
            const double est = sh.t0 + steps_us + reduce_us;
            if (est < best) {
                best = est;
                pl = WgradPlan{cfg, c.splits, c.chunk, c.spread ? 1 : 0, est};
                pl_steps = steps_us;
            }
            if (large) {
                const double fetch_est = sh.t0 + std::max(steps_us, c.spread ? fetch_us : 0.0) + reduce_us;
                if (fetch_est < best_local) {
                    best_local = fetch_est;
                    local = WgradPlan{cfg, c.splits, c.chunk, c.spread ? 1 : 0, fetch_est};
                }
            }
        }
    }
    if (!large || !pl.spread) return pl;
    // What the XCDs together fetch of a dealt slice while its tiles keep in step: ids go to the XCDs in turn, column tiles
    // fastest, so a column tile is on min(row tiles, 8 / gcd(column tiles, 8)) of them and a row tile on min(column tiles, 8).
    // Where that, at 6 TB/s, takes longer than the steps does a slice belong on one XCD (not for one row tile of very many
    // columns, whose x is fetched once per tap either way), and where a slice is so long that its tiles drift apart.
    const WgradTile &sh = WGRAD_TILES[pl.cfg];
    const int64_t rows = (K + sh.bm - 1) / sh.bm, cols = (RSC + sh.bn - 1) / sh.bn;
    const int64_t spread8 = cols % 8 == 0 ? 1 : cols % 4 == 0 ? 2 : cols % 2 == 0 ? 4 : 8;
    const double fetched = 2.0 * npix * (cols * std::min(rows, spread8) * sh.bn + rows * std::min<int64_t>(cols, 8) * sh.bm);
    return (fetched / 6e6 > 1.05 * pl_steps && (rows > 1 || cols < 64)) || pl.chunk > 8000 ? local : pl;
}

// The fewest slices that a caller has to bring room for where the direct-to-LDS kernel runs: as many as the first cost model
// of this planner, with four tiles, took with or without its fetch term.  Kept so that a workspace of a size that was
// accepted, or refused, still is.
int wgrad_least_slices(int64_t npix, int64_t x_elems, int K, int C, int RSC)
{
    struct Shape { int bm, bn, per_cu; double us_per_step; };
    static const Shape shapes[4] = {{256, 256, 1, 0.92}, {128, 128, 2, 0.55}, {64, 256, 2, 0.71}, {128, 256, 1, 0.88}};
    const double outputs = (double)K * RSC;
    const bool large = RSC / C <= 9 && 2 * (x_elems + npix * K) >= 40000000;
    double best[2] = {1e300, 1e300};
    int64_t slices[2] = {1, 1};
    for (const Shape &sh : shapes) {
        const int64_t tiles = (int64_t)((K + sh.bm - 1) / sh.bm) * ((RSC + sh.bn - 1) / sh.bn), cap = 32 * sh.per_cu;
        const double fetch_us = 2.0 * tiles * (sh.bm + sh.bn) * (double)npix / 9e6;
        for (int cand = 0; cand < 64 + 15; ++cand) {
            const bool spread = cand >= 64;
            const int64_t s = spread ? cand - 63 : 8 * (cand + 1);
            if (s > 1 && s * 128 > npix) continue;
            const int64_t chunk = ((npix + s - 1) / s + 31) / 32 * 32, splits = (npix + chunk - 1) / chunk;
            const int64_t rounds = spread ? (tiles * splits + 8 * cap - 1) / (8 * cap) : (tiles * ((splits + 7) / 8) + cap - 1) / cap;
            const double reduce_us = (splits > 1 ? splits * outputs * 8.0 : outputs * 6.0) / 11.5e6;
            const double steps_us = rounds * (chunk / 32 + 7) * sh.us_per_step;
            const double est[2] = {steps_us + reduce_us, std::max(steps_us, spread && large ? fetch_us : 0.0) + reduce_us};
            for (int i = 0; i < 2; ++i)
                if (est[i] < best[i]) { best[i] = est[i]; slices[i] = splits; }
        }
    }
    return (int)std::min(slices[0], slices[1]);
}

// the tiles of WGRAD_TILES
template <class T>
static hipError_t dispatch(const WgradArgs &a, int cfg, hipStream_t stream)
{
    switch (cfg) {
        case 0: return launch_cfg<T, 256, 256, 2, 4, 32, 4, true>(a, stream);
        case 1: return launch_cfg<T, 128, 128, 2, 4, 32, 4>(a, stream);
        case 2: return launch_cfg<T, 64, 64, 2, 2, 32, 4>(a, stream);
        case 3: return launch_cfg<T, 64, 128, 2, 4, 64, 3>(a, stream);
        case 4: return launch_cfg<T, 128, 64, 4, 2, 64, 4>(a, stream);
        case 5: return launch_cfg<T, 64, 64, 2, 2, 64, 3>(a, stream);
        case 6: return launch_cfg<T, 128, 128, 4, 4, 64, 3>(a, stream);
        case 7: return launch_cfg<T, 128, 256, 4, 4, 64, 3>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_wgrad_dma(const WgradArgs &a, bool is_bf16, int cfg, hipStream_t stream)
{
    // A step takes a coordinate at most one extent and two strides further than the padded image (with two and more outputs no stride
    // is larger than that): below 2^29 all of it fits 31 bits.  The register-staged kernel counts output pixels instead.
    if (a.H + 2 * (int64_t)a.ph >= 1 << 29 || a.W + 2 * (int64_t)a.pw >= 1 << 29) return launch_wgrad(a, is_bf16, stream);
    return is_bf16 ? dispatch<BF16>(a, cfg, stream) : dispatch<F16>(a, cfg, stream);
}

}  // namespace dlk
