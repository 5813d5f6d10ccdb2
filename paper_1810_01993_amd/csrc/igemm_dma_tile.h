// Implicit-GEMM convolution engine, direct-to-LDS variant (gfx950).
//
// Same GEMM view and tap addressing as the register-staged engine, but the
// activation and filter tiles travel global -> LDS without passing through
// registers: every wave issues `buffer_load_dwordx4 ... lds` instructions,
// each of which deposits 64 lanes x 16 bytes = 1 KB (16 tile rows of 32
// reduction elements) contiguously in LDS.  Out-of-range offsets (zero
// padding, ragged edges, steps past the end of the reduction) deposit zeros.
// A ring of three or four LDS buffers keeps one or two reduction steps in
// flight beyond the one awaited (the one-step kernel, igemm_short.hip, has no
// ring); one barrier per step, two where groups of waves work half a step apart.
// Because the LDS image of a load is contiguous, bank conflicts are avoided by
// swizzling which 16-byte slice of a row each lane fetches instead of padding
// the row pitch.
//
// Two reduction orders:
//   tap-major      kk = (tap*Cin + c) runs linearly; a 32-deep step may
//                  straddle taps.  Any Cin % 8 == 0.
//   channel-major  for each 32-channel chunk all taps are visited in turn, so
//                  a workgroup re-reads the same few input rows tap after tap
//                  while they are cached, and everything that changes from
//                  step to step is wave-uniform: the per-lane work per load is
//                  a bit extract, an or and an add.  Whether a tap of a row falls into
//                  the padding is looked up in a per-row bit mask built once.
//                  A ragged last chunk is zero-filled.  Needs <= 64 taps.
#pragma once
#include "device_common.h"
#include "kernels.h"

namespace dlk {

// Row r of a tile is 64 bytes = 4 slices of 16 bytes.  Logical slice v of row
// r lives at physical slice v ^ ((r >> 2) & 3).  A 16-byte LDS read is served
// 16 lanes (256 bytes, 64 banks) per cycle; the 16 consecutive rows such a
// group reads at one logical slice then fall on 16 different 16-byte bank
// groups: 4*(r & 3) + (v ^ (r >> 2)).  (Measured: twice the read rate of the
// 2-way conflict of an 8-row rule, four times an unswizzled 64-byte pitch.)
// With 64 reduction elements a row is 128 bytes = 8 slices, two rows span the banks, and the rule becomes
// v ^ ((row >> 1) & 7): again 16 consecutive rows at one slice meet 16 different bank groups.
template <int KB>
__device__ __forceinline__ int swz(int row) { return KB == 64 ? (row >> 1) & 7 : (row >> 2) & 3; }

// n / d with the multiplier and shift that FastDiv (kernels.h) computes for d
__device__ __forceinline__ int fast_div(int n, uint32_t mul, int32_t shr)
{
    return (int)((__umulhi((uint32_t)n, mul) + (uint32_t)n) >> shr);
}

typedef short bt_s16x4_t __attribute__((ext_vector_type(4)));

// BT: the filter operand is given reduction-major (see IgemmArgs::b_transposed); channel-major order only.
// Its tile is deposited as it lies in memory, [32 reduction channels][BN columns], 32-byte blocks of a
// row XOR-swizzled with the row index, and the MFMA fragments (8 consecutive reduction channels of one
// column per lane) come from ds_read_b64_tr_b16, as in the filter-gradient kernels.
// The body of the kernel: workgroup `tile` of the GEMM p (tiles are numbered column tile fastest),
// range `split` of a split reduction.
// KB: reduction elements of a step.  SHORT: the whole reduction is one step (STAGES == 1, no ring).
// RES: the residual input is there, aligned for 16-byte loads, and fetched into registers before the first step.
// PP: two groups of waves half a step apart.
template <class T, int BM, int BN, int WM, int WN, bool CMAJOR, bool BT, int KB = 32, int STAGES = 4, bool SHORT = false, bool RES = false, bool PP = false>
__device__ __forceinline__ void igemm_dma_tile(const IgemmArgs &p, const int tile, const int split)
{
    static_assert(!BT || CMAJOR, "a reduction-major filter needs the channel-major order");
    constexpr int NW = WM * WN;
    static_assert(!SHORT || STAGES == 1, "one step");
    static_assert(KB == 32 || (KB == 64 && CMAJOR && NW % 2 == 0), "64-deep steps: channel-major, swizzle independent of the load index");
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int AIW = BM * KB / 512 / NW, BIW = BN * KB / 512 / NW;   // load instructions per wave per step
    static_assert(BM * KB % (512 * NW) == 0 && BN * KB % (512 * NW) == 0, "every wave must issue the same number of loads");
    static_assert(TM >= 1 && TN >= 1, "wave tile too small");
    constexpr int IN_FLIGHT = SHORT ? 0 : (STAGES - 2) * (AIW + BIW);   // loads that may still be pending at the wait

    // Ring slots of both operands in one array; the epilogue re-uses it as staging space.
    __shared__ __align__(16) uint16_t lds[STAGES * (BM + BN) * KB];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    auto slot_a = [&](int s) { return lds + s * BM * KB; };
    auto slot_b = [&](int s) { return lds + STAGES * BM * KB + s * BN * KB; };
    // LDS byte address of this wave's first 1 KB piece of ring slot s
    const uint32_t dst0 = lds_addr(lds) + (uint32_t)wave * 1024;
    auto dst_a = [&](int s) { return dst0 + s * BM * KB * 2; };
    auto dst_b = [&](int s) { return dst0 + (STAGES * BM * KB + s * BN * KB) * 2; };

    const int M = p.NB * p.OH * p.OW;
    const int NT = p.TR * p.TS;                       // taps
    const int Kred = NT * p.Cin;
    const int tiles_n = (p.Nout + BN - 1) / BN;
    const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * BN;

    const i32x4_t rsA = make_rsrc_words(p.A, (uint32_t)p.NB * p.IH * p.IW * p.Cin * 2u);
    const i32x4_t rsB = make_rsrc_words(p.B, BT ? (uint32_t)p.b_elems * 2u : (uint32_t)p.Nout * Kred * 2u);

    // ---- what this lane fetches: row (RPL*inst + lane/SL), logical slice vec --
    constexpr int SL = KB / 8, RPL = 64 / SL;            // 16-byte slices of a row, rows of a load
    const int lrow = lane / SL;                          // row within a load
    const int vec = (lane % SL) ^ swz<KB>(wave * RPL + lrow);   // same for every load of this lane
    int a_ih[AIW], a_iw[AIW];
    uint32_t a_off[AIW];                                 // byte offset of (row's tap (0,0) pixel, channel 8*vec)
    uint32_t out_lo[AIW], out_hi[AIW];                   // channel-major: bit t set = tap t of this row is outside the image
#pragma unroll
    for (int i = 0; i < AIW; ++i) {
        const int m = m0 + (wave + i * NW) * RPL + lrow;
        out_lo[i] = out_hi[i] = ~0u;
        if (m < M) {
            const int n = fast_div(m, p.mul_hw, p.shr_hw), rem = m - n * (p.OH * p.OW);
            const int oh = fast_div(rem, p.mul_w, p.shr_w), ow = rem - oh * p.OW;
            a_ih[i] = oh * p.sh + p.th0;
            a_iw[i] = ow * p.sw + p.tw0;
            a_off[i] = (uint32_t)(((n * p.IH + a_ih[i]) * p.IW + a_iw[i]) * p.Cin + vec * 8) * 2u;
            if constexpr (CMAJOR) {
                uint64_t cols = 0, in = 0;               // taps of one filter row, then of all
                for (int js = 0; js < p.TS; ++js) cols |= (uint64_t)((unsigned)(a_iw[i] + js * p.dtw) < (unsigned)p.IW ? 1u : 0u) << js;
                for (int jr = 0; jr < p.TR; ++jr)
                    if ((unsigned)(a_ih[i] + jr * p.dth) < (unsigned)p.IH) in |= cols << (jr * p.TS);
                out_lo[i] = ~(uint32_t)in;
                out_hi[i] = ~(uint32_t)(in >> 32);
            }
        } else {
            a_off[i] = 0;
            a_ih[i] = -(1 << 28);                        // fails every bounds test
            a_iw[i] = 0;
        }
    }
    uint32_t b_off[BIW];                                 // byte offset of (filter row, reduction index 8*vec)
    bool b_ok[BIW];
#pragma unroll
    for (int i = 0; i < BIW; ++i) {
        const int j = n0 + (wave + i * NW) * RPL + lrow;
        b_ok[i] = j < p.Nout;
        b_off[i] = ((uint32_t)j * (uint32_t)Kred + vec * 8) * 2u;
    }
    // reduction-major filter: a load covers RPI_B reduction rows of BN columns (LPR_B lanes of 16 bytes each);
    // load `inst` = wave + i*NW of a step holds rows inst*RPI_B .. +RPI_B-1, so row & 3 does not depend on i
    constexpr int LPR_B = BN / 8, RPI_B = 64 / LPR_B;
    constexpr int BT_SHIFT = BN >= 128 ? 1 : 0;          // rows of >= 8 blocks: spread 4 rows x 2 blocks over 8 bank ranges
    static_assert(!BT || (NW * RPI_B) % 4 == 0, "swizzle must not depend on the load index");
    const int bt_row = lane / LPR_B;                     // row within a load
    const int bt_row3 = (wave * RPI_B + bt_row) & 3;
    const int bt_pc = lane % LPR_B;                      // physical 16-byte chunk within the row
    const int bt_blk = BN >= 64 ? ((bt_pc >> 1) ^ (bt_row3 << BT_SHIFT)) : (bt_pc >> 1);
    const int bt_col = n0 + ((bt_blk << 1) | (bt_pc & 1)) * 8;
    const bool bt_ok = bt_col < p.Nout;

    // ---- reduction cursor ---------------------------------------------------
    // channel-major: (t, jr, js, c0) are wave-uniform; tap-major: (kk, c, js, jr) per lane
    // channels [c_first, c_end) of the reduction belong to this workgroup (all of them unless the reduction is split)
    int c_first = 0, c_end = p.Cin;
    if (CMAJOR && p.ksplits > 1) {
        c_first = split * p.split_chunks * BK;
        c_end = min(p.Cin, c_first + p.split_chunks * BK);
    }
    int t = 0, jr = 0, js = 0, c0 = c_first;              // (channel-major: jr only sets up the first step)
    int kk = vec * 8, c = 0;
    if constexpr (!CMAJOR) { c = kk % p.Cin; js = (kk / p.Cin) % p.TS; jr = (kk / p.Cin) / p.TS; }
    const int lane_c = vec * 8;
    const int nk = CMAJOR ? ((c_end - c_first + KB - 1) / KB) * NT : (Kred + KB - 1) / KB;
    // Channel-major: what a step adds to the lanes' offsets is kept as two running scalars, and what is outside as bits that
    // turn an offset into one out of range, so that a load costs three or two vector instructions (the waves of a small
    // tile spend as long on issuing a step as on multiplying it).
    const uint32_t a_js = (uint32_t)(p.dtw * p.Cin) * 2u, a_jr = (uint32_t)((p.dth * p.IW - p.TS * p.dtw) * p.Cin) * 2u;
    const uint32_t a_ch = (uint32_t)(KB - p.TR * p.dth * p.IW * p.Cin) * 2u;
    const uint32_t b_js = (uint32_t)(BT ? p.b_ss : p.Cin) * 2u, b_jr = BT ? (uint32_t)(p.b_sr - p.TS * p.b_ss) * 2u : 0u;
    const uint32_t b_ch = BT ? (uint32_t)(KB * p.b_ldk - p.TR * p.b_sr) * 2u : (uint32_t)(KB - NT * p.Cin) * 2u;
    uint32_t tap_a = (uint32_t)((jr * p.dth * p.IW + js * p.dtw) * p.Cin + c0) * 2u;
    uint32_t tap_b = BT ? (uint32_t)(p.b_base + jr * p.b_sr + js * p.b_ss + c0 * p.b_ldk) * 2u : (uint32_t)(t * p.Cin + c0) * 2u;
    uint32_t out_cur[AIW], b_out[BIW];
    // the part of the reduction that begins at channel c0: what of a ragged last chunk, or behind the end, does not exist
    auto open_chunk = [&]() {
        if (c0 + KB > c_end) {
            const bool gone = lane_c >= c_end - c0;
#pragma unroll
            for (int i = 0; i < AIW; ++i) {
                if (gone) out_lo[i] = out_hi[i] = ~0u;
            }
#pragma unroll
            for (int i = 0; i < BIW; ++i) {
                if constexpr (BT) {
                    if (c0 + (wave + i * NW) * RPI_B + bt_row >= c_end) b_out[i] = OOB_OFFSET;
                } else if (gone) b_out[i] = OOB_OFFSET;
            }
        }
    };
    auto select_mask = [&]() {                           // the word of the mask that holds tap t
#pragma unroll
        for (int i = 0; i < AIW; ++i) out_cur[i] = t < 32 ? out_lo[i] : out_hi[i];
    };
    if constexpr (CMAJOR) {
#pragma unroll
        for (int i = 0; i < BIW; ++i) {
            if constexpr (BT) {
                b_off[i] = (uint32_t)(bt_col + ((wave + i * NW) * RPI_B + bt_row) * p.b_ldk) * 2u;
                b_out[i] = bt_ok ? 0u : OOB_OFFSET;
            } else b_out[i] = b_ok[i] ? 0u : OOB_OFFSET;
        }
        open_chunk();
        select_mask();
    }

    // Issue the loads of the next reduction step into ring slot s.
    auto issue = [&](int s) __attribute__((always_inline)) {
        const uint32_t sa = dst_a(s), sb = dst_b(s);
        if constexpr (CMAJOR) {
#pragma unroll
            for (int i = 0; i < AIW; ++i) {
                const uint32_t outside = (uint32_t)__builtin_amdgcn_sbfe((int)out_cur[i], t & 31, 1) & OOB_OFFSET;   // bit t, all ones or zero
                dma_load_16B(rsA, sa + i * NW * 1024, (a_off[i] + tap_a) | outside);
            }
#pragma unroll
            for (int i = 0; i < BIW; ++i) dma_load_16B(rsB, sb + i * NW * 1024, (b_off[i] + tap_b) | b_out[i]);
            ++t;
            tap_a += a_js;
            tap_b += b_js;
            if (t == 32) select_mask();
            if (++js == p.TS) {
                js = 0;
                tap_a += a_jr;
                tap_b += b_jr;
                if (t == NT) {
                    t = 0;
                    c0 += KB;
                    tap_a += a_ch;
                    tap_b += b_ch;
                    open_chunk();
                    select_mask();
                }
            }
        } else {
            const bool kin = kk < Kred;
            const int dh = jr * p.dth, dw = js * p.dtw;
            const uint32_t tap_a = (uint32_t)((dh * p.IW + dw) * p.Cin + (c - lane_c)) * 2u;
#pragma unroll
            for (int i = 0; i < AIW; ++i) {
                const int ih = a_ih[i] + dh, iw = a_iw[i] + dw;
                const bool ok = kin && (unsigned)ih < (unsigned)p.IH && (unsigned)iw < (unsigned)p.IW;
                dma_load_16B(rsA, sa + i * NW * 1024, ok ? a_off[i] + tap_a : OOB_OFFSET);
            }
#pragma unroll
            for (int i = 0; i < BIW; ++i)
                dma_load_16B(rsB, sb + i * NW * 1024,
                             (kin && b_ok[i]) ? b_off[i] + (uint32_t)(kk - lane_c) * 2u : OOB_OFFSET);
            kk += KB;
            c += KB;
            while (c >= p.Cin) {
                c -= p.Cin;
                if (++js == p.TS) { js = 0; ++jr; }
            }
        }
    };

    floatx16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // fragment addressing: row (lane % 32) of a 32-row MFMA tile, slices 2*ks + lane/32
    const int frow = lane & 31;
    const int fsw = swz<KB>(frow);                       // tile bases are multiples of 32 rows
    constexpr int KS = KB / 16;                          // 16-deep slices of a step
    int foff[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) foff[ks] = frow * KB + (((ks * 2 + (lane >> 5)) ^ fsw) << 3);

    // MFMAs of one slot (KS 16-deep slices); the fragments of all slices are
    // requested from LDS before the first MFMA is issued.
    // transpose-read addressing of a [32][BN] tile: lane = 16*g + q points at reduction row
    // 8*(g>>1) + 4*half + q/4 (+ 16*ks) and columns 16*(g&1) + 4*(q%4)..+3 of a 32-column MFMA tile
    const int tg = lane >> 4, tq = lane & 15;
    const int t_row = 8 * (tg >> 1) + (tq >> 2);
    const int t_sw = BN >= 64 ? ((t_row & 3) << BT_SHIFT) : 0;        // same for row + 4 and row + 16
    const int t_sub = 4 * (tq & 3), t_blk = tg & 1;
    auto load_frags = [&](u32x4_t (&a)[TM], u32x4_t (&b)[TN], const uint16_t *sa, const uint16_t *sb, int ks) {
        const uint16_t *wa = sa + wm * TM * 32 * KB + foff[ks];
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const u32x4_t *>(wa + i * 32 * KB);
        if constexpr (BT) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int blk = ((wn * TN + j) * 2 + t_blk) ^ t_sw;
                const uint16_t *lo = sb + (16 * ks + t_row) * BN + blk * 16 + t_sub;
                const bt_s16x4_t l4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((bt_s16x4_t __attribute__((address_space(3))) *)lo);
                const bt_s16x4_t h4 =
                    __builtin_amdgcn_ds_read_tr16_b64_v4i16((bt_s16x4_t __attribute__((address_space(3))) *)(lo + 4 * BN));
                const u32x2_t l2 = __builtin_bit_cast(u32x2_t, l4), h2 = __builtin_bit_cast(u32x2_t, h4);
                b[j][0] = l2[0]; b[j][1] = l2[1]; b[j][2] = h2[0]; b[j][3] = h2[1];
            }
        } else {
            const uint16_t *wb = sb + wn * TN * 32 * KB + foff[ks];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const u32x4_t *>(wb + j * 32 * KB);
        }
    };
    // One step: fragments of slot u, the loads of a later step into slot next, then the products.  The fragments are
    // requested first: a wave waits in line to issue its loads, and the LDS answers meanwhile.
    auto step = [&](int u, int next) __attribute__((always_inline)) {
        u32x4_t fa[KS][TM], fb[KS][TN];
#pragma unroll
        for (int s = 0; s < KS; ++s) load_frags(fa[s], fb[s], slot_a(u), slot_b(u), s);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!SHORT) issue(next);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = T::mfma(fb[s][j], fa[s][i], acc[i][j]);   // rows = output channels
    };

    // Wait until this wave's loads for the oldest pending step have landed,
    // then meet the other waves: after the barrier the step's tile is complete
    // in LDS and nobody still reads the slot that is refilled next.
    auto wait_and_sync = [&]() {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(IN_FLIGHT) : "memory");
    };

    // The residual's rows of this wave's tile, 16 bytes per lane the way the output is written.  Fetched here, ahead of
    // the first step's loads (and so awaited with them): in the epilogue every 32-row slab waited for its own round trip
    // (6912 pixels, 256 -> 1024 17.6 -> 16.4 us, 3015 pixels 10.4 -> 9.8 us).  Only for tiles of at most 128 columns, whose
    // residual takes at most 32 registers (256 x 256: 64).
    constexpr int CH = TN * 32;                          // channels per wave
    constexpr int LPR = CH / 8;                          // lanes per row when writing out
    const bool dense = (p.osh == 1 && p.osw == 1 && p.FH == p.OH && p.FW == p.OW);
    auto out_row = [&](int m) -> size_t {                // element offset of output row m
        if (dense) return (size_t)m * p.ldd;
        const int n = fast_div(m, p.mul_hw, p.shr_hw), rem = m - n * (p.OH * p.OW);
        const int oh = fast_div(rem, p.mul_w, p.shr_w), ow = rem - oh * p.OW;
        return ((size_t)(n * p.FH + oh * p.osh + p.ooh) * p.FW + ow * p.osw + p.oow) * p.ldd;
    };
    u32x4_t resid[RES ? TM : 1][RES ? LPR / 2 : 1];
    if constexpr (RES) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int it = 0; it < LPR / 2; ++it) {
                const int m = m0 + (wm * TM + i) * 32 + it * (64 / LPR) + lane / LPR;
                const int col = n0 + wn * CH + (lane % LPR) * 8;
                resid[i][it] = u32x4_t{0, 0, 0, 0};
                if (m < M && col < p.Nout) resid[i][it] = *reinterpret_cast<const u32x4_t *>(p.resid + out_row(m) + col);
            }
    }

    // The step count is rounded up to a whole turn of the ring (the extra
    // steps load and multiply zeros) so that the unrolled loop has one exit.
    const int nturns = (nk + STAGES - 1) / STAGES;
    if constexpr (SHORT) {
        issue(0);
        wait_and_sync();
        step(0, 0);
    } else if constexpr (PP) {
        // Two groups of waves, one of each on every SIMD, half a step apart: one reads its fragments and issues loads
        // while the other multiplies.  Both barriers of a step leave STAGES - 2 steps of this wave's loads pending: at the
        // one that opens its read phase of step s it has issued up to step s + STAGES - 2, so s has landed; at the other,
        // where the other group may open its read phase of s + 1, it has issued one step more, so s + 1 has.  Its LDS reads
        // are complete at either, so the slot refilled in a read phase, that of s - 1, is no longer read by anyone.
        static_assert(STAGES >= 3 && NW == 8, "one wave of each group per SIMD");
        auto hand_over = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            wait_and_sync();
            __builtin_amdgcn_sched_barrier(0);
        };
        if (nk > 0) {
#pragma unroll
            for (int u = 0; u < STAGES - 1; ++u) issue(u);
            const bool late = wave >= NW / 2;
            if (late) hand_over();
            for (int turn = 0; turn < nturns; ++turn) {
#pragma unroll
                for (int u = 0; u < STAGES; ++u) {
                    u32x4_t fa[KS][TM], fb[KS][TN];
                    hand_over();
#pragma unroll
                    for (int s = 0; s < KS; ++s) load_frags(fa[s], fb[s], slot_a(u), slot_b(u), s);
                    __builtin_amdgcn_sched_barrier(0);
                    issue((u + STAGES - 1) % STAGES);
                    hand_over();
#pragma unroll
                    for (int s = 0; s < KS; ++s)
#pragma unroll
                        for (int i = 0; i < TM; ++i)
#pragma unroll
                            for (int j = 0; j < TN; ++j) acc[i][j] = T::mfma(fb[s][j], fa[s][i], acc[i][j]);
                }
            }
            if (!late) hand_over();
        }
    } else if (nk > 0) {
#pragma unroll
        for (int u = 0; u < STAGES - 1; ++u) issue(u);
        for (int turn = 0; turn < nturns; ++turn) {
#pragma unroll
            for (int u = 0; u < STAGES; ++u) {
                wait_and_sync();
                step(u, (u + STAGES - 1) % STAGES);
            }
        }
    }
    // every wave's loads (the trailing ones deposit zeros) and LDS reads are over before LDS is reused
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- epilogue ---------------------------------------------------------------
    // The filter rode in the first MFMA operand, so register v of lane l holds output
    // channel 8*(v/4) + 4*(l/32) + v%4 of tile row l%32: four consecutive channels per
    // register quartet.  Each wave rounds one 32-row slab of its tile at a time, parks it in a
    // private LDS area as [row][channel] (pitch: the wave's channels + 8 bytes, conflict-free
    // for the 8-byte writes) and writes it out 16 bytes per lane, whole rows of the wave's
    // channel range at a time.
    if (CMAJOR && p.ksplits > 1) {
        // split reduction: fp32 partial sums, four consecutive channels per store
        float *out = p.part + (size_t)split * M * p.Nout;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m0 + (wm * TM + i) * 32 + (lane & 31);
            if (m >= M) continue;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int col = n0 + (wn * TN + j) * 32 + 8 * g + 4 * (lane >> 5);
                    float *dst = out + (size_t)m * p.Nout + col;
                    if (col + 3 < p.Nout && (p.Nout & 3) == 0) {
                        floatx4_t v4;
                        v4[0] = acc[i][j][4 * g]; v4[1] = acc[i][j][4 * g + 1]; v4[2] = acc[i][j][4 * g + 2]; v4[3] = acc[i][j][4 * g + 3];
                        *reinterpret_cast<floatx4_t *>(dst) = v4;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (col + e < p.Nout) dst[e] = acc[i][j][4 * g + e];
                    }
                }
        }
        return;
    }
    constexpr int EP = CH + 4;                           // staging pitch in 16-bit elements
    static_assert(NW * 32 * EP <= STAGES * (BM + BN) * KB, "staging area must fit the ring");
    uint16_t *stg = lds + wave * 32 * EP;
    const bool vec_ok = (p.ldd % 8 == 0) && (p.Nout % 8 == 0) && ((reinterpret_cast<uintptr_t>(p.D) & 15) == 0);
    const bool tail = p.bias != nullptr || p.relu != 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        // A residual input is added before the rounding.  Its 32-row slab is fetched the way the output is
        // written (16 bytes per lane, whole rows of the wave's channel range) into the staging area, and every
        // lane then picks up the four values that belong to its accumulators.
        if constexpr (RES) {
#pragma unroll
            for (int it = 0; it < LPR / 2; ++it) {
                const int row = it * (64 / LPR) + lane / LPR, c8 = (lane % LPR) * 8;
                *reinterpret_cast<u32x2_t *>(stg + row * EP + c8) = u32x2_t{resid[i][it][0], resid[i][it][1]};
                *reinterpret_cast<u32x2_t *>(stg + row * EP + c8 + 4) = u32x2_t{resid[i][it][2], resid[i][it][3]};
            }
        } else if (p.resid) {
#pragma unroll
            for (int it = 0; it < LPR / 2; ++it) {
                const int row = it * (64 / LPR) + lane / LPR, c8 = (lane % LPR) * 8;
                const int m = m0 + (wm * TM + i) * 32 + row;
                const int col = n0 + wn * CH + c8;
                u32x2_t lo{0, 0}, hi{0, 0};
                if (m < M && col < p.Nout) {
                    const uint16_t *src = p.resid + out_row(m) + col;
                    if (vec_ok && (reinterpret_cast<uintptr_t>(p.resid) & 15) == 0) {
                        const u32x4_t v4 = *reinterpret_cast<const u32x4_t *>(src);
                        lo[0] = v4[0]; lo[1] = v4[1]; hi[0] = v4[2]; hi[1] = v4[3];
                    } else {
                        uint32_t w4[4] = {0, 0, 0, 0};
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (col + e < p.Nout) w4[e >> 1] |= (uint32_t)src[e] << (16 * (e & 1));
                        lo[0] = w4[0]; lo[1] = w4[1]; hi[0] = w4[2]; hi[1] = w4[3];
                    }
                }
                *reinterpret_cast<u32x2_t *>(stg + row * EP + c8) = lo;
                *reinterpret_cast<u32x2_t *>(stg + row * EP + c8 + 4) = hi;
            }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int row = lane & 31, ch = j * 32 + 8 * g + 4 * (lane >> 5);
                floatx4_t c{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                if (RES || p.resid) {
                    const u32x2_t r = *reinterpret_cast<const u32x2_t *>(stg + row * EP + ch);
                    c[0] += T::to_float((uint16_t)(r[0] & 0xffffu));
                    c[1] += T::to_float((uint16_t)(r[0] >> 16));
                    c[2] += T::to_float((uint16_t)(r[1] & 0xffffu));
                    c[3] += T::to_float((uint16_t)(r[1] >> 16));
                }
                if (tail) c = apply_tail4(c, p.bias, p.relu, n0 + wn * CH + ch, p.Nout);
                u32x2_t pk;
                pk[0] = (uint32_t)T::from_float(c[0]) | ((uint32_t)T::from_float(c[1]) << 16);
                pk[1] = (uint32_t)T::from_float(c[2]) | ((uint32_t)T::from_float(c[3]) << 16);
                *reinterpret_cast<u32x2_t *>(stg + row * EP + ch) = pk;
            }
#pragma unroll
        for (int it = 0; it < LPR / 2; ++it) {           // 32 rows x LPR lanes, 64 lanes at a time
            const int row = it * (64 / LPR) + lane / LPR, c8 = (lane % LPR) * 8;
            const u32x2_t lo = *reinterpret_cast<const u32x2_t *>(stg + row * EP + c8);
            const u32x2_t hi = *reinterpret_cast<const u32x2_t *>(stg + row * EP + c8 + 4);
            const int m = m0 + (wm * TM + i) * 32 + row;
            const int col = n0 + wn * CH + c8;
            if (m >= M || col >= p.Nout) continue;
            uint16_t *dst = p.D + out_row(m) + col;
            if (vec_ok) {
                u32x4_t v4;
                v4[0] = lo[0]; v4[1] = lo[1]; v4[2] = hi[0]; v4[3] = hi[1];
                *reinterpret_cast<u32x4_t *>(dst) = v4;
            } else {
                const uint32_t w4[4] = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (col + e < p.Nout) dst[e] = (uint16_t)(w4[e >> 1] >> (16 * (e & 1)));
            }
        }
    }
}

}  // namespace dlk
