// Implicit-GEMM convolution engine for gfx950 (forward pass and, through a
// re-laid-out filter, the data gradient).
//
// GEMM view: M = N*OH*OW output pixels, N = output channels, reduction over
// (tap, input channel).  The im2col matrix is never materialised: every load
// computes its own source pixel from (output pixel, tap), which is where
// stride, padding and dilation enter.  This file holds the host-side choice of
// kernel and tile for one implicit GEMM, the element-wise kernel for channel
// counts that are not a multiple of 8, and the filter re-layout for data
// gradients that cannot read the filter in place.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace dlk {

// ===========================================================================
// Scalar kernel: any channel count; elements are fetched one by one.  Used
// only when Cin is not a multiple of 8.
// ===========================================================================
template <class T>
__global__ __launch_bounds__(256) void igemm_scalar_kernel(const IgemmArgs p)
{
    constexpr int BM = 128, BN = 64, WN = 2, TM = 2, TN = 1, RPP = 64, PA = 2, PB = 1;
    __shared__ __align__(16) uint16_t sA[BM * LDS_PITCH];
    __shared__ __align__(16) uint16_t sB[BN * LDS_PITCH];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int M = p.NB * p.OH * p.OW;
    const int Kred = p.TR * p.TS * p.Cin;
    const int tiles_n = (p.Nout + BN - 1) / BN;
    const int m0 = (blockIdx.x / tiles_n) * BM, n0 = (blockIdx.x % tiles_n) * BN;

    const int vec = tid & 3, row0 = tid >> 2;
    int a_pix[PA], a_ih[PA], a_iw[PA];
#pragma unroll
    for (int i = 0; i < PA; ++i) {
        const int m = m0 + row0 + i * RPP;
        if (m < M) {
            const int n = m / (p.OH * p.OW), rem = m - n * (p.OH * p.OW);
            const int oh = rem / p.OW, ow = rem - oh * p.OW;
            a_pix[i] = n * p.IH * p.IW;
            a_ih[i] = oh * p.sh + p.th0;
            a_iw[i] = ow * p.sw + p.tw0;
        } else {
            a_pix[i] = 0;
            a_ih[i] = -(1 << 28);
            a_iw[i] = 0;
        }
    }

    floatx16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][0][v] = 0.f;

    const int nk = (Kred + BK - 1) / BK;
    for (int kt = 0; kt < nk; ++kt) {
        uint16_t ea[PA][8], eb[PB][8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k1 = kt * BK + vec * 8 + e;
            const bool kin = k1 < Kred;
            const int t = k1 / p.Cin, c1 = k1 - t * p.Cin;
            const int r1 = t / p.TS, s1 = t - r1 * p.TS;
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                const int ih = a_ih[i] + r1 * p.dth, iw = a_iw[i] + s1 * p.dtw;
                const bool ok = kin && (unsigned)ih < (unsigned)p.IH && (unsigned)iw < (unsigned)p.IW;
                ea[i][e] = ok ? p.A[(size_t)(a_pix[i] + ih * p.IW + iw) * p.Cin + c1] : (uint16_t)0;
            }
            const int j = n0 + row0;
            eb[0][e] = (kin && j < p.Nout) ? p.B[(size_t)j * Kred + k1] : (uint16_t)0;
        }
        __syncthreads();                                 // previous step's fragment reads are done
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            u32x4_t v;
#pragma unroll
            for (int d = 0; d < 4; ++d) v[d] = (uint32_t)ea[i][2 * d] | ((uint32_t)ea[i][2 * d + 1] << 16);
            *reinterpret_cast<u32x4_t *>(sA + (row0 + i * RPP) * LDS_PITCH + vec * 8) = v;
        }
        {
            u32x4_t v;
#pragma unroll
            for (int d = 0; d < 4; ++d) v[d] = (uint32_t)eb[0][2 * d] | ((uint32_t)eb[0][2 * d + 1] << 16);
            *reinterpret_cast<u32x4_t *>(sB + row0 * LDS_PITCH + vec * 8) = v;
        }
        __syncthreads();
        mma_step<T, TM, TN, BK>(sA + wm * TM * 32 * LDS_PITCH, sB + wn * TN * 32 * LDS_PITCH, lane, acc);
    }

    const bool dense = (p.osh == 1 && p.osw == 1 && p.FH == p.OH && p.FW == p.OW);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int m = m0 + (wm * TM + i) * 32 + acc_row(v, lane);
            if (m >= M) continue;
            size_t row_off;
            if (dense) {
                row_off = (size_t)m * p.ldd;
            } else {
                const int n = m / (p.OH * p.OW), rem = m - n * (p.OH * p.OW);
                const int oh = rem / p.OW, ow = rem - oh * p.OW;
                row_off = ((size_t)(n * p.FH + oh * p.osh + p.ooh) * p.FW + ow * p.osw + p.oow) * p.ldd;
            }
            const int col = n0 + wn * 32 + (lane & 31);
            if (col < p.Nout) {
                const float r = p.resid ? T::to_float(p.resid[row_off + col]) : 0.f;
                p.D[row_off + col] = T::from_float(apply_tail(acc[i][0][v] + r, p.bias, p.relu, col));
            }
        }
}

// ===========================================================================
// Host side: tile selection and launch
// ===========================================================================
// Tuning override: DLCONV_IGEMM_CFG=<n> forces tile n for every vector-path launch (used by the tile sweeps; unset in
// normal use).
static int forced_cfg() { return tuning_knob("DLCONV_IGEMM_CFG", -1); }

static bool choose_c_outer(const IgemmArgs &a)
{
    // channel-major order needs the tap mask to fit 64 bits and no chunk that is mostly padding
    return a.TR * a.TS <= 64 && (a.Cin % 32 == 0 || a.Cin >= 128);
}

// ---- tile and split of the reduction ---------------------------------------------
// Estimated time of a GEMM in us: t0 + (steps * step + fix) * (tiles a compute unit works through).  The last factor is
// the number of rounds where a compute unit holds one tile, and the tiles themselves, rounded up while they are few, where it
// holds several.  t0, step and fix per tile, for 1x1 filters and for more taps, are fitted to 465 random GEMMs (forward and
// data gradient, 400..260000 pixels, 32..2048 x 40..2048 channels, 1x1 to 5x5; fp16) timed with every tile: the choice is
// 3 % slower than the best tile of each on average, 26 % at worst.
struct TileCost { double t0, step, fix; };
struct TileInfo {
    int bm, bn, kb, per_cu;
    TileCost cost[2];           // 1x1, more taps
};
static const TileInfo TILES[TILE_COUNT] = {
    {64, 32, 32, 6, {{6.18, 0.068, 0.050}, {4.49, 0.075, 0.050}}},
    {64, 64, 32, 4, {{5.25, 0.100, 0.361}, {3.95, 0.098, 0.102}}},
    {64, 64, 64, 2, {{4.42, 0.159, 1.153}, {3.78, 0.160, 0.974}}},
    {128, 64, 64, 2, {{4.08, 0.256, 1.479}, {3.10, 0.247, 1.229}}},
    {128, 128, 32, 2, {{3.88, 0.215, 1.661}, {3.00, 0.193, 1.445}}},
    {128, 128, 64, 1, {{3.00, 0.414, 3.796}, {3.00, 0.342, 3.684}}},
    {256, 128, 64, 1, {{3.00, 0.675, 4.538}, {3.00, 0.511, 4.149}}},
    {256, 256, 32, 1, {{3.00, 0.491, 5.601}, {3.00, 0.443, 5.970}}},
};

static int64_t tile_count(const TileInfo &t, int64_t M, int Nout) { return ((M + t.bm - 1) / t.bm) * ((Nout + t.bn - 1) / t.bn); }

static double tiles_per_cu(int per_cu, int64_t tiles)
{
    const double n = tiles / 256.0;
    if (n > 2 * per_cu) return n + 0.3 * per_cu;
    return n > per_cu ? 2 * per_cu : std::ceil(n);
}

static double tile_work(const IgemmArgs &a, int tile, int steps)
{
    const TileCost &c = TILES[tile].cost[a.TR * a.TS == 1 ? 0 : 1];
    return steps * c.step + c.fix;
}

static int tile_steps(const IgemmArgs &a, int tile) { return (a.Cin + TILES[tile].kb - 1) / TILES[tile].kb * a.TR * a.TS; }

// Whether the choice among tiles for GEMM a considers this one at all.  The narrowest is for at most 32 columns; the two
// largest leave nothing beside them on a compute unit to cover their epilogues, which weigh as much as a short reduction (1x1,
// 41402 pixels, 128 -> 2048: 256 x 256 82 us, 128 x 128 50).
static bool tile_considered(const IgemmArgs &a, int tile)
{
    if (tile == TILE_64x32) return a.Nout <= 32;
    if (tile == TILE_256x128_K64 || tile == TILE_256x256) return a.TR * a.TS > 1 || a.Cin >= 512;
    return true;
}

// Tap-major order (few channels): 32-deep steps across the taps, and waves that spend longer on an address.  Constants of their
// own, fitted to 7500 random layers (forward, 50..800000 pixels, 8..120 x 8..1040 channels, 1x1 to 7x7; fp16) timed with every
// tile: 0.4 % behind the best of each on average, 1.3x at worst.  While all tiles are resident, rounds count in halves, those of
// 64 x 64 tiles up to the second in quarters: 260 of them on 256 compute units take 1.3x as long as 256, not twice (2 x 50 x 71,
// 120 -> 528, 7x7, stride 2: 35.5 us; 135 tiles of 128 x 64, which an estimate in halves preferred, 52.3), 530 take 2.5x (1 x 177
// x 192, 56 -> 64, 7x7: 36.0 us; 128 x 64 27.4).  Tiles wider than the columns are left out, and the largest for short
// reductions, whose epilogue nothing covers (147000 pixels, 120 -> 256, 1x1: 45 us, 128 x 128 30).
struct TapMajorTile { int tile, bm, bn, per_cu; TileCost cost; };
static const TapMajorTile TAP_MAJOR_TILES[] = {{TILE_64x32, 64, 32, 6, {3.75, 0.113, 0.22}},
                                               {TILE_64x64, 64, 64, 4, {3.36, 0.129, 0.51}},
                                               {TILE_128x64, 128, 64, 3, {3.41, 0.191, 0.98}},
                                               {TILE_128x128, 128, 128, 2, {2.50, 0.226, 2.05}},
                                               {TILE_256x256, 256, 256, 1, {2.50, 0.633, 6.22}}};

static int best_tap_major_tile(const IgemmArgs &a, double *us)
{
    const int64_t M = (int64_t)a.NB * a.OH * a.OW;
    const int steps = (a.TR * a.TS * a.Cin + BK - 1) / BK;
    // An output of more than 240 MB (the last-level cache holds 256) and little else to do: rows of it as wide as a tile can (500000
    // pixels, 24 -> 440, 1x1: 124 us, 128 x 128 166, cut 151; below that size 128 x 128 is 1.2x as fast), cut only where the last
    // tile would be mostly empty (506000 pixels, 24 -> 320: cut 102 us, 142 in one; from 400 MB on one launch is as fast from 65
    // columns on).  These times are not the sum of steps that the estimates below are.
    if (M * a.Nout >= 120000000 && a.Nout > 128 && steps < 16) {
        const int rem = a.Nout % 256;
        const bool cut = a.Nout > 256 && rem > 0 && rem <= (M * a.Nout < 200000000 ? 128 : 64);
        *us = cut ? 1e9 : 0;
        return TILE_256x256;
    }
    int best = -1;
    for (const TapMajorTile &t : TAP_MAJOR_TILES) {
        if ((t.tile == TILE_64x32) != (a.Nout <= 32) || (t.bn >= 128 && a.Nout <= 64) || (t.bn == 256 && (a.Nout <= 128 || steps < 16))) continue;
        const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((a.Nout + t.bn - 1) / t.bn);
        const int parts = t.tile == TILE_64x64 && tiles <= 512 ? 4 : 2;
        const double load = tiles <= 256 * t.per_cu ? std::max(1.0, std::ceil(tiles * parts / 256.0) / parts) : tiles_per_cu(t.per_cu, tiles);
        const double est = t.cost.t0 + (steps * t.cost.step + t.cost.fix) * load;
        if (best < 0 || est < *us) { best = t.tile; *us = est; }
    }
    return best;
}

static int best_tile(const IgemmArgs &a, double *us)
{
    if (!choose_c_outer(a)) return best_tap_major_tile(a, us);
    const int64_t M = (int64_t)a.NB * a.OH * a.OW;
    int best = -1;
    for (int t = 0; t < TILE_COUNT; ++t) {
        if (!tile_considered(a, t)) continue;
        const double est = TILES[t].cost[a.TR * a.TS == 1 ? 0 : 1].t0 + tile_work(a, t, tile_steps(a, t)) * tiles_per_cu(TILES[t].per_cu, tile_count(TILES[t], M, a.Nout));
        if (best < 0 || est < *us) { best = t; *us = est; }
    }
    return best;
}

// How a GEMM runs: tile, and the ranges its reduction is cut into (1: not cut) of `chunks` 32-channel chunks each.
struct IgemmPlan { int tile, ksplits, chunks; };

// GEMMs with few tiles and a long reduction leave most compute units idle, or walk it in many steps of small tiles.  Cut
// into ranges that run side by side, with an ordered reduce of their fp32 partial sums (4 us, and 8 bytes per output
// and range at 8 TB/s): 6912 pixels, 2048 -> 256, 3x3: 216 tiles of 128 x 64 84 us, 54 tiles of 256 x 128 in four ranges 66 us
// with the reduce.  room: bytes of scratch for the partial sums.
static IgemmPlan make_plan(const IgemmArgs &a, size_t room)
{
    IgemmPlan pl{0, 1, 0};
    if (forced_cfg() >= 0) { pl.tile = forced_cfg(); return pl; }
    double us = 0;
    pl.tile = best_tile(a, &us);
    if (!choose_c_outer(a)) return pl;
    const bool dense = a.osh == 1 && a.osw == 1 && a.FH == a.OH && a.FW == a.OW && a.ldd == a.Nout;
    const int64_t M = (int64_t)a.NB * a.OH * a.OW;
    if (!dense || a.Nout % 8 != 0 || M * a.Nout > (4 << 20)) return pl;
    const int chunks = (a.Cin + BK - 1) / BK;
    for (int tile : {(int)TILE_64x64_K64, (int)TILE_128x64_K64, (int)TILE_128x128_K64, (int)TILE_256x128_K64}) {
        const TileInfo &t = TILES[tile];
        for (int ks : {2, 3, 4, 6, 8}) {
            const int per = (chunks + 2 * ks - 1) / (2 * ks) * 2;             // whole 64-channel steps
            const int ranges = (chunks + per - 1) / per;
            if (ranges != ks || (size_t)ks * M * a.Nout * sizeof(float) > room) continue;
            const double est = t.cost[a.TR * a.TS == 1 ? 0 : 1].t0 + tile_work(a, tile, per / 2 * a.TR * a.TS) * tiles_per_cu(t.per_cu, tile_count(t, M, a.Nout) * ks) +
                               4.0 + 8.0 * ks * M * a.Nout / 8e6;
            if (est < us) { us = est; pl = IgemmPlan{tile, ks, per}; }
        }
    }
    return pl;
}

size_t igemm_split_bytes(const IgemmArgs &a)
{
    if (a.Cin % 8 != 0 || thin_rows_applicable(a) || thin_cols_applicable(a)) return 0;
    const IgemmPlan pl = make_plan(a, SIZE_MAX);
    return pl.ksplits > 1 ? (size_t)pl.ksplits * a.NB * a.OH * a.OW * a.Nout * sizeof(float) : 0;
}

bool igemm_accepts_transposed_b(const IgemmArgs &a)
{
    return a.Cin % 8 == 0 && a.Nout % 8 == 0 && !(forced_cfg() < 0 && thin_rows_applicable(a)) && choose_c_outer(a);
}

template <class T>
static hipError_t dispatch(const IgemmArgs &a, hipStream_t stream)
{
    const int64_t M = (int64_t)a.NB * a.OH * a.OW;
    if (forced_cfg() < 0 && thin_rows_applicable(a)) return launch_thin_rows(a, std::is_same<T, BF16>::value, stream);
    if (forced_cfg() < 0 && thin_cols_applicable(a)) return launch_thin_cols(a, std::is_same<T, BF16>::value, stream);
    if (a.Cin % 8 != 0) {
        const int64_t tiles = ((M + 127) / 128) * ((a.Nout + 63) / 64);
        if (tiles <= 0 || tiles > 0x7fffffff) return hipErrorInvalidValue;
        DLK_LAUNCH("igemm_scalar_kernel", igemm_scalar_kernel<T>, dim3((unsigned)tiles), dim3(256), 0, stream, a);
        return dlk::launch_status();
    }
    constexpr bool bf16 = std::is_same<T, BF16>::value;
    IgemmArgs b = a;
    set_divisors(b);
    b.c_outer = choose_c_outer(a);
    b.ksplits = 1;
    b.split_chunks = 0;
    const IgemmPlan pl = make_plan(a, a.part ? a.part_bytes : 0);
    if (pl.ksplits > 1) {
        b.ksplits = pl.ksplits;
        b.split_chunks = pl.chunks;
        hipError_t e = launch_igemm_dma(b, bf16, pl.tile, stream);
        if (e != hipSuccess) return e;
        return launch_splitk_reduce_tail(a.part, pl.ksplits, M * a.Nout, a.D, bf16 ? 1 : 0, a.bias, a.relu, a.Nout, a.resid, stream);
    }
    // whole reduction in one step: before the choice between ring tiles, which all spend three or four steps on it
    if (b.c_outer && forced_cfg() < 0 && igemm_short_applicable(b)) return launch_igemm_short(b, bf16, stream);
    // A short last column tile (e.g. 304 = 256 + 48 output channels) would run mostly empty: where two launches are estimated
    // to take less than one, the remainder gets a narrower tile.
    const int rem = a.Nout % 256;
    if (forced_cfg() < 0 && a.Nout > 256 && rem != 0 && rem <= 128) {
        IgemmArgs lo = b, hi = b;
        lo.Nout = a.Nout - rem;
        hi.Nout = rem;
        double whole = 0, us_lo = 0, us_hi = 0;
        best_tile(b, &whole);
        const int t_lo = best_tile(lo, &us_lo), t_hi = best_tile(hi, &us_hi);
        if (us_lo + us_hi < whole) {
            if (a.b_transposed) hi.b_base = a.b_base + lo.Nout;
            else hi.B = a.B + (size_t)lo.Nout * a.TR * a.TS * a.Cin;
            hi.D = a.D + lo.Nout;
            if (a.bias) hi.bias = a.bias + lo.Nout;
            if (a.resid) hi.resid = a.resid + lo.Nout;
            hipError_t e = launch_igemm_dma(lo, bf16, t_lo, stream);
            if (e != hipSuccess) return e;
            return launch_igemm_dma(hi, bf16, t_hi, stream);
        }
    }
    return launch_igemm_dma(b, bf16, pl.tile, stream);
}

int igemm_batch_cfg(const IgemmArgs *a, int n)
{
    if (n < 2 || n > IgemmBatch::MAX || forced_cfg() >= 0) return -1;
    for (int i = 0; i < n; ++i)
        if (a[i].Cin % 8 != 0 || thin_rows_applicable(a[i]) || thin_cols_applicable(a[i]) || !choose_c_outer(a[i]) || a[i].b_transposed != a[0].b_transposed)
            return -1;
    // one tile for all: the tiles of all GEMMs together, each with the work of its own reduction
    int best = -1;
    double best_us = 0;
    for (int tile : {(int)TILE_64x32, (int)TILE_64x64, (int)TILE_128x64_K64, (int)TILE_128x128, (int)TILE_256x256}) {
        const TileInfo &t = TILES[tile];
        int64_t tiles = 0;
        double work = 0;
        for (int i = 0; i < n; ++i) {
            const int64_t own = tile_count(t, (int64_t)a[i].NB * a[i].OH * a[i].OW, a[i].Nout);
            tiles += own;
            work += own * tile_work(a[i], tile, tile_steps(a[i], tile));
        }
        const bool considered = tile == TILE_64x32 ? a[0].Nout <= 32 : true;
        const double us = t.cost[1].t0 + work / tiles * tiles_per_cu(t.per_cu, tiles);
        if (considered && (best < 0 || us < best_us)) { best = tile; best_us = us; }
    }
    return best;
}

hipError_t launch_igemm_batch(const IgemmBatch &b, bool is_bf16, hipStream_t stream)
{
    const int cfg = igemm_batch_cfg(b.a, b.n);
    if (cfg < 0) return hipErrorInvalidValue;
    IgemmBatch c = b;
    std::sort(c.a, c.a + c.n, [](const IgemmArgs &x, const IgemmArgs &y) { return x.TR * x.TS > y.TR * y.TS; });
    for (int i = 0; i < c.n; ++i) {
        set_divisors(c.a[i]);
        c.a[i].c_outer = 1;
        c.a[i].ksplits = 1;
        c.a[i].split_chunks = 0;
        c.a[i].part = nullptr;
    }
    return launch_igemm_dma_batch(c, is_bf16, cfg, stream);
}

hipError_t launch_igemm(const IgemmArgs &a, bool is_bf16, hipStream_t stream)
{
    return is_bf16 ? dispatch<BF16>(a, stream) : dispatch<F16>(a, stream);
}

// ---- filter re-layout for the data gradient -------------------------------
__global__ void filter_relayout_kernel(const FilterRelayoutArgs p)
{
    const int64_t total = (int64_t)p.C * p.TR * p.TS * p.K;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        int64_t t = i;
        const int k = (int)(t % p.K); t /= p.K;
        const int js = (int)(t % p.TS); t /= p.TS;
        const int jr = (int)(t % p.TR); t /= p.TR;
        const int c = (int)t;
        const int r = p.r0 + jr * p.rstep, s = p.s0 + js * p.sstep;
        p.wt[i] = p.w[(((int64_t)k * p.R + r) * p.S + s) * p.C + c];
    }
}

// Zero fill of the input-gradient pixels that no filter tap reaches (a 1x1 filter with stride 2 reads one pixel
// in four): pixel (h, w) belongs to stride-parity class (h % sh) * sw + (w % sw); the classes whose bit is set in
// `mask` are cleared, 16 bytes per thread, all of them in one sweep over the tensor (C % 8 == 0).
__global__ __launch_bounds__(256) void zero_classes_kernel(uint16_t *__restrict__ dx, int64_t pieces, int H, int W, int C8, int sh,
                                                           int sw, uint64_t mask)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < pieces; i += (int64_t)gridDim.x * 256) {
        const int64_t pix = i / C8;
        const int w = (int)(pix % W), h = (int)((pix / W) % H);
        if ((mask >> ((h % sh) * sw + (w % sw))) & 1) *reinterpret_cast<u32x4_t *>(dx + i * 8) = u32x4_t{0, 0, 0, 0};
    }
}

hipError_t launch_zero_classes(uint16_t *dx, int N, int H, int W, int C, int sh, int sw, uint64_t mask, hipStream_t stream)
{
    if (C % 8 != 0 || sh < 1 || sw < 1 || sh * sw > 64) return hipErrorInvalidValue;
    const int64_t pieces = (int64_t)N * H * W * (C / 8);
    if (pieces <= 0 || mask == 0) return hipSuccess;
    const int64_t want = (pieces + 256 * 8 - 1) / (256 * 8);          // about eight pieces per thread
    const dim3 grid((unsigned)(want < 65535 ? want : 65535)), block(256);
    DLK_LAUNCH("zero_classes_kernel", zero_classes_kernel, grid, block, 0, stream, dx, pieces, H, W, C / 8, sh, sw, mask);
    return dlk::launch_status();
}

// Channel padding for the kernels that move 16-byte pieces: one piece of eight channels per thread, assembled from
// 2-byte loads (neighbouring threads read neighbouring elements, the cache makes whole lines of them).
__global__ __launch_bounds__(256) void pad_channels_kernel(const uint16_t *__restrict__ src, uint16_t *__restrict__ dst, int64_t pieces,
                                                           const uint16_t *__restrict__ src2, uint16_t *__restrict__ dst2,
                                                           int64_t pieces2, int C)
{
    const int C8 = (C + 7) / 8;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < pieces + pieces2; i += (int64_t)gridDim.x * 256) {
        const bool second = i >= pieces;
        const int64_t j = second ? i - pieces : i;
        const int64_t row = j / C8;
        const int c0 = (int)(j - row * C8) * 8;
        const uint16_t *from = (second ? src2 : src) + row * C + c0;
        u32x4_t v;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t lo = c0 + 2 * d < C ? from[2 * d] : 0u, hi = c0 + 2 * d + 1 < C ? from[2 * d + 1] : 0u;
            v[d] = lo | (hi << 16);
        }
        *reinterpret_cast<u32x4_t *>((second ? dst2 : dst) + j * 8) = v;
    }
}

hipError_t launch_pad_channels(const uint16_t *src, uint16_t *dst, int64_t rows, const uint16_t *src2, uint16_t *dst2,
                               int64_t rows2, int C, hipStream_t stream)
{
    const int64_t C8 = (C + 7) / 8, pieces = rows * C8, pieces2 = rows2 * C8, want = (pieces + pieces2 + 255) / 256;
    if (want <= 0) return hipSuccess;
    const dim3 grid((unsigned)(want < 16384 ? want : 16384)), block(256);
    DLK_LAUNCH("pad_channels_kernel", pad_channels_kernel, grid, block, 0, stream, src, dst, pieces, src2, dst2, pieces2, C);
    return dlk::launch_status();
}

hipError_t launch_filter_relayout(const FilterRelayoutArgs &a, hipStream_t stream)
{
    const int64_t total = (int64_t)a.C * a.TR * a.TS * a.K;
    if (total <= 0) return hipSuccess;
    const int blocks = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
    DLK_LAUNCH("filter_relayout_kernel", filter_relayout_kernel, dim3(blocks), dim3(256), 0, stream, a);
    return dlk::launch_status();
}

}  // namespace dlk
