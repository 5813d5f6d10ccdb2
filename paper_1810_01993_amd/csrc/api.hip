// C boundary: argument validation, workspace sizing, and the mapping of the
// three convolution passes and the loss onto the gfx950 kernels.  Everything
// here runs on the host; validation happens before any launch.
#include <algorithm>
#include <cmath>
#include <hip/hip_runtime.h>

#include "../../include/dlconv.h"
#include "kernels.h"

namespace dlk {
thread_local LaunchLog *launch_log = nullptr;
}

namespace {

constexpr int64_t MAX_ELEMS = 0x7FF00000;     // 32-bit byte offsets, with room above for the out-of-range marker

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int gcd(int a, int b) { while (b) { int t = a % b; a = b; b = t; } return a; }

struct Geometry {
    int32_t P, Q;
    int64_t x_elems, w_elems, y_elems;
};

dl_status check_desc(const dl_conv_desc *d, Geometry *g)
{
    if (!d) return DL_ERR_NULL;
    if (d->N < 1 || d->H < 1 || d->W < 1 || d->C < 1 || d->K < 1 || d->R < 1 || d->S < 1) return DL_ERR_SHAPE;
    if (d->stride_h < 1 || d->stride_w < 1 || d->dil_h < 1 || d->dil_w < 1 || d->pad_h < 0 || d->pad_w < 0)
        return DL_ERR_SHAPE;
    if (d->dtype != DL_F16 && d->dtype != DL_BF16) return DL_ERR_DTYPE;
    if (d->dw_dtype != d->dtype && d->dw_dtype != DL_F32) return DL_ERR_DTYPE;
    const int64_t span_h = (int64_t)d->H + 2 * (int64_t)d->pad_h - (int64_t)d->dil_h * (d->R - 1) - 1;
    const int64_t span_w = (int64_t)d->W + 2 * (int64_t)d->pad_w - (int64_t)d->dil_w * (d->S - 1) - 1;
    if (span_h < 0 || span_w < 0) return DL_ERR_SHAPE;
    const int64_t P = span_h / d->stride_h + 1, Q = span_w / d->stride_w + 1;
    // padded coordinates and tensor sizes must fit the kernels' 32-bit index math
    if ((int64_t)d->H + 2 * (int64_t)d->pad_h >= MAX_ELEMS || (int64_t)d->W + 2 * (int64_t)d->pad_w >= MAX_ELEMS)
        return DL_ERR_SHAPE;
    const int64_t xe = (int64_t)d->N * d->H * d->W;
    const int64_t ye = (int64_t)d->N * P * Q;
    const int64_t we = (int64_t)d->R * d->S * d->C;
    if (xe >= MAX_ELEMS || ye >= MAX_ELEMS || we >= MAX_ELEMS) return DL_ERR_SHAPE;
    if (xe * d->C >= MAX_ELEMS || ye * d->K >= MAX_ELEMS || we * d->K >= MAX_ELEMS) return DL_ERR_SHAPE;
    g->P = (int32_t)P;
    g->Q = (int32_t)Q;
    g->x_elems = xe * d->C;
    g->y_elems = ye * d->K;
    g->w_elems = we * d->K;
    return DL_OK;
}

// Taps of one axis that reach input positions congruent to `a` modulo the
// stride: r = r0 + j*rstep, j < count, and the output position they read is
// (pos/stride-class index) + t0 + j*dt.
struct AxisTaps { int r0, rstep, count, t0, dt; };

AxisTaps class_taps(int a, int R, int stride, int pad, int dil)
{
    AxisTaps t{0, 1, 0, 0, 0};
    t.rstep = stride / gcd(dil, stride);
    int r0 = -1;
    for (int r = 0; r < R && r < t.rstep; ++r)
        if (((a + pad - r * dil) % stride + stride) % stride == 0) { r0 = r; break; }
    if (r0 < 0) return t;                               // no tap reaches this class
    t.r0 = r0;
    t.count = (R - 1 - r0) / t.rstep + 1;
    t.t0 = (a + pad - r0 * dil) / stride;               // exact by construction
    t.dt = -(t.rstep * dil) / stride;                   // exact: rstep*dil is a multiple of stride
    return t;
}

// ---- one implicit GEMM, with a halo-tile kernel where one applies -------------
// Where the coefficients of the GEMM's filter operand live in the caller's
// filter tensor: element (row j, tap (jr, js), reduction channel c) is
// src[base + j*sj + jr*sr + js*ss + c*sc].
struct FilterSrc { const uint16_t *src; int64_t base, sj, sr, ss, sc; };

// Scratch one implicit GEMM needs: the blocked filter copy of a halo kernel, or the fp32 partial
// sums of a split reduction of the plain engine (never both).  least: the fewest bytes it runs with (the plain engine splits
// less, or not at all, in less room).
size_t igemm_scratch_bytes(const dlk::IgemmArgs &a, bool least = false)
{
    if (!dlk::igemm_halo_takes(a)) return least ? 0 : align_up(dlk::igemm_split_bytes(a), 256);
    // (the 5x5 kernel for at most 32 output channels may split its reduction on small maps: partial sums behind the copy)
    const size_t part = dlk::igemm_narrow5x5_applicable(a) ? align_up(dlk::igemm_narrow5x5_split_bytes(a), 256) : 0;
    return align_up(dlk::igemm_blocked_filter_bytes(a), 256) + part;
}

// a.B: plain [Nout][taps*Cin] filter (may be null if a halo kernel takes the GEMM).
// room: bytes at scratch.
hipError_t run_igemm(const dlk::IgemmArgs &a, bool bf16, const FilterSrc &fs, uint16_t *scratch, size_t room, hipStream_t stream)
{
    if (!dlk::igemm_halo_takes(a)) {
        dlk::IgemmArgs g = a;
        g.part = room > 0 ? reinterpret_cast<float *>(scratch) : nullptr;
        g.part_bytes = room;
        return dlk::launch_igemm(g, bf16, stream);
    }
    dlk::FilterBlockArgs f{};
    f.src = fs.src; f.dst = scratch;
    f.base = fs.base; f.sj = fs.sj; f.sr = fs.sr; f.ss = fs.ss; f.sc = fs.sc;
    f.Nrows = a.Nout; f.TR = a.TR; f.TS = a.TS; f.Cin = a.Cin;
    const hipError_t e = dlk::launch_filter_block(f, stream);
    if (e != hipSuccess) return e;
    dlk::IgemmArgs h = a;
    h.B = scratch;
    h.part = reinterpret_cast<float *>(reinterpret_cast<char *>(scratch) + align_up(dlk::igemm_blocked_filter_bytes(h), 256));
    return dlk::launch_igemm_halo(h, bf16, stream);
}

// ---- channel counts that are not a multiple of 8 -------------------------------
// The kernels that move 16-byte pieces need C % 8 == 0; the element-wise ones are up to 10 times slower.
// So the activation tensor (and the forward filter) may first be copied with its channels padded with zeros, and the
// layer runs on the copy: 361 x 577 x 6 -> 64, 7x7 stride 2, batch 2: forward 56 -> 28 us, filter gradient 148 -> 35 us,
// 5 us of either being the copy; 60 x 90 x 100 -> 64, 3x3: 92 -> 14 us and 41 -> 20 us.  Which layers gain from it:
// fwd_copies_pay, wgrad_padded_workspace.  Zero channels meet zero coefficients, so the sums are those of the layer itself.
inline dl_conv_desc padded_desc(const dl_conv_desc *d)
{
    dl_conv_desc e = *d;
    e.C = (d->C + 7) / 8 * 8;
    return e;
}
inline size_t padded_bytes(const dl_conv_desc *e, int64_t rows) { return align_up((size_t)rows * e->C * sizeof(uint16_t), 256); }

dlk::IgemmArgs fwd_args(const dl_conv_desc *d, const Geometry &g)
{
    dlk::IgemmArgs a{};
    a.NB = d->N; a.IH = d->H; a.IW = d->W; a.Cin = d->C;
    a.OH = g.P; a.OW = g.Q; a.Nout = d->K;
    a.TR = d->R; a.TS = d->S;
    a.sh = d->stride_h; a.sw = d->stride_w;
    a.th0 = -d->pad_h; a.dth = d->dil_h; a.tw0 = -d->pad_w; a.dtw = d->dil_w;
    a.FH = g.P; a.FW = g.Q; a.osh = 1; a.osw = 1; a.ooh = 0; a.oow = 0; a.ldd = d->K;
    return a;
}

// 16 x 16 output patches of a layer, the unit of the stem's kernels.
int64_t stem_patches(const dl_conv_desc *d, const Geometry &g) { return (int64_t)d->N * ((g.P + 15) / 16) * ((g.Q + 15) / 16); }

// The stem's forward kernel (no residual input there).  One patch per compute unit is always worth it; every further round costs
// 2.3..5.8 us however little of its patches is inside the image, the plain engine 0.09..0.16 us per thousand pixels, so many
// maps that are narrow or small stay with that one: 306 x 1 x 566, 16 -> 16: 63.8 us, 13.8 there (4800 random layers; filled
// patches, 65000 pixels a round, are never among them).
bool use_stem_fwd(const dl_conv_desc *d, const Geometry &g)
{
    if (!dlk::stem_fwd_applicable(d->C, d->K, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w, d->dil_h, d->dil_w)) return false;
    const int64_t round_pixels = d->C == 8 ? (d->K > 32 ? 33000 : 22000) : d->K > 32 ? 45000 : 33000;
    return (int64_t)d->N * g.P * g.Q >= round_pixels * ((stem_patches(d, g) - 1) / 256);
}

// Whether the forward pass of d gains from the channel-padded copies, on which it is the GEMM a of the layer e.  The lines
// come from 9000 random layers timed both ways (fp16, C 1..400, 1..256 outputs, maps of 8 x 8 to 768 x 1500).
bool fwd_copies_pay(const dl_conv_desc *d, const dl_conv_desc *e, const dlk::IgemmArgs &a)
{
    const int64_t taps = (int64_t)d->R * d->S, red = taps * d->C;
    // the stem's kernel: 361 x 577 x 6 -> 64, batch 2: 56 us without the copies, 21 with them; one channel left as it was
    if (use_stem_fwd(e, Geometry{a.OH, a.OW, 0, 0, 0}) && !a.resid) return d->C > 1;
    if (red <= 24) return false;                         // 60 x 90 x 17 -> 64, 1x1: 9.1 us, 9.9 through the copy
    const int64_t steps = (red + 31) / 32;               // of the element-wise kernel
    const int64_t strides = (int64_t)d->stride_h * d->stride_w;
    // estimated times in us; the copy reads and writes all of x, also the pixels that a stride leaves out
    const double m = (double)a.NB * a.OH * a.OW, pix = (double)d->N * d->H * d->W, tiles = std::ceil(m / 128) * std::ceil(d->K / 64.0);
    const double copy = 2.0 * pix * (d->C + e->C) / 4.3e6;
    const double filled = d->K / (64.0 * std::ceil(d->K / 64.0));
    const double fetched = taps > 1 || strides == 1 ? 2.0 * pix * d->C : std::min(2.0 * pix * d->C, m * std::ceil(d->C / 32.0 + 1) * 64);
    const double own = 5.0 + 2.6 * steps + std::max(0.0, tiles - 155) * steps * (5.1e-3 + 2.1e-3 * filled) * (1 + 0.36 * std::min(1.0, fetched / 3e8));
    if (taps == 1) {
        // the one-step kernel: 1.2-2.2x with stride 1; with stride 2 0.8x on 27 channels and 96 or 128 outputs, 1.2-1.8x on 256
        if (dlk::igemm_short_applicable(a)) return strides == 1 || d->K >= 192;
        // else by the estimates (8-9 % off): 506 x 512 x 299 -> 1, stride 2, batch 2: 74 us without the copy, 197 with it
        const double cols = d->K <= 32 ? 32 : std::ceil(d->K / 64.0) * 64;
        const double lines = std::min(2.0 * pix * e->C, m * std::ceil(e->C / 64.0) * 128);
        const double padded = 5.9 + copy + 0.14 * std::ceil(e->C / 32.0) + std::max(m * cols * e->C * 6.4e-9, (2.0 * m * d->K + lines) / 3.4e6);
        return own > 1.03 * padded;
    }
    // More taps: the copy has to be small beside the element-wise kernel's work (786 x 475 x 9 -> 12, 2x2 stride 2, batch 2:
    // 21 us without, 28 with it), and the padded reduction may not have too many steps of 32 against that kernel's;
    // a halo kernel takes whole 32-channel chunks of every tap.
    if (copy > 1.0 && own < (steps == 1 ? 6 : steps <= 3 ? 4 : 2) * copy) return false;
    if (!dlk::igemm_halo_takes(a)) return 2 * ((taps * e->C + 31) / 32) <= 7 * steps;
    // 3x3, measured with 3..13 channels: 64 outputs 0.7-1.0x up to 5 channels, 1.0-1.1x with 6 and 7; at most 16 outputs
    // 0.6-0.97x up to 10 channels, 1.0-1.2x with 11; above 64 outputs 0.98x and more from 4 channels on (dilated 0.6-0.8x
    // with 6 and 7)
    const bool dense3 = d->R == 3 && d->S == 3 && d->dil_h == 1 && d->dil_w == 1;
    if (taps <= 9) return red >= (!dense3 ? 90 : d->K > 64 ? 36 : d->K > 16 ? 54 : 99);
    // 5x5: 0.5-0.9x with one channel; up to 32 outputs 1.1-1.4x with two; above that 0.8-1.2x with two, 0.9-1.3x with three;
    // 7x7: 0.43x with one, 0.74x with three, 1.3x with five
    return taps * ((e->C + 31) / 32) <= (d->K > 32 ? 9 : 13) * steps;
}

// Scratch of a forward pass on the channel-padded copies (0: the layer takes its own tensors): the copies, then what
// the implicit GEMM on them needs.  Layers that the streaming kernel for few channels takes stay with it.
size_t fwd_padded_workspace(const dl_conv_desc *d, const Geometry &g, bool resid)
{
    if (d->C % 8 == 0 || dlk::thin_rows_applicable(fwd_args(d, g))) return 0;
    const dl_conv_desc e = padded_desc(d);
    Geometry ge;
    if (check_desc(&e, &ge) != DL_OK) return 0;              // the copy would exceed the index range
    dlk::IgemmArgs a = fwd_args(&e, ge);
    a.resid = resid ? reinterpret_cast<const uint16_t *>(uintptr_t(16)) : nullptr;      // only tested for null
    if (!fwd_copies_pay(d, &e, a)) return 0;
    return padded_bytes(&e, (int64_t)d->N * d->H * d->W) + padded_bytes(&e, (int64_t)d->K * d->R * d->S) +
           igemm_scratch_bytes(a);
}

// The data gradient of one stride-parity class (ca, cb) of the input pixels.
struct DgradClass {
    dlk::IgemmArgs args;        // pointers unset
    AxisTaps th, tw;
    bool empty, has_taps;
    size_t wt_bytes, blk_bytes;
};

DgradClass dgrad_class(const dl_conv_desc *d, const Geometry &g, int ca, int cb, bool least = false)
{
    DgradClass c{};
    const int OH = ca < d->H ? (d->H - ca + d->stride_h - 1) / d->stride_h : 0;
    const int OW = cb < d->W ? (d->W - cb + d->stride_w - 1) / d->stride_w : 0;
    c.th = class_taps(ca, d->R, d->stride_h, d->pad_h, d->dil_h);
    c.tw = class_taps(cb, d->S, d->stride_w, d->pad_w, d->dil_w);
    c.empty = OH == 0 || OW == 0;
    c.has_taps = c.th.count > 0 && c.tw.count > 0;
    c.wt_bytes = align_up((size_t)d->C * c.th.count * c.tw.count * d->K * sizeof(uint16_t), 256);
    dlk::IgemmArgs &a = c.args;
    a.NB = d->N; a.IH = g.P; a.IW = g.Q; a.Cin = d->K;
    a.OH = OH; a.OW = OW; a.Nout = d->C;
    a.TR = c.has_taps ? c.th.count : 0; a.TS = c.has_taps ? c.tw.count : 1;
    a.sh = 1; a.sw = 1;
    a.th0 = c.th.t0; a.dth = c.th.dt; a.tw0 = c.tw.t0; a.dtw = c.tw.dt;
    a.FH = d->H; a.FW = d->W; a.osh = d->stride_h; a.osw = d->stride_w; a.ooh = ca; a.oow = cb;
    a.ldd = d->C;
    c.blk_bytes = (c.empty || !c.has_taps) ? 0 : igemm_scratch_bytes(a, least);
    return c;
}

bool use_dgrad_stem(const dl_conv_desc *d)
{
    return dlk::dgrad_stem_applicable(d->N, d->H, d->W, d->C, d->K, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w,
                                      d->dil_h, d->dil_w);
}

size_t dgrad_stem_workspace(const dl_conv_desc *d) { return align_up(dlk::dgrad_stem_filter_bytes(d->C, d->K), 256); }

// least: the fewest bytes it runs with
size_t dgrad_workspace(const dl_conv_desc *d, const Geometry &g, bool stem, bool least = false)
{
    if (stem) return dgrad_stem_workspace(d);
    size_t total = 0;
    for (int ca = 0; ca < d->stride_h; ++ca)
        for (int cb = 0; cb < d->stride_w; ++cb) {
            const DgradClass c = dgrad_class(d, g, ca, cb, least);
            total += c.wt_bytes + c.blk_bytes;
        }
    return total;
}

bool use_wgrad3x3(const dl_conv_desc *d)
{
    return dlk::wgrad3x3_applicable(d->N, d->H, d->W, d->C, d->K, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w,
                                    d->dil_h, d->dil_w);
}

bool use_wgrad5x5(const dl_conv_desc *d)
{
    return dlk::wgrad5x5_applicable(d->N, d->H, d->W, d->C, d->K, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w,
                                    d->dil_h, d->dil_w);
}

// (not for a few pixels of 16 channels and less than 32 outputs: setting up its image takes longer than the general kernel does;
// 8 x 8 x 16 -> 8: 10.3 us, 7.3 there)
bool use_wgrad_stem(const dl_conv_desc *d, const Geometry &g)
{
    if (d->C == 16 && d->K < 32 && (int64_t)d->N * g.P * g.Q < 64) return false;
    return dlk::wgrad_stem_applicable(d->C, d->K, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w, d->dil_h, d->dil_w);
}

// Patches that lie mostly outside narrow or small maps: the stem's filter gradient multiplies all of each, and writes a slice of
// partial sums per patch up to 256.  Both kernels' times as fitted to 4100 random layers (us; the general one's is its planner's estimate with
// its deviation on this filter): 188 x 2 x 56, 16 -> 40: 27.0 us, 13.4 on the general kernel.
bool stem_patches_filled(const dl_conv_desc *d, const Geometry &g)
{
    const int64_t patches = stem_patches(d, g);
    return patches <= 2 || (int64_t)d->N * g.P * g.Q >= patches * (d->C == 8 ? 96 : 192);
}

bool wgrad_stem_pays(const dl_conv_desc *d, const Geometry &g, int splits, const dlk::WgradPlan &general)
{
    if (general.cfg < 0) return true;
    const int64_t patches = stem_patches(d, g);
    const double run = (double)((patches + splits - 1) / splits), sums = 1e-6 * splits * g.w_elems;
    return d->C == 8 ? 6.4 + 2.1 * run + 2.8 * sums <= 1.14 * general.us - 4.3 : 8.25 + 2.85 * run + 2.0 * sums <= 1.07 * general.us - 3.6;
}

// Plan of the kernels that serve any layer, for a workspace of `room` bytes.  A caller that brings fewer bytes than the
// preferred plan takes (say, the size that an earlier version of the library asked for) gets as many slices as they hold, down
// to *least.
dlk::WgradPlan wgrad_general_plan(const dl_conv_desc *d, const Geometry &g, size_t room, int *least)
{
    const int64_t npix = (int64_t)d->N * g.P * g.Q;
    const int RSC = d->R * d->S * d->C;
    const bool thin = dlk::thin_wgrad_applicable(d->K, d->C, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w);
    const dlk::WgradPlan best = dlk::wgrad_make_plan(npix, g.x_elems, d->K, d->C, RSC, thin, true, INT64_MAX);
    const size_t slice = (size_t)g.w_elems * sizeof(float);
    *least = best.splits;
    if (best.cfg < 0 || (room != 0 && best.splits * slice <= room)) return best;
    *least = std::min(best.splits, dlk::wgrad_least_slices(npix, g.x_elems, d->K, d->C, RSC));
    const int64_t fit = (int64_t)(room / slice);
    return fit < *least ? best : dlk::wgrad_make_plan(npix, g.x_elems, d->K, d->C, RSC, thin, false, fit);  // (too little: the caller refuses)
}

dlk::WgradPlan wgrad_plan(const dl_conv_desc *d, const Geometry &g, size_t room = SIZE_MAX)
{
    if (use_wgrad5x5(d)) {
        const dlk::WgradStripPlan p5 = dlk::wgrad5x5_make_plan(d->N, d->H, d->W, d->C, d->K);
        return dlk::WgradPlan{-4, p5.slices, 0, 0, 0};
    }
    if (use_wgrad3x3(d)) {
        const dlk::WgradStripPlan p3 = dlk::wgrad3x3_make_plan(d->N, d->H, d->W, d->C, d->K);
        return dlk::WgradPlan{-3, p3.slices, 0, 0, 0};
    }
    const bool stem = use_wgrad_stem(d, g);
    const int splits = stem ? dlk::wgrad_stem_splits(d->N, d->K, g.P, g.Q) : 0;
    const size_t slice = (size_t)g.w_elems * sizeof(float);
    const dlk::WgradPlan stem_plan{-5, splits, 0, 0, 0};
    if (stem && splits * slice <= room && stem_patches_filled(d, g)) return stem_plan;
    int least;
    const dlk::WgradPlan general = wgrad_general_plan(d, g, room, &least);
    // (the stem's also where there is room for its slices alone)
    if (stem && splits * slice <= room && (wgrad_stem_pays(d, g, splits, general) || general.splits * slice > room)) return stem_plan;
    return general;
}

size_t wgrad_own_workspace(const dl_conv_desc *d, const Geometry &g, size_t room = SIZE_MAX)
{
    return (size_t)wgrad_plan(d, g, room).splits * (size_t)g.w_elems * sizeof(float);
}

// The fewest bytes a filter gradient runs with.
size_t wgrad_least_workspace(const dl_conv_desc *d, const Geometry &g)
{
    const dlk::WgradPlan best = wgrad_plan(d, g);
    int least = best.splits;
    if (best.cfg >= 0 || best.cfg == -5) {
        wgrad_general_plan(d, g, 0, &least);
        least = std::min(least, best.splits);
        if (use_wgrad_stem(d, g)) least = std::min(least, dlk::wgrad_stem_splits(d->N, d->K, g.P, g.Q));
    }
    return (size_t)least * (size_t)g.w_elems * sizeof(float);
}

// As fwd_padded_workspace, for the filter gradient: partial sums of the padded filter, then the copy of x.
size_t wgrad_padded_workspace(const dl_conv_desc *d, const Geometry &g)
{
    if (d->C % 8 == 0) return 0;
    const dl_conv_desc e = padded_desc(d);
    Geometry ge;
    if (check_desc(&e, &ge) != DL_OK) return 0;
    // only where the copy gets a faster kernel, and never instead of the streaming kernel for few output channels
    if (wgrad_plan(d, g).cfg != -1 || wgrad_plan(&e, ge).cfg == -1) return 0;
    // A 1x1 layer with a stride has all of x copied and reads a part of it: the copy (4.3 TB/s) has to take less than seven
    // tenths of what the element-wise kernel's tiles take (5e-4 us per pixel of a 128 x 128 tile).  501 x 962 x 242 -> 64,
    // stride 2, batch 2: 244 us without, 325 with it; 659 x 1209 x 141 -> 48: 389 and 312 us.
    if (d->R * d->S == 1 && d->stride_h * d->stride_w > 1) {
        const double copy = 2.0 * d->N * d->H * d->W * (d->C + e.C) / 4.3e6;
        const double tiles = 5e-4 * ((d->K + 127) / 128) * ((d->C + 127) / 128) * d->N * g.P * g.Q;
        if (copy > 3.0 + 0.7 * tiles) return 0;
    }
    return align_up(wgrad_own_workspace(&e, ge), 256) + padded_bytes(&e, (int64_t)d->N * d->H * d->W);
}

size_t wgrad_workspace(const dl_conv_desc *d, const Geometry &g)
{
    return std::max(wgrad_own_workspace(d, g), wgrad_padded_workspace(d, g));
}

dl_status hip_status(hipError_t e) { return e == hipSuccess ? DL_OK : DL_ERR_LAUNCH; }

}  // namespace

extern "C" {

dl_status dl_logits_ce_workspace_bytes(int64_t n_pixels, int32_t C, size_t *bytes)
{
    if (!bytes) return DL_ERR_NULL;
    if (n_pixels < 0 || C < 32 || C > 2048 || C % 8 != 0) return DL_ERR_SHAPE;
    const size_t blocks = (size_t)dlk::logits_ce_blocks(n_pixels, C);
    *bytes = align_up(blocks * 3 * (size_t)C * sizeof(float), 256) + align_up(blocks * sizeof(float), 256);
    return DL_OK;
}

dl_status logits_ce_fused_fwd_bwd(const void *x, const void *w, int32_t dtype, const uint8_t *labels,
                                  const float *class_weights, float scale, int64_t n_pixels, int32_t C, void *logits,
                                  float *loss, void *dlogits, void *dx, void *dw, int32_t dw_dtype, void *workspace,
                                  size_t workspace_bytes, void *hip_stream)
{
    if (!w || !class_weights || !loss || !dw) return DL_ERR_NULL;
    if (n_pixels < 0 || C < 32 || C > 2048 || C % 8 != 0 || n_pixels >= MAX_ELEMS / C) return DL_ERR_SHAPE;
    if (n_pixels > 0 && (!x || !labels || !dx)) return DL_ERR_NULL;
    if ((dtype != DL_F16 && dtype != DL_BF16) || (dw_dtype != dtype && dw_dtype != DL_F32)) return DL_ERR_DTYPE;
    if (!aligned16(x) || !aligned16(w) || !aligned16(dx) || !aligned16(dw)) return DL_ERR_ALIGN;
    size_t need = 0;
    dl_logits_ce_workspace_bytes(n_pixels, C, &need);
    if (!workspace || workspace_bytes < need) return DL_ERR_WORKSPACE;
    if (!aligned16(workspace)) return DL_ERR_ALIGN;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int blocks = dlk::logits_ce_blocks(n_pixels, C);
    dlk::LogitsCeArgs a{};
    a.x = static_cast<const uint16_t *>(x);
    a.w = static_cast<const uint16_t *>(w);
    a.labels = labels;
    a.cw = class_weights;
    a.scale = scale;
    a.n = n_pixels;
    a.C = C;
    a.logits = static_cast<uint16_t *>(logits);
    a.dlogits = static_cast<uint16_t *>(dlogits);
    a.dx = static_cast<uint16_t *>(dx);
    a.partial_dw = static_cast<float *>(workspace);
    a.partial_loss = reinterpret_cast<float *>(static_cast<char *>(workspace) + align_up((size_t)blocks * 3 * C * sizeof(float), 256));
    if (dlk::launch_logits_ce(a, dtype == DL_BF16, stream) != hipSuccess) return DL_ERR_LAUNCH;
    if (dlk::launch_splitk_reduce(a.partial_dw, blocks, (int64_t)3 * C, dw, dw_dtype, stream) != hipSuccess) return DL_ERR_LAUNCH;
    return hip_status(dlk::launch_ce_finish(a.partial_loss, blocks, scale, loss, stream));
}

const char *dl_status_string(dl_status s)
{
    switch (s) {
        case DL_OK: return "ok";
        case DL_ERR_NULL: return "null pointer";
        case DL_ERR_SHAPE: return "invalid shape";
        case DL_ERR_DTYPE: return "unsupported dtype";
        case DL_ERR_ALIGN: return "tensor base not 16-byte aligned";
        case DL_ERR_WORKSPACE: return "workspace missing or too small";
        case DL_ERR_UNSUPPORTED: return "unsupported configuration";
        case DL_ERR_LAUNCH: return "HIP launch failed";
    }
    return "unknown status";
}

dl_status dl_conv_out_shape(const dl_conv_desc *desc, int32_t *P, int32_t *Q)
{
    if (!desc || !P || !Q) return DL_ERR_NULL;
    Geometry g;
    const dl_status st = check_desc(desc, &g);
    if (st != DL_OK) return st;
    *P = g.P;
    *Q = g.Q;
    return DL_OK;
}

dl_status dl_conv_workspace_bytes(const dl_conv_desc *desc, int pass, size_t *bytes)
{
    if (!desc || !bytes) return DL_ERR_NULL;
    Geometry g;
    const dl_status st = check_desc(desc, &g);
    if (st != DL_OK) return st;
    switch (pass) {
        case DL_PASS_FWD: {
            // with a residual input some kernels are not available and the choice of scratch changes: enough for either
            dlk::IgemmArgs a = fwd_args(desc, g);
            const size_t plain = igemm_scratch_bytes(a);
            a.resid = reinterpret_cast<const uint16_t *>(uintptr_t(16));     // any non-null value: only tested for null
            *bytes = std::max({plain, igemm_scratch_bytes(a), fwd_padded_workspace(desc, g, false), fwd_padded_workspace(desc, g, true)});
            return DL_OK;
        }
        case DL_PASS_BWD_DATA: *bytes = dgrad_workspace(desc, g, use_dgrad_stem(desc)); return DL_OK;
        case DL_PASS_BWD_FILTER: *bytes = wgrad_workspace(desc, g); return DL_OK;
    }
    return DL_ERR_UNSUPPORTED;
}

dl_status dl_conv_least_workspace_bytes(const dl_conv_desc *desc, int pass, size_t *bytes)
{
    if (!bytes) return DL_ERR_NULL;
    Geometry g;
    const dl_status st = check_desc(desc, &g);
    if (st != DL_OK) return st;
    switch (pass) {
        case DL_PASS_FWD: {
            dlk::IgemmArgs a = fwd_args(desc, g);
            const size_t plain = igemm_scratch_bytes(a, true);
            a.resid = reinterpret_cast<const uint16_t *>(uintptr_t(16));
            *bytes = std::max(plain, igemm_scratch_bytes(a, true));
            return DL_OK;
        }
        case DL_PASS_BWD_DATA:
            *bytes = dgrad_workspace(desc, g, use_dgrad_stem(desc), true);
            if (desc->C % 8 != 0) *bytes = std::min(*bytes, dgrad_workspace(desc, g, false, true));
            return DL_OK;
        case DL_PASS_BWD_FILTER: *bytes = wgrad_least_workspace(desc, g); return DL_OK;
    }
    return DL_ERR_UNSUPPORTED;
}

namespace {
dl_status run_fwd(const dl_conv_desc *d, const void *x, const void *w, const float *bias, const void *residual, int relu,
                  void *y, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!d || !x || !w || !y) return DL_ERR_NULL;
    if (residual && !aligned16(residual)) return DL_ERR_ALIGN;
    Geometry g;
    const dl_status st = check_desc(d, &g);
    if (st != DL_OK) return st;
    if (!aligned16(x) || !aligned16(w) || !aligned16(y)) return DL_ERR_ALIGN;
    if (bias && (reinterpret_cast<uintptr_t>(bias) & 3u)) return DL_ERR_ALIGN;
    dlk::IgemmArgs a = fwd_args(d, g);
    a.resid = static_cast<const uint16_t *>(residual);    // decides which kernels may take the launch
    const size_t need = igemm_scratch_bytes(a, true);
    if (need > 0 && (!workspace || workspace_bytes < need)) return DL_ERR_WORKSPACE;
    if (need > 0 && !aligned16(workspace)) return DL_ERR_ALIGN;
    if (!residual && use_stem_fwd(d, g)) {
        dlk::StemFwdArgs f{};
        f.x = static_cast<const uint16_t *>(x);
        f.w = static_cast<const uint16_t *>(w);
        f.y = static_cast<uint16_t *>(y);
        f.N = d->N; f.H = d->H; f.W = d->W; f.C = d->C; f.K = d->K; f.P = g.P; f.Q = g.Q;
        f.bias = bias;
        f.relu = relu ? 1 : 0;
        return hip_status(dlk::launch_stem_fwd(f, d->dtype == DL_BF16, static_cast<hipStream_t>(hip_stream)));
    }
    // (a workspace too small for the copies, or none, still runs the layer on its own tensors)
    const size_t padded = fwd_padded_workspace(d, g, residual != nullptr);
    if (padded > 0 && workspace && workspace_bytes >= padded && aligned16(workspace)) {
        const dl_conv_desc e = padded_desc(d);
        const int64_t xrows = (int64_t)d->N * d->H * d->W, wrows = (int64_t)d->K * d->R * d->S;
        char *const xp = static_cast<char *>(workspace), *const wp = xp + padded_bytes(&e, xrows);
        if (dlk::launch_pad_channels(static_cast<const uint16_t *>(x), reinterpret_cast<uint16_t *>(xp), xrows,
                                     static_cast<const uint16_t *>(w), reinterpret_cast<uint16_t *>(wp), wrows, d->C,
                                     static_cast<hipStream_t>(hip_stream)) != hipSuccess)
            return DL_ERR_LAUNCH;
        const size_t used = padded_bytes(&e, xrows) + padded_bytes(&e, wrows);
        return run_fwd(&e, xp, wp, bias, residual, relu, y, xp + used, padded - used, hip_stream);
    }
    a.A = static_cast<const uint16_t *>(x);
    a.B = static_cast<const uint16_t *>(w);
    a.D = static_cast<uint16_t *>(y);
    a.bias = bias;
    a.relu = relu ? 1 : 0;
    const FilterSrc fs{a.B, 0, (int64_t)d->R * d->S * d->C, (int64_t)d->S * d->C, d->C, 1};
    const size_t room = workspace && aligned16(workspace) ? workspace_bytes : 0;
    return hip_status(run_igemm(a, d->dtype == DL_BF16, fs, static_cast<uint16_t *>(workspace), room,
                                static_cast<hipStream_t>(hip_stream)));
}
}  // namespace

dl_status conv2d_fwd(const dl_conv_desc *d, const void *x, const void *w, void *y, void *workspace,
                     size_t workspace_bytes, void *hip_stream)
{
    return run_fwd(d, x, w, nullptr, nullptr, 0, y, workspace, workspace_bytes, hip_stream);
}

dl_status conv2d_fwd_bias_relu(const dl_conv_desc *d, const void *x, const void *w, const float *bias, int32_t relu,
                               void *y, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_fwd(d, x, w, bias, nullptr, relu, y, workspace, workspace_bytes, hip_stream);
}

dl_status conv2d_fwd_bias_add_relu(const dl_conv_desc *d, const void *x, const void *w, const float *bias,
                                   const void *residual, int32_t relu, void *y, void *workspace, size_t workspace_bytes,
                                   void *hip_stream)
{
    return run_fwd(d, x, w, bias, residual, relu, y, workspace, workspace_bytes, hip_stream);
}

dl_status conv2d_bwd_data(const dl_conv_desc *d, const void *dy, const void *w, void *dx, void *workspace,
                          size_t workspace_bytes, void *hip_stream)
{
    if (!d || !dy || !w || !dx) return DL_ERR_NULL;
    Geometry g;
    const dl_status st = check_desc(d, &g);
    if (st != DL_OK) return st;
    if (!aligned16(dy) || !aligned16(w) || !aligned16(dx)) return DL_ERR_ALIGN;
    // the stem kernel's filter copy is rounded up to 32 output channels: for channel counts that the general path served
    // from fewer bytes, those bytes are still enough
    const bool stem = use_dgrad_stem(d) && (d->C % 8 == 0 || (workspace && workspace_bytes >= dgrad_stem_workspace(d)));
    const size_t need = dgrad_workspace(d, g, stem, true);
    if (need > 0 && (!workspace || workspace_bytes < need)) return DL_ERR_WORKSPACE;
    if (need > 0 && !aligned16(workspace)) return DL_ERR_ALIGN;
    // what there is beyond that is for partial sums; only without strides is a class dense, and so its reduction ever split
    const size_t spare = d->stride_h == 1 && d->stride_w == 1 ? workspace_bytes - need : 0;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const bool bf16 = d->dtype == DL_BF16;

    if (stem) {
        // few input channels, 7x7 stride 2: all parity classes in one workgroup, operands resident in LDS
        dlk::FilterBlockArgs f{};
        f.src = static_cast<const uint16_t *>(w);
        f.dst = static_cast<uint16_t *>(workspace);
        f.base = 0; f.sj = 1; f.sr = (int64_t)d->S * d->C; f.ss = d->C; f.sc = (int64_t)d->R * d->S * d->C;
        f.Nrows = d->C; f.TR = d->R; f.TS = d->S; f.Cin = d->K;
        if (dlk::launch_filter_block(f, stream) != hipSuccess) return DL_ERR_LAUNCH;
        dlk::DgradStemArgs a{};
        a.dy = static_cast<const uint16_t *>(dy);
        a.wblk = f.dst;
        a.dx = static_cast<uint16_t *>(dx);
        a.N = d->N; a.H = d->H; a.W = d->W; a.C = d->C; a.K = d->K; a.P = g.P; a.Q = g.Q;
        return hip_status(dlk::launch_dgrad_stem(a, bf16, stream));
    }

    // Input pixels (h, w) fall into stride_h*stride_w parity classes; within a
    // class the contributing taps and the output pixels they pair with form
    // regular grids, so each class is one dense implicit GEMM over dy with the
    // filter re-laid-out as [c][tap][k].  Classes that take the plain engine with
    // one tile shape share a launch (longest reductions first, so that its end is
    // short); the others are launched one by one.
    struct Pending { dlk::IgemmArgs a; FilterSrc fs; uint16_t *blk; size_t room; };
    Pending pending[dlk::IgemmBatch::MAX];
    int n_pending = 0;
    bool overflow = false;
    size_t ws_off = 0;
    // classes that no tap reaches (e.g. three of the four of a 1x1 stride-2 layer) are all zeros: one fill for all
    uint64_t zero_mask = 0;
    if (d->C % 8 == 0 && d->stride_h * d->stride_w <= 64) {
        for (int ca = 0; ca < d->stride_h; ++ca)
            for (int cb = 0; cb < d->stride_w; ++cb) {
                const DgradClass c = dgrad_class(d, g, ca, cb, true);
                if (!c.empty && !c.has_taps) zero_mask |= 1ull << (ca * d->stride_w + cb);
            }
        if (zero_mask && dlk::launch_zero_classes(static_cast<uint16_t *>(dx), d->N, d->H, d->W, d->C, d->stride_h, d->stride_w,
                                                  zero_mask, stream) != hipSuccess)
            return DL_ERR_LAUNCH;
    }
    for (int ca = 0; ca < d->stride_h; ++ca)
        for (int cb = 0; cb < d->stride_w; ++cb) {
            DgradClass c = dgrad_class(d, g, ca, cb, true);
            uint16_t *wt = reinterpret_cast<uint16_t *>(static_cast<char *>(workspace) + ws_off);
            uint16_t *blk = reinterpret_cast<uint16_t *>(static_cast<char *>(workspace) + ws_off + c.wt_bytes);
            ws_off += c.wt_bytes + c.blk_bytes;
            const size_t room = c.blk_bytes + spare;
            if (c.empty || ((zero_mask >> (ca * d->stride_w + cb)) & 1)) continue;
            dlk::IgemmArgs &a = c.args;
            a.A = static_cast<const uint16_t *>(dy);
            a.D = static_cast<uint16_t *>(dx);
            a.B = static_cast<const uint16_t *>(w);     // never read when there are no taps
            const bool halo = c.has_taps && dlk::igemm_halo_takes(a);
            const int64_t SC = (int64_t)d->S * d->C;
            // the plain engine can take the filter as it lies in memory (reduction-major for this GEMM)
            const bool direct = c.has_taps && !halo && dlk::igemm_accepts_transposed_b(a);
            if (direct) {
                a.b_transposed = 1;
                a.b_base = (int32_t)(c.th.r0 * SC + (int64_t)c.tw.r0 * d->C);
                a.b_sr = (int32_t)(c.th.rstep * SC);
                a.b_ss = (int32_t)((int64_t)c.tw.rstep * d->C);
                a.b_ldk = (int32_t)((int64_t)d->R * SC);
                a.b_elems = (int32_t)g.w_elems;
            } else if (c.has_taps && !halo) {
                dlk::FilterRelayoutArgs f{};
                f.w = static_cast<const uint16_t *>(w);
                f.wt = wt;
                f.K = d->K; f.R = d->R; f.S = d->S; f.C = d->C;
                f.r0 = c.th.r0; f.rstep = c.th.rstep; f.TR = c.th.count;
                f.s0 = c.tw.r0; f.sstep = c.tw.rstep; f.TS = c.tw.count;
                if (dlk::launch_filter_relayout(f, stream) != hipSuccess) return DL_ERR_LAUNCH;
                a.B = wt;
            }
            const FilterSrc fs{static_cast<const uint16_t *>(w), c.th.r0 * SC + (int64_t)c.tw.r0 * d->C, 1,
                               c.th.rstep * SC, (int64_t)c.tw.rstep * d->C, (int64_t)d->R * SC};
            if (c.has_taps && !halo && !overflow) {
                if (n_pending < dlk::IgemmBatch::MAX) {
                    pending[n_pending++] = Pending{a, fs, blk, room};
                    continue;
                }
                overflow = true;                        // more classes than one launch holds: one by one after all
            }
            if (run_igemm(a, bf16, fs, blk, room, stream) != hipSuccess) return DL_ERR_LAUNCH;
        }
    if (n_pending > 0) {
        dlk::IgemmBatch b{};
        b.n = n_pending;
        for (int i = 0; i < n_pending; ++i) b.a[i] = pending[i].a;
        if (!overflow && dlk::igemm_batch_cfg(b.a, b.n) >= 0) {
            if (dlk::launch_igemm_batch(b, bf16, stream) != hipSuccess) return DL_ERR_LAUNCH;
        } else {
            for (int i = 0; i < n_pending; ++i)
                if (run_igemm(pending[i].a, bf16, pending[i].fs, pending[i].blk, pending[i].room, stream) != hipSuccess) return DL_ERR_LAUNCH;
        }
    }
    return DL_OK;
}

namespace {
// dw_c: channels of dw itself, smaller than d->C where d describes a channel-padded copy
dl_status run_wgrad(const dl_conv_desc *d, const Geometry &g, const dlk::WgradPlan &plan, const void *x, const void *dy, void *dw,
                    int dw_c, void *workspace, hipStream_t stream)
{
    dlk::WgradArgs a{};
    a.x = static_cast<const uint16_t *>(x);
    a.dy = static_cast<const uint16_t *>(dy);
    a.partial = static_cast<float *>(workspace);
    a.N = d->N; a.H = d->H; a.W = d->W; a.C = d->C; a.K = d->K; a.R = d->R; a.S = d->S; a.P = g.P; a.Q = g.Q;
    a.sh = d->stride_h; a.sw = d->stride_w; a.ph = d->pad_h; a.pw = d->pad_w; a.dh = d->dil_h; a.dw = d->dil_w;
    a.splits = plan.splits;
    a.chunk = plan.chunk;
    a.spread = plan.spread;
    hipError_t e;
    if (plan.cfg == -3) {
        const dlk::WgradStripPlan p3 = dlk::wgrad3x3_make_plan(d->N, d->H, d->W, d->C, d->K);
        dlk::WgradStripArgs w{};
        w.x = a.x; w.dy = a.dy; w.partial = a.partial;
        w.N = d->N; w.H = d->H; w.W = d->W; w.C = d->C; w.K = d->K;
        w.slices = p3.slices; w.rs = p3.rs; w.xs = p3.xs;
        e = dlk::launch_wgrad3x3(w, d->dtype == DL_BF16, stream);
    } else if (plan.cfg == -4) {
        const dlk::WgradStripPlan p5 = dlk::wgrad5x5_make_plan(d->N, d->H, d->W, d->C, d->K);
        dlk::WgradStripArgs w{};
        w.x = a.x; w.dy = a.dy; w.partial = a.partial;
        w.N = d->N; w.H = d->H; w.W = d->W; w.C = d->C; w.K = d->K;
        w.slices = p5.slices; w.rs = p5.rs; w.xs = p5.xs;
        e = dlk::launch_wgrad5x5(w, d->dtype == DL_BF16, stream);
    } else if (plan.cfg == -5) {
        dlk::WgradStemArgs w{};
        w.x = a.x; w.dy = a.dy; w.partial = a.partial;
        w.N = d->N; w.H = d->H; w.W = d->W; w.C = d->C; w.K = d->K; w.P = g.P; w.Q = g.Q;
        w.splits = plan.splits;
        e = dlk::launch_wgrad_stem(w, d->dtype == DL_BF16, stream);
    } else
    e = plan.cfg >= 0    ? dlk::launch_wgrad_dma(a, d->dtype == DL_BF16, plan.cfg, stream)
                   : plan.cfg == -2 ? dlk::launch_thin_wgrad(a, d->dtype == DL_BF16, stream)
                                    : dlk::launch_wgrad(a, d->dtype == DL_BF16, stream);
    if (e != hipSuccess) return DL_ERR_LAUNCH;
    if (dw_c != d->C)
        return hip_status(dlk::launch_splitk_reduce_padded(a.partial, plan.splits, g.w_elems / d->C, dw_c, d->C, dw, d->dw_dtype, stream));
    e = dlk::launch_splitk_reduce(a.partial, plan.splits, g.w_elems, dw, d->dw_dtype, stream);
    return hip_status(e);
}
}  // namespace

dl_status conv2d_bwd_filter(const dl_conv_desc *d, const void *x, const void *dy, void *dw, void *workspace,
                            size_t workspace_bytes, void *hip_stream)
{
    if (!d || !x || !dy || !dw) return DL_ERR_NULL;
    Geometry g;
    const dl_status st = check_desc(d, &g);
    if (st != DL_OK) return st;
    if (!aligned16(x) || !aligned16(dy) || !aligned16(dw)) return DL_ERR_ALIGN;
    const dlk::WgradPlan plan = wgrad_plan(d, g, workspace_bytes);
    if (!workspace || workspace_bytes < (size_t)plan.splits * (size_t)g.w_elems * sizeof(float)) return DL_ERR_WORKSPACE;
    if (!aligned16(workspace)) return DL_ERR_ALIGN;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const size_t padded = wgrad_padded_workspace(d, g);
    if (padded > 0 && workspace_bytes >= padded) {
        const dl_conv_desc e = padded_desc(d);
        Geometry ge;
        check_desc(&e, &ge);
        char *const xp = static_cast<char *>(workspace) + align_up(wgrad_own_workspace(&e, ge), 256);
        if (dlk::launch_pad_channels(static_cast<const uint16_t *>(x), reinterpret_cast<uint16_t *>(xp), (int64_t)d->N * d->H * d->W,
                                     nullptr, nullptr, 0, d->C, stream) != hipSuccess)
            return DL_ERR_LAUNCH;
        return run_wgrad(&e, ge, wgrad_plan(&e, ge), xp, dy, dw, d->C, workspace, stream);
    }
    return run_wgrad(d, g, plan, x, dy, dw, d->C, workspace, stream);
}


dl_status dl_conv_describe(const dl_conv_desc *d, int pass, char *buf, size_t buf_bytes)
{
    if (!d || !buf) return DL_ERR_NULL;
    if (buf_bytes < 2) return DL_ERR_SHAPE;
    Geometry g;
    const dl_status st = check_desc(d, &g);
    if (st != DL_OK) return st;
    if (pass != DL_PASS_FWD && pass != DL_PASS_BWD_DATA && pass != DL_PASS_BWD_FILTER) return DL_ERR_UNSUPPORTED;
    // The entry point itself runs, on stand-in addresses that only pointer arithmetic ever touches,
    // with every launch turned into a log line.
    void *const a = reinterpret_cast<void *>(uintptr_t(1) << 40);
    void *const b = reinterpret_cast<void *>(uintptr_t(2) << 40);
    void *const c = reinterpret_cast<void *>(uintptr_t(3) << 40);
    void *const ws = reinterpret_cast<void *>(uintptr_t(4) << 40);
    size_t ws_bytes = 0;
    dl_conv_workspace_bytes(d, pass, &ws_bytes);
    dlk::LaunchLog log;
    dlk::launch_log = &log;
    dl_status r;
    if (pass == DL_PASS_FWD) r = conv2d_fwd(d, a, b, c, ws, ws_bytes, nullptr);
    else if (pass == DL_PASS_BWD_DATA) r = conv2d_bwd_data(d, a, b, c, ws, ws_bytes, nullptr);
    else r = conv2d_bwd_filter(d, a, b, c, ws, ws_bytes, nullptr);
    dlk::launch_log = nullptr;
    if (r != DL_OK) return r;
    const size_t n = log.text.size() < buf_bytes - 1 ? log.text.size() : buf_bytes - 1;
    log.text.copy(buf, n);
    buf[n] = 0;
    return DL_OK;
}

// The transposed convolution and its two gradients are the three passes of the underlying
// convolution with the operand roles exchanged: the layer's input stands where that
// convolution's output gradient stands, its output where the data gradient stands.
dl_status conv2d_transpose_fwd(const dl_conv_desc *d, const void *x, const void *w, void *y, void *workspace,
                               size_t workspace_bytes, void *hip_stream)
{
    return conv2d_bwd_data(d, x, w, y, workspace, workspace_bytes, hip_stream);
}

dl_status conv2d_transpose_bwd_data(const dl_conv_desc *d, const void *dy, const void *w, void *dx, void *workspace,
                                    size_t workspace_bytes, void *hip_stream)
{
    return conv2d_fwd(d, dy, w, dx, workspace, workspace_bytes, hip_stream);
}

dl_status conv2d_transpose_bwd_filter(const dl_conv_desc *d, const void *x, const void *dy, void *dw,
                                      void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return conv2d_bwd_filter(d, dy, x, dw, workspace, workspace_bytes, hip_stream);
}

dl_status dl_bias_relu_bwd_workspace_bytes(int64_t n_pixels, int32_t K, size_t *bytes)
{
    if (!bytes) return DL_ERR_NULL;
    if (n_pixels < 0 || K < 1 || n_pixels * K >= MAX_ELEMS) return DL_ERR_SHAPE;
    *bytes = (size_t)dlk::tail_bwd_blocks(n_pixels, K) * K * sizeof(float);
    return DL_OK;
}

dl_status bias_relu_bwd(const void *dy, const void *y, int32_t dtype, int64_t n_pixels, int32_t K, int32_t relu,
                        void *dz, float *dbias, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!dbias) return DL_ERR_NULL;
    if (n_pixels < 0 || K < 1 || n_pixels * K >= MAX_ELEMS) return DL_ERR_SHAPE;
    if (n_pixels > 0 && (!dy || (relu && (!y || !dz)))) return DL_ERR_NULL;
    if (dtype != DL_F16 && dtype != DL_BF16) return DL_ERR_DTYPE;
    if (!aligned16(dy) || !aligned16(y) || !aligned16(dz) || (reinterpret_cast<uintptr_t>(dbias) & 3u)) return DL_ERR_ALIGN;
    // a smaller workspace than the query asks for gives longer slabs, down to a least number of them
    const size_t row = (size_t)K * sizeof(float);
    if (!workspace || workspace_bytes < dlk::tail_bwd_least_blocks(n_pixels, K) * row) return DL_ERR_WORKSPACE;
    if (!aligned16(workspace)) return DL_ERR_ALIGN;
    dlk::TailBwdArgs a{};
    a.rows = (int32_t)std::min<size_t>(dlk::tail_bwd_blocks(n_pixels, K), workspace_bytes / row);
    a.dy = static_cast<const uint16_t *>(dy);
    a.y = static_cast<const uint16_t *>(y);
    a.dz = static_cast<uint16_t *>(dz);
    a.partial = static_cast<float *>(workspace);
    a.dbias = dbias;
    a.npix = n_pixels;
    a.K = K;
    a.relu = relu ? 1 : 0;
    return hip_status(dlk::launch_tail_bwd(a, dtype == DL_BF16, static_cast<hipStream_t>(hip_stream)));
}

dl_status dl_larc_workspace_bytes(int32_t n_tensors, size_t *bytes)
{
    if (!bytes) return DL_ERR_NULL;
    if (n_tensors < 0) return DL_ERR_SHAPE;
    *bytes = (size_t)n_tensors * dlk::LARC_SLICES * 2 * sizeof(float);
    return DL_OK;
}

dl_status larc_sgd_step(const dl_larc_tensor *tensors, int32_t n_tensors, int32_t grad_dtype, float lr, float trust,
                        float weight_decay, float momentum, float eps, int32_t clip, float *rates, void *workspace,
                        size_t workspace_bytes, void *hip_stream)
{
    if (n_tensors < 0) return DL_ERR_SHAPE;
    if (n_tensors == 0) return DL_OK;
    if (!tensors) return DL_ERR_NULL;
    if (grad_dtype != DL_F16 && grad_dtype != DL_BF16 && grad_dtype != DL_F32) return DL_ERR_DTYPE;
    for (int i = 0; i < n_tensors; ++i) {
        if (!tensors[i].w || !tensors[i].g) return DL_ERR_NULL;
        if (tensors[i].count < 1 || tensors[i].count >= MAX_ELEMS) return DL_ERR_SHAPE;
        if ((reinterpret_cast<uintptr_t>(tensors[i].w) & 3u) || (reinterpret_cast<uintptr_t>(tensors[i].v) & 3u) ||
            (reinterpret_cast<uintptr_t>(tensors[i].g) & (grad_dtype == DL_F32 ? 3u : 1u)))
            return DL_ERR_ALIGN;
        if (momentum != 0.f && !tensors[i].v) return DL_ERR_NULL;
    }
    const size_t need = (size_t)n_tensors * dlk::LARC_SLICES * 2 * sizeof(float);
    if (!workspace || workspace_bytes < need) return DL_ERR_WORKSPACE;
    if (!aligned16(workspace)) return DL_ERR_ALIGN;
    for (int first = 0; first < n_tensors; first += dlk::LARC_MAX) {
        dlk::LarcBatch b{};
        b.n = n_tensors - first < dlk::LARC_MAX ? n_tensors - first : dlk::LARC_MAX;
        for (int i = 0; i < b.n; ++i) {
            const dl_larc_tensor &t = tensors[first + i];
            b.t[i] = dlk::LarcTensor{static_cast<float *>(t.w), t.g, momentum != 0.f ? static_cast<float *>(t.v) : nullptr,
                                     t.count};
        }
        b.partial = static_cast<float *>(workspace);
        b.rates = rates;
        b.lr = lr; b.trust = trust; b.wd = weight_decay; b.momentum = momentum; b.eps = eps;
        b.clip = clip ? 1 : 0;
        b.first = first;
        if (dlk::launch_larc(b, grad_dtype, static_cast<hipStream_t>(hip_stream)) != hipSuccess) return DL_ERR_LAUNCH;
    }
    return DL_OK;
}

dl_status dl_ce_workspace_bytes(int64_t n_pixels, size_t *bytes)
{
    if (!bytes) return DL_ERR_NULL;
    if (n_pixels < 0) return DL_ERR_SHAPE;
    *bytes = (size_t)dlk::ce_num_blocks(n_pixels) * sizeof(float);
    return DL_OK;
}

namespace {
dl_status run_ce(const void *logits, int32_t dtype, const uint8_t *labels, const float *weights, bool per_pixel,
                 float scale, int64_t n_pixels, float *loss, void *dlogits, void *workspace, size_t workspace_bytes,
                 void *hip_stream)
{
    if (!loss || (!weights && (!per_pixel || n_pixels > 0))) return DL_ERR_NULL;
    if (n_pixels < 0 || n_pixels >= MAX_ELEMS * 16) return DL_ERR_SHAPE;
    if (n_pixels > 0 && (!logits || !labels || !dlogits)) return DL_ERR_NULL;
    if (dtype != DL_F16 && dtype != DL_BF16) return DL_ERR_DTYPE;
    if (!aligned16(logits) || !aligned16(labels) || !aligned16(dlogits) || (per_pixel && !aligned16(weights)))
        return DL_ERR_ALIGN;
    const size_t need = (size_t)dlk::ce_num_blocks(n_pixels) * sizeof(float);
    if (!workspace || workspace_bytes < need) return DL_ERR_WORKSPACE;
    if (!aligned16(workspace)) return DL_ERR_ALIGN;
    return hip_status(dlk::launch_weighted_ce(static_cast<const uint16_t *>(logits), dtype == DL_BF16, labels, weights,
                                              per_pixel, scale, n_pixels, loss, static_cast<uint16_t *>(dlogits),
                                              static_cast<float *>(workspace), static_cast<hipStream_t>(hip_stream)));
}
}  // namespace

dl_status weighted_pixel_ce_fwd_bwd(const void *logits, int32_t dtype, const uint8_t *labels,
                                    const float *class_weights, float scale, int64_t n_pixels, float *loss,
                                    void *dlogits, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_ce(logits, dtype, labels, class_weights, false, scale, n_pixels, loss, dlogits, workspace,
                  workspace_bytes, hip_stream);
}

dl_status weighted_pixel_ce_fwd_bwd_static(const void *logits, int32_t dtype, const uint8_t *labels,
                                           const float *class_weights, float scale, int64_t n_pixels, float *loss,
                                           void *dlogits, void *hip_stream)
{
    // the same checks as the entry point with a workspace, then the size limit of this one
    if (!loss || !class_weights) return DL_ERR_NULL;
    if (n_pixels < 0 || n_pixels > DL_CE_STATIC_MAX_PIXELS) return DL_ERR_SHAPE;
    if (n_pixels > 0 && (!logits || !labels || !dlogits)) return DL_ERR_NULL;
    if (dtype != DL_F16 && dtype != DL_BF16) return DL_ERR_DTYPE;
    if (!aligned16(logits) || !aligned16(labels) || !aligned16(dlogits)) return DL_ERR_ALIGN;
    float *partials = nullptr;
    if (dlk::ce_static_partials(&partials) != hipSuccess) return DL_ERR_LAUNCH;
    return hip_status(dlk::launch_weighted_ce(static_cast<const uint16_t *>(logits), dtype == DL_BF16, labels, class_weights,
                                              false, scale, n_pixels, loss, static_cast<uint16_t *>(dlogits), partials,
                                              static_cast<hipStream_t>(hip_stream)));
}

dl_status weighted_pixel_ce_map_fwd_bwd(const void *logits, int32_t dtype, const uint8_t *labels,
                                        const float *weight_map, float scale, int64_t n_pixels, float *loss,
                                        void *dlogits, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_ce(logits, dtype, labels, weight_map, true, scale, n_pixels, loss, dlogits, workspace, workspace_bytes,
                  hip_stream);
}

}  // extern "C"
