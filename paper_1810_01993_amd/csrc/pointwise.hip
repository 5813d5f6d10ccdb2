// Backward of the point-wise tail of a convolution layer, y = max(s + bias[k], 0), in one
// streaming pass over the [pixels][K] tensors:
//   dz[i][k]  = dy[i][k] where y[i][k] > 0, else 0     (the gradient the convolution's own
//                                                       data- and filter-gradient kernels take)
//   dbias[k]  = sum over pixels of dz[i][k]
// 6 bytes of traffic per element (dy and y in, dz out) instead of the 10 of a masking pass
// followed by a column-sum pass.  A thread owns VEC consecutive channels (8 = one 16-byte
// access, or 1 for channel counts that are not a multiple of 8) and walks down the pixels of
// its workgroup's slab with fp32 running sums; the pixel lanes of a workgroup are then added
// in a fixed order through LDS, every workgroup writes one fp32 partial row, and the ordered
// reduce kernel adds the rows: the result does not depend on timing.
//
// Bound by memory once enough loads are in flight: a workgroup covers at most 256 channels where they are
// whole 128-byte lines (so it has at least eight pixel lanes of 16-byte pieces; see tail_bwd_shape), a thread has four pixels' loads in flight, and on small maps it gets no more than those four
// pixels.  Measured (fp16 / bf16, before -> after; before, a thread had two pixels in flight and at least 32
// pixels to itself, which put 27 workgroups on the smallest of these): 6912 x 1024 32.0 -> 11.6 us (3.7 TB/s),
// 6912 x 256 21.2 -> 5.3 us, 110592 x 256 48.3 -> 32.3 us (5.3 TB/s), 110592 x 64 25.8 -> 13.7 us.
// dz is stored without the non-temporal hint of the loads, since the convolution gradients read it next, unless it
// exceeds what the last-level cache (256 MB) could keep of it: 884736 x 256 (453 MB) 273 us without, 263 with;
// 442368 x 256 (226 MB) 119 and 135.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace dlk {

constexpr int TB_THREADS = 256;

// How the [npix][K] tensor is dealt to workgroups: columns of workgroups side by side, gpb channel groups x lanes
// pixel lanes in each.
struct TailBwdShape { int groups, columns, gpb, lanes; };
static TailBwdShape tail_bwd_split(int K, int vec, int cap, bool even)
{
    TailBwdShape s;
    s.groups = (K + vec - 1) / vec;
    s.columns = (s.groups + cap - 1) / cap;
    s.gpb = even ? (s.groups + s.columns - 1) / s.columns : s.groups < cap ? s.groups : cap;
    s.lanes = TB_THREADS / s.gpb;
    return s;
}

// Without 16-byte pieces a workgroup of 256 channels has one pixel lane: from 4 M elements on (8 M without ReLU, where
// nothing is stored) it covers at most 64 (four and more lanes), and consecutive workgroups of an XCD take the columns of
// one slab side by side, so that the pieces of a 128-byte line that two of them write meet in its L2.  Measured (ReLU,
// against 256 channels): 442368 x 257 559 -> 330 us, 1000000 x 100 357 -> 199 us; below the line 3015 x 257 8.8 us, 9.4
// with 64.
//
// With 16-byte pieces a column is 256 channels wide where they are whole 128-byte lines (K % 64 == 0), and on tensors of
// less than 16 M elements.  Other rows share lines with their neighbours wherever they are cut: up to 512 channels they
// are not cut, wider ones into columns of at most 512 channels, interleaved as above.  Measured (fp16, ReLU; columns of
// 256 channels -> now): 884736 x 304 481 -> 311 us (5.2 TB/s), 442368 x 520 430 -> 345 us, 110592 x 520 89 -> 74 us,
// 442368 x 1160 936 -> 789 us; below the line 3015 x 304 8.7 us, 9.3 with one column.
static bool tail_bwd_large(const TailBwdArgs &a)
{
    return a.K % 64 != 0 && a.npix * a.K >= (a.K % 8 == 0 ? 1 << 24 : a.relu ? 1 << 22 : 1 << 23);
}
static TailBwdShape tail_bwd_shape(const TailBwdArgs &a)
{
    const int vec = a.K % 8 == 0 ? 8 : 1;
    return tail_bwd_large(a) ? tail_bwd_split(a.K, vec, 64, true) : tail_bwd_split(a.K, vec, TB_THREADS / vec, false);
}

// STREAM: dz is stored past the caches.  INTERLEAVE: see tail_bwd_shape (a template parameter: as an argument, its load is one
// more round trip before a workgroup begins, 0.2 us of the 5-14 us launches).
template <class T, int VEC, bool STREAM, bool INTERLEAVE>
__global__ __launch_bounds__(TB_THREADS) void tail_bwd_kernel(const TailBwdArgs p)
{
    __shared__ __align__(16) float red[TB_THREADS * VEC];
    __shared__ float part[TB_THREADS];
    int slab = blockIdx.x, column = blockIdx.y;
    if constexpr (INTERLEAVE) {                                     // the grid is one row of workgroups
        const int slot = blockIdx.x / 8;
        column = slot % p.columns;
        slab = slot / p.columns * 8 + blockIdx.x % 8;
        if (slab >= p.rows) return;                                 // the whole workgroup
    }
    const int gl = threadIdx.x % p.gpb, pl = threadIdx.x / p.gpb;
    const int g = column * p.gpb + gl;
    const bool active = pl < p.lanes && g < p.groups;
    const int k0 = g * VEC;
    const int64_t begin = (int64_t)slab * p.chunk, end = min(p.npix, begin + p.chunk);
    float sum[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) sum[e] = 0.f;
    if (active) {
        using Piece = std::conditional_t<VEC == 8, u32x4_t, uint16_t>;
        // (an element's line is read by many threads, at different times: the hint that it is not needed again is for
        // whole pieces only)
        auto load = [&](const uint16_t *src, size_t off) {
            const Piece *q = reinterpret_cast<const Piece *>(src + off);
            if constexpr (VEC == 8) return __builtin_nontemporal_load(q);
            else return *q;
        };
        auto one = [&](Piece gv, Piece yv, size_t off) {
            if constexpr (VEC == 8) {
                if (p.relu) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t lo = T::to_float((uint16_t)(yv[d] & 0xffffu)) > 0.f ? 0xffffu : 0u;
                        const uint32_t hi = T::to_float((uint16_t)(yv[d] >> 16)) > 0.f ? 0xffff0000u : 0u;
                        gv[d] &= lo | hi;
                    }
                    if constexpr (STREAM) __builtin_nontemporal_store(gv, reinterpret_cast<Piece *>(p.dz + off));
                    else *reinterpret_cast<Piece *>(p.dz + off) = gv;
                }
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    sum[2 * d] += T::to_float((uint16_t)(gv[d] & 0xffffu));
                    sum[2 * d + 1] += T::to_float((uint16_t)(gv[d] >> 16));
                }
            } else {
                if (p.relu) {
                    if (!(T::to_float(yv) > 0.f)) gv = 0;
                    p.dz[off] = gv;
                }
                sum[0] += T::to_float(gv);
            }
        };
        const size_t step = (size_t)p.lanes * p.K;
        size_t off = (size_t)(begin + pl) * p.K + k0;
        int64_t i = begin + pl;
        for (; i + 3 * p.lanes < end; i += 4 * p.lanes, off += 4 * step) {
            Piece gv[4], yv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) gv[u] = load(p.dy, off + u * step);
            if (p.relu) {
#pragma unroll
                for (int u = 0; u < 4; ++u) yv[u] = load(p.y, off + u * step);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) yv[u] = Piece{};
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) one(gv[u], yv[u], off + u * step);
        }
        for (; i < end; i += p.lanes, off += step) {
            const Piece gv = load(p.dy, off);
            one(gv, p.relu ? load(p.y, off) : Piece{}, off);
        }
    }
    // Pixel lanes of a channel, added in a fixed order: the channels of the workgroup are dealt to the threads,
    // up to 16 threads per channel with a contiguous range of pixel lanes each, then those parts in ascending order.
    const int cols = p.gpb * VEC;
    if (pl < p.lanes) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) red[threadIdx.x * VEC + e] = sum[e];      // row pl, column gl * VEC + e
    }
    __syncthreads();
    if (cols > TB_THREADS) {                                        // up to seven pixel lanes: a thread adds whole channels
        for (int col = threadIdx.x; col < cols; col += TB_THREADS) {
            const int k = column * cols + col;
            float s = 0.f;
            for (int l = 0; l < p.lanes; ++l) s += red[l * cols + col];
            if (k < p.K) p.partial[(size_t)slab * p.K + k] = s;
        }
        return;
    }
    const int parts = min(16, TB_THREADS / cols), per = (p.lanes + parts - 1) / parts;
    const int col = threadIdx.x % cols, q = threadIdx.x / cols;
    float s = 0.f;
    if (q < parts)
        for (int l = q * per; l < min(p.lanes, (q + 1) * per); ++l) s += red[l * cols + col];
    part[threadIdx.x] = s;
    __syncthreads();
    const int k = column * cols + col;
    if (q == 0 && k < p.K) {
        for (int r = 1; r < parts; ++r) s += part[r * cols + col];
        p.partial[(size_t)slab * p.K + k] = s;
    }
}

// Partial rows (workgroups along the pixels): four pixels per thread of workgroups that cover at most 256 channels
// while that gives no more than about 1024 workgroups, then longer slabs, and at most 1024 rows for the reduce kernel.
int tail_bwd_blocks(int64_t npix, int K)
{
    if (npix <= 0) return 1;
    const int vec = K % 8 == 0 ? 8 : 1, groups = (K + vec - 1) / vec;
    const int gpb = groups < TB_THREADS / vec ? groups : TB_THREADS / vec, lanes = TB_THREADS / gpb;
    const int64_t columns = (groups + gpb - 1) / gpb;
    int64_t per = npix * columns / ((int64_t)lanes * 1024);          // pixels per thread
    per = per < 4 ? 4 : (per + 3) / 4 * 4;
    const int64_t b = (npix + lanes * per - 1) / (lanes * per);
    return (int)(b > 1024 ? 1024 : b);
}

// The fewest rows the entry point takes a workspace for: about 32 pixels per thread of workgroups that hold up to
// 2048 channels (256 without 16-byte pieces), which is what a workspace query answered before slabs became shorter.
int tail_bwd_least_blocks(int64_t npix, int K)
{
    const int blocks = tail_bwd_blocks(npix, K), vec = K % 8 == 0 ? 8 : 1;
    const int64_t groups = (K + vec - 1) / vec, slab = TB_THREADS / (groups < TB_THREADS ? groups : TB_THREADS) * 32;
    const int64_t b = (npix + slab - 1) / slab;
    return b < 1 ? 1 : b < blocks ? (int)b : blocks;
}

hipError_t launch_tail_bwd(const TailBwdArgs &a0, bool is_bf16, hipStream_t stream)
{
    TailBwdArgs a = a0;
    const int blocks = a.rows;
    if (blocks < 1) return hipErrorInvalidValue;
    a.chunk = (a.npix + blocks - 1) / blocks;
    if (a.chunk < 1) a.chunk = 1;
    const TailBwdShape s = tail_bwd_shape(a);
    a.groups = s.groups;
    a.columns = s.columns;
    a.gpb = s.gpb;
    a.lanes = s.lanes;
    const bool interleave = s.columns > 1 && tail_bwd_large(a);
    const int64_t wgs = interleave ? (int64_t)(blocks + 7) / 8 * 8 * s.columns : blocks;
    if (wgs > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)wgs, interleave ? 1u : (unsigned)s.columns), block(TB_THREADS);
    const bool stream_dz = a.npix * a.K * 2 > 300000000 && !interleave;     // (cut lines have to meet in the L2)
    const auto go = [&](auto type) {
        using T = decltype(type);
        if (a.K % 8 != 0 && interleave) DLK_LAUNCH("tail_bwd_kernel", (tail_bwd_kernel<T, 1, false, true>), grid, block, 0, stream, a);
        else if (a.K % 8 != 0) DLK_LAUNCH("tail_bwd_kernel", (tail_bwd_kernel<T, 1, false, false>), grid, block, 0, stream, a);
        else if (interleave) DLK_LAUNCH("tail_bwd_kernel", (tail_bwd_kernel<T, 8, false, true>), grid, block, 0, stream, a);
        else if (stream_dz) DLK_LAUNCH("tail_bwd_kernel", (tail_bwd_kernel<T, 8, true, false>), grid, block, 0, stream, a);
        else DLK_LAUNCH("tail_bwd_kernel", (tail_bwd_kernel<T, 8, false, false>), grid, block, 0, stream, a);
    };
    if (is_bf16) go(BF16{});
    else go(F16{});
    hipError_t e = dlk::launch_status();
    if (e != hipSuccess) return e;
    return launch_splitk_reduce(a.partial, blocks, a.K, a.dbias, 2, stream);
}

}  // namespace dlk
