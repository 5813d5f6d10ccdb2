// LARC weight update (layer-wise adaptive rate control) for many tensors in two launches.
//
// Per tensor t with fp32 weights w, gradient g (fp16, bf16 or fp32) and optional fp32 momentum
// buffer v:
//     local = trust * ||w|| / (||g|| + wd * ||w|| + eps)      (lr itself if ||w|| or ||g|| is 0)
//     rate  = clip ? min(local, lr) : local * lr
//     v    <- momentum * v + rate * (g + wd * w);   w <- w - v
// Launch 1: every workgroup adds w^2 and g^2 over its slice of its tensor (fp32, fixed order) and
// writes two partial sums.  Launch 2 (same grid): every workgroup adds its tensor's partials by a
// fixed tree (so all of them derive the very same rate), then updates its slice.  The tensor table
// travels as a kernel argument (no device-side table to upload), at most LARC_MAX tensors per pair
// of launches.
//
// Bound by memory.  A tensor is cut into slices of 8192 elements, or LARC_SLICES longer ones where it
// has more: the first version cut every tensor into 256, so that most of its workgroups had a few
// elements and all of them began launch 2 with one thread adding 512 values.  Launch 2 takes the slices
// in the reverse of launch 1's order: what that launch read last is what the last-level cache still holds.
// Measured (63 filters, 40.3 M parameters, fp16 gradients, momentum): launch 1 60.7 -> 49.3 us (4.9 TB/s),
// launch 2 150 -> 113 us (6.4 TB/s, part of it from the cache).
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace dlk {

constexpr int LARC_THREADS = 256;

template <class G> __device__ __forceinline__ float larc_grad(const void *g, int64_t i);
template <> __device__ __forceinline__ float larc_grad<F16>(const void *g, int64_t i) { return F16::to_float(static_cast<const uint16_t *>(g)[i]); }
template <> __device__ __forceinline__ float larc_grad<BF16>(const void *g, int64_t i) { return BF16::to_float(static_cast<const uint16_t *>(g)[i]); }
template <> __device__ __forceinline__ float larc_grad<float>(const void *g, int64_t i) { return static_cast<const float *>(g)[i]; }

// four consecutive gradient values starting at element i (i % 4 == 0, tensor base suitably aligned)
template <class G> __device__ __forceinline__ floatx4_t larc_grad4(const void *g, int64_t i)
{
    if constexpr (std::is_same<G, float>::value) {
        return *reinterpret_cast<const floatx4_t *>(static_cast<const float *>(g) + i);
    } else {
        const u32x2_t v = *reinterpret_cast<const u32x2_t *>(static_cast<const uint16_t *>(g) + i);
        return floatx4_t{G::to_float((uint16_t)(v[0] & 0xffffu)), G::to_float((uint16_t)(v[0] >> 16)),
                         G::to_float((uint16_t)(v[1] & 0xffffu)), G::to_float((uint16_t)(v[1] >> 16))};
    }
}
// 16-byte accesses are possible when the tensor's bases allow it (slices start at multiples of 4 elements)
template <class G> __device__ __forceinline__ bool larc_vec_ok(const LarcTensor &t)
{
    const uintptr_t gmask = std::is_same<G, float>::value ? 15u : 7u;
    return ((reinterpret_cast<uintptr_t>(t.w) | reinterpret_cast<uintptr_t>(t.v)) & 15u) == 0 &&
           (reinterpret_cast<uintptr_t>(t.g) & gmask) == 0;
}

// Elements per slice (a multiple of 4) and slices of a tensor.
__host__ __device__ __forceinline__ int64_t larc_slice_elems(int64_t count)
{
    const int64_t least = ((count + LARC_SLICES - 1) / LARC_SLICES + 3) / 4 * 4;
    return least < 8192 ? 8192 : least;
}

// Sums over the workgroup by a fixed tree; every thread gets them.
__device__ __forceinline__ void larc_block_sum(float &a, float &b, float (&red)[2][LARC_THREADS / 64])
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = a; red[1][threadIdx.x >> 6] = b; }
    __syncthreads();
    a = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    b = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
}

// The slice of this workgroup: b.start[] holds the running number of slices, workgroup ids count through them.
// Every lane compares one entry; LARC_MAX + 1 entries, the last of which (and all beyond b.n) is the grid size.
__device__ __forceinline__ int larc_tensor(const LarcBatch &b, int id)
{
    static_assert(LARC_MAX == 64, "one table entry per lane");
    const int lane = threadIdx.x & 63;
    return __builtin_amdgcn_readfirstlane(__popcll(__ballot(b.start[lane + 1] <= id)));
}
__device__ __forceinline__ void larc_slice(int64_t count, int slice, int64_t *begin, int64_t *end)
{
    const int64_t chunk = larc_slice_elems(count);
    *begin = min(count, slice * chunk);
    *end = min(count, *begin + chunk);
}

constexpr int LARC_UNROLL = 4, LARC_TRIP = 4 * LARC_THREADS;          // elements of one pass of the workgroup

template <class G>
__global__ __launch_bounds__(LARC_THREADS) void larc_norm_kernel(const LarcBatch b)
{
    const int ti = larc_tensor(b, blockIdx.x), slice = (int)blockIdx.x - b.start[ti];
    const LarcTensor &t = b.t[ti];
    int64_t begin, end;
    larc_slice(t.count, slice, &begin, &end);
    float sw = 0.f, sg = 0.f;
    int64_t i0 = begin;
    if (larc_vec_ok<G>(t)) {
        const int64_t vend = begin + (end - begin) / 4 * 4;
        auto add = [&](floatx4_t w, floatx4_t g) {
            sw += (w[0] * w[0] + w[1] * w[1]) + (w[2] * w[2] + w[3] * w[3]);
            sg += (g[0] * g[0] + g[1] * g[1]) + (g[2] * g[2] + g[3] * g[3]);
        };
        int64_t i = begin + 4 * threadIdx.x;
        for (; i + (LARC_UNROLL - 1) * LARC_TRIP < vend; i += LARC_UNROLL * LARC_TRIP) {
            floatx4_t w[LARC_UNROLL], g[LARC_UNROLL];
#pragma unroll
            for (int u = 0; u < LARC_UNROLL; ++u) w[u] = *reinterpret_cast<const floatx4_t *>(t.w + i + u * LARC_TRIP);
#pragma unroll
            for (int u = 0; u < LARC_UNROLL; ++u) g[u] = larc_grad4<G>(t.g, i + u * LARC_TRIP);
#pragma unroll
            for (int u = 0; u < LARC_UNROLL; ++u) add(w[u], g[u]);
        }
        for (; i < vend; i += LARC_TRIP) add(*reinterpret_cast<const floatx4_t *>(t.w + i), larc_grad4<G>(t.g, i));
        i0 = vend;
    }
    for (int64_t i = i0 + threadIdx.x; i < end; i += LARC_THREADS) {
        const float w = t.w[i], g = larc_grad<G>(t.g, i);
        sw += w * w;
        sg += g * g;
    }
    __shared__ float red[2][LARC_THREADS / 64];
    larc_block_sum(sw, sg, red);
    if (threadIdx.x == 0) {
        float *out = b.partial + ((size_t)(b.first + ti) * LARC_SLICES + slice) * 2;
        out[0] = sw;
        out[1] = sg;
    }
}

template <class G>
__global__ __launch_bounds__(LARC_THREADS) void larc_update_kernel(const LarcBatch b)
{
    static_assert(LARC_SLICES <= LARC_THREADS, "one partial sum per thread");
    const int id = (int)gridDim.x - 1 - (int)blockIdx.x;                // the reverse of the first launch's order
    const int ti = larc_tensor(b, id), first = b.start[ti], slice = id - first, slices = b.start[ti + 1] - first;
    const LarcTensor &t = b.t[ti];
    float sw = 0.f, sg = 0.f;
    if ((int)threadIdx.x < slices) {
        const float *p = b.partial + ((size_t)(b.first + ti) * LARC_SLICES + threadIdx.x) * 2;
        sw = p[0];
        sg = p[1];
    }
    __shared__ float red[2][LARC_THREADS / 64];
    larc_block_sum(sw, sg, red);
    const float wn = sqrtf(sw), gn = sqrtf(sg);
    const float local = (wn > 0.f && gn > 0.f) ? b.trust * wn / (gn + b.wd * wn + b.eps) : (b.clip ? b.lr : 1.f);
    const float rate = b.clip ? fminf(local, b.lr) : local * b.lr;
    if (threadIdx.x == 0 && slice == 0 && b.rates) b.rates[b.first + ti] = rate;
    int64_t begin, end;
    larc_slice(t.count, slice, &begin, &end);
    int64_t i0 = begin;
    if (larc_vec_ok<G>(t)) {
        const int64_t vend = begin + (end - begin) / 4 * 4;
        auto put = [&](int64_t i, floatx4_t w, floatx4_t g, floatx4_t v) {
            floatx4_t step;
#pragma unroll
            for (int e = 0; e < 4; ++e) step[e] = rate * (g[e] + b.wd * w[e]);
            if (t.v) {
#pragma unroll
                for (int e = 0; e < 4; ++e) step[e] += b.momentum * v[e];
                *reinterpret_cast<floatx4_t *>(t.v + i) = step;
            }
            *reinterpret_cast<floatx4_t *>(t.w + i) = w - step;
        };
        auto vel = [&](int64_t i) {
            return t.v ? *reinterpret_cast<const floatx4_t *>(t.v + i) : floatx4_t{0.f, 0.f, 0.f, 0.f};
        };
        int64_t i = begin + 4 * threadIdx.x;
        for (; i + (LARC_UNROLL - 1) * LARC_TRIP < vend; i += LARC_UNROLL * LARC_TRIP) {
            floatx4_t w[LARC_UNROLL], g[LARC_UNROLL], v[LARC_UNROLL];
#pragma unroll
            for (int u = 0; u < LARC_UNROLL; ++u) w[u] = *reinterpret_cast<const floatx4_t *>(t.w + i + u * LARC_TRIP);
#pragma unroll
            for (int u = 0; u < LARC_UNROLL; ++u) g[u] = larc_grad4<G>(t.g, i + u * LARC_TRIP);
#pragma unroll
            for (int u = 0; u < LARC_UNROLL; ++u) v[u] = vel(i + u * LARC_TRIP);
#pragma unroll
            for (int u = 0; u < LARC_UNROLL; ++u) put(i + u * LARC_TRIP, w[u], g[u], v[u]);
        }
        for (; i < vend; i += LARC_TRIP) put(i, *reinterpret_cast<const floatx4_t *>(t.w + i), larc_grad4<G>(t.g, i), vel(i));
        i0 = vend;
    }
    for (int64_t i = i0 + threadIdx.x; i < end; i += LARC_THREADS) {
        const float w = t.w[i];
        float step = rate * (larc_grad<G>(t.g, i) + b.wd * w);
        if (t.v) {
            step += b.momentum * t.v[i];
            t.v[i] = step;
        }
        t.w[i] = w - step;
    }
}

template <class G>
static hipError_t larc_launch(const LarcBatch &b, hipStream_t stream)
{
    const dim3 grid((unsigned)b.start[LARC_MAX]), block(LARC_THREADS);
    DLK_LAUNCH("larc_norm_kernel", larc_norm_kernel<G>, grid, block, 0, stream, b);
    hipError_t e = dlk::launch_status();
    if (e != hipSuccess) return e;
    DLK_LAUNCH("larc_update_kernel", larc_update_kernel<G>, grid, block, 0, stream, b);
    return dlk::launch_status();
}

hipError_t launch_larc(const LarcBatch &b0, int grad_dtype, hipStream_t stream)
{
    if (b0.n < 1 || b0.n > LARC_MAX) return hipErrorInvalidValue;
    LarcBatch b = b0;
    int32_t slices = 0;                                  // at most LARC_MAX * LARC_SLICES
    for (int i = 0; i < LARC_MAX; ++i) {
        b.start[i] = slices;
        if (i < b.n) slices += (int32_t)((b.t[i].count + larc_slice_elems(b.t[i].count) - 1) / larc_slice_elems(b.t[i].count));
    }
    b.start[LARC_MAX] = slices;
    if (grad_dtype == 0) return larc_launch<F16>(b, stream);
    if (grad_dtype == 1) return larc_launch<BF16>(b, stream);
    return larc_launch<float>(b, stream);
}

}  // namespace dlk
