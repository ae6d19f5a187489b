// Data-parallel gradient path: one ring step of Alg. 2 with the identity as
// compute_partial_output, i.e. "O <- B_in + O" on one slice of the local fp32
// gradient bucket, in place.  HBM-bound: 12 bytes per element (read slice, read
// B_in, write slice).  16-byte accesses, several independent loads in flight
// per lane, one pass over the slice.  A variant also carries the emulated delivery:
// B_in is read from the neighbour's buffer and stored on to the landing buffer in the
// same pass (16 bytes per element instead of a copy's 8 plus the add's 12).
#include "cf_internal.h"

namespace cf {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int DP_THREADS = 256;
constexpr int DP_UNROLL = 4;

// The slices start wherever a multiple of the slice length falls, so three streams out of four may be 4-byte aligned only.
// The 16-byte accesses of this architecture need no more than that: a wave then touches one line more per access.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

// All adds of a rank step in ONE launch: segment s adds src[s] into dst[s], `n` elements each; workgroup b works on chunk
// b % per_seg of segment b / per_seg, U independent vectors per lane and stream in flight.
// LAND: the delivery carried by the consumer -- src is the neighbour's buffer, and what is read from it is also stored
// to `land`, this rank's landing buffer: 16 bytes per element (two reads, two writes) where a copy followed by the add
// moves 20.  Two sizes of the argument: a single step's (a short one is cheaper to enqueue: 0.15 us) and a rank step's.
template <int MAX>
struct AddSegments {
    float *dst[MAX];
    const float *src[MAX];
    float *land[MAX];
};
constexpr int MAX_SEGMENTS = 16;

// Every element is touched exactly once: the streams bypass the caches' retention (non-temporal), which measured ~25% faster
// than cached accesses on MI355X -- unless all that a launch touches stays in the caches (CACHED).
template <bool CACHED>
__device__ __forceinline__ f32x4_u load4(const f32x4_u *p)
{
    if constexpr (CACHED)
        return *p;
    else
        return __builtin_nontemporal_load(p);
}
template <bool CACHED>
__device__ __forceinline__ void store4(f32x4_t v, f32x4_u *p)
{
    if constexpr (CACHED)
        *p = v;
    else
        __builtin_nontemporal_store(v, p);
}

template <bool LAND, int T, int U, bool CACHED, int SEG>
__global__ __launch_bounds__(T) void dp_reduce_kernel(AddSegments<SEG> a, int64_t n, int per_seg)
{
    const int seg = SEG == 1 ? 0 : blockIdx.x / per_seg, chunk = SEG == 1 ? blockIdx.x : blockIdx.x % per_seg;
    float *const dst = a.dst[seg];
    const float *const src = a.src[seg];
    float *const land = a.land[seg];
    const int64_t n4 = n / 4;
    const int64_t base = (int64_t)chunk * T * U + threadIdx.x;
    f32x4_u *const dst4 = reinterpret_cast<f32x4_u *>(dst);
    const f32x4_u *const src4 = reinterpret_cast<const f32x4_u *>(src);
    f32x4_u *const land4 = reinterpret_cast<f32x4_u *>(land);
    f32x4_u x[U], y[U];
    if (chunk < per_seg - 1) {                       // (every chunk but the last is whole)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = load4<CACHED>(&dst4[base + u * T]);
            y[u] = load4<CACHED>(&src4[base + u * T]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            store4<CACHED>(y[u] + x[u], &dst4[base + u * T]);         // "O <- B_in + O"
            if constexpr (LAND)
                store4<CACHED>(y[u], &land4[base + u * T]);
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = base + u * T;
        if (i < n4) {
            y[u] = load4<CACHED>(&src4[i]);
            store4<CACHED>(y[u] + load4<CACHED>(&dst4[i]), &dst4[i]);
            if constexpr (LAND)
                store4<CACHED>(y[u], &land4[i]);
        }
    }
    if (chunk == per_seg - 1 && (int)threadIdx.x < (int)(n - n4 * 4)) {          // the last elements of the segment
        const int64_t i = n4 * 4 + threadIdx.x;
        const float b = src[i];
        dst[i] = b + dst[i];
        if constexpr (LAND)
            land[i] = b;
    }
}

// dst <- (((dst + src[0]) + src[1]) + ...) in ONE pass: the pairwise gradient reduce, where every round's arrival
// is added to the same slice.  4 (n + 2) bytes per element instead of 12 n for n separate passes; the additions
// are taken in the order of the separate passes, so the result is the same bit for bit.
struct AddBatch {
    static constexpr int MAX = 15;
    const float *src[MAX];
};

// LAND: as above -- source s is also stored to land[s].  INIT: dst <- ((src[0] + src[1]) + ...), what it held is not read.
// That sum is read again by the launch behind it and stays in the caches (pairwise rank steps, us, against a non-temporal
// store: 4 x 768 x 3000 x 264 55.2 -> 52.4, 8 x 512 x 4096 x 1376 82.5 -> 73.6, 4 x 390 x 8192 x 512 59.0 -> 49.7).
// U: vectors per lane, (n_src + 1) * U loads in flight.
template <bool LAND, bool INIT, int U>
__global__ __launch_bounds__(DP_THREADS) void dp_reduce_multi_kernel(float *__restrict__ dst, AddBatch ab, int n_src,
                                                                    int64_t n, AddBatch lb)
{
    const int64_t n4 = n / 4;
    const int64_t base = (int64_t)blockIdx.x * DP_THREADS * U + threadIdx.x;
    f32x4_u *const dst4 = reinterpret_cast<f32x4_u *>(dst);
    f32x4_u a[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (!INIT && base + u * DP_THREADS < n4)
            a[u] = __builtin_nontemporal_load(&dst4[base + u * DP_THREADS]);
    for (int s = 0; s < n_src; ++s) {
        const f32x4_u *__restrict__ src = reinterpret_cast<const f32x4_u *>(ab.src[s]);
        f32x4_u *__restrict__ land = reinterpret_cast<f32x4_u *>(const_cast<float *>(lb.src[s]));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (base + u * DP_THREADS < n4) {
                const f32x4_u b = __builtin_nontemporal_load(&src[base + u * DP_THREADS]);
                a[u] = INIT && s == 0 ? b : a[u] + b;
                if constexpr (LAND)
                    __builtin_nontemporal_store(b, &land[base + u * DP_THREADS]);
            }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (base + u * DP_THREADS < n4)
            store4<INIT>(a[u], &dst4[base + u * DP_THREADS]);
    if (blockIdx.x == gridDim.x - 1 && (int)threadIdx.x < (int)(n - n4 * 4)) {
        const int64_t i = n4 * 4 + threadIdx.x;
        float x = INIT ? 0.0f : dst[i];
        for (int s = 0; s < n_src; ++s) {
            const float b = ab.src[s][i];
            x = INIT && s == 0 ? b : x + b;
            if constexpr (LAND)
                const_cast<float *>(lb.src[s])[i] = b;
        }
        dst[i] = x;
    }
}

// Several equally long device-to-device copies in ONE launch (the deliveries of a whole rank step when they are
// all enqueued in front of the persistent kernel): workgroup b moves chunk b % per_buf of buffer b / per_buf,
// 16 bytes per lane and access, four independent vectors in flight, non-temporal both ways like the reduce above.
struct CopyBatch {
    static constexpr int MAX = 16;
    const void *src[MAX];
    void *dst[MAX];
};

__global__ __launch_bounds__(DP_THREADS) void copy_batch_kernel(CopyBatch cb, int64_t n16, int per_buf)
{
    const int buf = blockIdx.x / per_buf, chunk = blockIdx.x % per_buf;
    const f32x4_t *__restrict__ src = static_cast<const f32x4_t *>(cb.src[buf]);
    f32x4_t *__restrict__ dst = static_cast<f32x4_t *>(cb.dst[buf]);
    const int64_t base = (int64_t)chunk * DP_THREADS * DP_UNROLL + threadIdx.x;
    f32x4_t v[DP_UNROLL];
#pragma unroll
    for (int u = 0; u < DP_UNROLL; ++u)
        if (base + u * DP_THREADS < n16)
            v[u] = __builtin_nontemporal_load(&src[base + u * DP_THREADS]);
#pragma unroll
    for (int u = 0; u < DP_UNROLL; ++u)
        if (base + u * DP_THREADS < n16)
            __builtin_nontemporal_store(v[u], &dst[base + u * DP_THREADS]);
}

__global__ __launch_bounds__(64) void set_words_kernel(unsigned *dst, int count, unsigned value)
{
    for (int i = threadIdx.x; i < count; i += 64)
        __hip_atomic_store(&dst[i], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(256) void fill_ff_kernel(unsigned *dst, size_t nwords)
{
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < nwords; i += stride)
        dst[i] = 0xFFFFFFFFu;
}

template <int SEG>
hipError_t launch_adds(float *const *dst, const float *const *src, float *const *land, int n_seg, int64_t n, int per_seg,
                       int threads, bool long_segments, bool cached, hipStream_t s)
{
    AddSegments<SEG> a = {};
    for (int i = 0; i < n_seg; ++i) {
        a.dst[i] = dst[i];
        a.src[i] = src[i];
        a.land[i] = land != nullptr ? land[i] : nullptr;
    }
    const dim3 grid((unsigned)((int64_t)per_seg * n_seg)), block(threads);
#define CF_ADD(T, U, C)                                                                                       \
    do {                                                                                                      \
        if (land != nullptr)                                                                                  \
            hipLaunchKernelGGL((dp_reduce_kernel<true, T, U, C, SEG>), grid, block, 0, s, a, n, per_seg);     \
        else                                                                                                  \
            hipLaunchKernelGGL((dp_reduce_kernel<false, T, U, C, SEG>), grid, block, 0, s, a, n, per_seg);    \
    } while (0)
    if (threads == 64)
        CF_ADD(64, 1, false);
    else if (long_segments)
        CF_ADD(256, 1, false);
    else if (cached)
        CF_ADD(256, 4, true);
    else
        CF_ADD(256, 4, false);
#undef CF_ADD
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dp_reduce_segments(float *const *dst, const float *const *src, float *const *land, int n_seg, int64_t n,
                                     hipStream_t s)
{
    if (n <= 0 || n_seg <= 0)
        return hipSuccess;
    // A grid that covers the slices once measured faster than a grid-stride loop over a chip-sized grid (5.9 vs 4.4 TB/s at
    // 125M elements).  Seven segments landing their arrivals, buffers in turn, TB/s for (threads, vectors per lane):
    //   125M elements: (64, 1) 6.1, (256, 1) 5.9, (256, 4) 5.4, (64, 2) 5.2;   10M: 6.25, 6.1, 6.2, 5.7;
    //   3M: 5.5, 5.8, 5.9, 6.2;   20M, segments off the 16-byte grid: 5.5, 5.7, 5.6, 5.1.
    // Up to 64 MB in all the caches keep what a launch touches, and non-temporal accesses only cost (us, cached against
    // non-temporal, slices off the 16-byte grid): one segment of 1M elements landing its arrival 4.2 / 5.1, 3M 8.3 / 10.0,
    // 5M (80 MB) 15.7 / 15.4; one of 5M without a landing (60 MB) 10.0 / 11.8, 8M 18.4 / 17.5; three of 1M 8.4 / 10.0, five 15.6 /
    // 15.5.
    uintptr_t bits = 0;
    for (int i = 0; i < n_seg; ++i)
        bits |= reinterpret_cast<uintptr_t>(dst[i]) | reinterpret_cast<uintptr_t>(src[i]) |
                (land != nullptr ? reinterpret_cast<uintptr_t>(land[i]) : 0);
    const bool long_segments = n >= (int64_t)8 << 20, aligned = (bits & 15u) == 0;
    const int threads = long_segments && aligned ? 64 : 256;
    const int per_wg = threads * (long_segments ? 1 : 4);
    const int64_t per_seg = (n / 4 + per_wg) / per_wg;
    const bool cached = !long_segments && (double)n * n_seg * (land != nullptr ? 16 : 12) <= 64e6;
    int at = 0;
    while (at < n_seg) {                             // (as many segments per launch as its arguments and its grid take)
        int take = n_seg - at < MAX_SEGMENTS ? n_seg - at : MAX_SEGMENTS;
        while (take > 1 && per_seg * take >= ((int64_t)1 << 31))
            --take;
        if (per_seg * take >= ((int64_t)1 << 31))
            return hipErrorInvalidValue;
        float *const *l = land != nullptr ? &land[at] : nullptr;
        hipError_t e = take == 1 ? launch_adds<1>(&dst[at], &src[at], l, 1, n, (int)per_seg, threads, long_segments, cached, s)
                                 : launch_adds<MAX_SEGMENTS>(&dst[at], &src[at], l, take, n, (int)per_seg, threads, long_segments, cached, s);
        if (e != hipSuccess)
            return e;
        at += take;
    }
    return hipSuccess;
}

hipError_t launch_dp_reduce_multi(float *dst, const float *const *src, int n_src, int64_t n, hipStream_t s, float *const *land,
                                  bool init)
{
    if (n <= 0 || n_src <= 0)
        return hipSuccess;
    if (init && n_src > AddBatch::MAX)
        return hipErrorInvalidValue;
    if (n_src > AddBatch::MAX || (n_src == 1 && !init)) {    // one pass per source: the same additions in the same order
        for (int i = 0; i < n_src; ++i) {
            hipError_t e = launch_dp_reduce_segments(&dst, &src[i], land != nullptr ? &land[i] : nullptr, 1, n, s);
            if (e != hipSuccess)
                return e;
        }
        return hipSuccess;
    }
    AddBatch ab = {}, lb = {};
    for (int i = 0; i < n_src; ++i) {
        ab.src[i] = src[i];
        lb.src[i] = land != nullptr ? land[i] : nullptr;
    }
    // Short slices: one vector per lane, twice the workgroups (7 sources, us for one / two vectors: 30 thousand elements 4.6 / 6.4,
    // 1M 12.0 / 14.9, 2M 23.7 / 22.3, 3M 34.1 / 33.2, 10M 108 / 110).
    const bool short_slice = n < 3 << 19;
    const int64_t per_wg = (int64_t)DP_THREADS * (short_slice ? 1 : 2);
    const int64_t want = (n / 4 + per_wg) / per_wg;
    if (want >= ((int64_t)1 << 31))
        return hipErrorInvalidValue;
#define CF_MULTI_U(L, I, U) \
    hipLaunchKernelGGL((dp_reduce_multi_kernel<L, I, U>), dim3((unsigned)want), dim3(DP_THREADS), 0, s, dst, ab, n_src, n, lb)
#define CF_MULTI(L, I)              \
    do {                            \
        if (short_slice)            \
            CF_MULTI_U(L, I, 1);    \
        else                        \
            CF_MULTI_U(L, I, 2);    \
    } while (0)
    if (init && land != nullptr)
        CF_MULTI(true, true);
    else if (init)
        CF_MULTI(false, true);
    else if (land != nullptr)
        CF_MULTI(true, false);
    else
        CF_MULTI(false, false);
#undef CF_MULTI
#undef CF_MULTI_U
    return hipGetLastError();
}

bool copy_batch_takes(const void *const *src, void *const *dst, int n, size_t bytes)
{
    if (n < 1 || n > CopyBatch::MAX || bytes == 0 || bytes % 16 != 0)
        return false;
    const int64_t per_buf = (int64_t)((bytes / 16 + (size_t)DP_THREADS * DP_UNROLL - 1) / ((size_t)DP_THREADS * DP_UNROLL));
    if (per_buf * n >= ((int64_t)1 << 31))
        return false;
    for (int i = 0; i < n; ++i)
        if (((reinterpret_cast<uintptr_t>(src[i]) | reinterpret_cast<uintptr_t>(dst[i])) & 15u) != 0)
            return false;
    return true;
}

hipError_t launch_copy_batch(const void *const *src, void *const *dst, int n, size_t bytes, hipStream_t s)
{
    CopyBatch cb = {};
    for (int i = 0; i < n; ++i) {
        cb.src[i] = src[i];
        cb.dst[i] = dst[i];
    }
    const int64_t n16 = (int64_t)(bytes / 16);
    const int per_buf = (int)((n16 + (int64_t)DP_THREADS * DP_UNROLL - 1) / ((int64_t)DP_THREADS * DP_UNROLL));
    hipLaunchKernelGGL(copy_batch_kernel, dim3((unsigned)(per_buf * n)), dim3(DP_THREADS), 0, s, cb, n16, per_buf);
    return hipGetLastError();
}

hipError_t launch_set_words(unsigned *dst, int count, unsigned value, hipStream_t s)
{
    if (count <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(set_words_kernel, dim3(1), dim3(64), 0, s, dst, count, value);
    return hipGetLastError();
}

hipError_t launch_fill_ff(void *dst, size_t bytes, hipStream_t s)
{
    const size_t nwords = bytes / 4;
    if (nwords == 0)
        return hipSuccess;
    size_t want = (nwords + 255) / 256;
    const int blocks = (int)(want < 2048 ? want : 2048);
    hipLaunchKernelGGL(fill_ff_kernel, dim3(blocks), dim3(256), 0, s, static_cast<unsigned *>(dst), nwords);
    return hipGetLastError();
}

}  // namespace cf
