// Chunk GEMM for FEW ROWS (decoded tokens, the smallest layers): out[r x n] = A[r x k] W (+ B_in), bf16 or fp32 operands,
// fp32 accumulation, the fused epilogue of the tile kernels ("O <- B_in + O", "B_out <- O", or the slice store of Alg. 1).
//
// What bounds it: with a handful of rows every weight is used a handful of times, so the time is that of reading W once
// -- or, at a few megabytes, the latency of one trip to memory plus a launch.  The 128-row tiles of the other kernels
// walk the k range as a serial chain on a few dozen compute units for that.  Here instead:
//  * a workgroup owns 16 NC columns and up to 16 MF rows, and its NW waves split the K RANGE: wave w takes the k slices
//    w, w + NW, ... of 128 bytes each; every wave runs its own ring of LDS stages (direct global -> LDS loads, two to four
//    slices in flight, awaited by its own vmcnt), so there is no barrier in the k loop, and the partial tiles of the waves
//    meet once, in LDS, in wave order (deterministic);
//  * v_mfma_f32_16x16x32_bf16 / v_mfma_f32_16x16x4_f32, the weights on the "A" side, the activations on the "B" side as in
//    the tile kernels.  Loads straight into the MFMA register layout (no LDS) were built first: neighbouring lanes of a
//    fragment are different ROWS, and a 16-byte load whose lanes lie in different lines runs at a quarter of the
//    L1's rate (8 x 1536 x 4096: 8.6 us against 5.5 through LDS);
//  * the rows of ALL steps of a rank step can be packed into one launch (segments: every step has its own left operand,
//    B_in, landing buffer and output), so that W is read once and not once per step;
//  * the received partial is requested before the k loop and added at the end; a delivery carried by the launch is
//    stored on by the threads that read it (reduce-scatter) or by extra workgroups (all-gather: the slices);
//  * where even that leaves compute units idle and a single bf16 step has a workspace, KSPLIT workgroups share a tile: partial tiles and
//    an arrival counter with the device-coherent cache policy, summed in split order by the last to arrive.
// Measured (one step, B_in added; us, before = 128 x 128 tiles): 8 x 4096 x 1376 bf16 18.1 -> 4.4 (an empty kernel: 2.25),
// 8 x 8192 x 3584 24.7 -> 13.4 (4.4 TB/s of W), 128 x 8192 x 3584 34 -> 18.7, 128 x 256 x 512 fp32 16.2 -> 3.9; eight steps of 8 x 1536 x 4096 packed into one launch 42.5 -> 8.6.
#include "cf_internal.h"

namespace cf {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));

constexpr unsigned OOB = 0x80000000u;                // byte offset beyond any buffer this kernel accepts
constexpr int COHERENT = 1 | 16;                     // buffer cache-policy bits sc0 | sc1

// Two sizes of the kernel argument: one segment (a single step: every pointer is a scalar, and a short argument is
// cheaper to enqueue), or the steps of a rank step.
template <int SEG>
struct RowsParams {
    static constexpr int MORE = SEG == 1 ? 1 : GemmParams::MAX_RECV_MORE;
    const void *W;
    int64_t lda, ldw, ldo;
    int seg_rows, n_seg, N, K;                       // rows per segment (step), segments
    int tiles_n, tiles_r, ksplit, copy_wgs;
    float *ws;
    unsigned *counters;
    const void *A[SEG];
    const float *recv[SEG];                          // B_in of the segment (nullable), added to the product
    float *land[SEG];                                // nullable: where B_in (copy_wgs == 0) or the slice A lands
    void *out[SEG];
    int n_more;                                      // further partials of the LAST segment, added after its recv
    const float *more[MORE];
    float *more_land[MORE];
};

// Entry `s` (different from lane to lane) of a pointer table in the kernel argument: the whole table comes in through the
// scalar cache and the lane picks its entry.  Indexed directly it would be a vector load from the argument's memory, one
// trip more in front of the first operand load.
template <int SEG, typename T>
__device__ __forceinline__ T pick(T const (&table)[SEG], int s)
{
    T v = table[0];
#pragma unroll
    for (int i = 1; i < SEG; ++i)
        v = s == i ? table[i] : v;
    return v;
}

// Wave-wide 16-byte-per-lane loads straight into LDS (lane L lands at lds_addr + 16 L), awaited by the caller (vmcnt).
__device__ __forceinline__ void direct_load_16(i32x4_t rsrc, unsigned voffset, int soffset, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voffset), "s"(rsrc), "s"(soffset)
                 : "memory");
}
__device__ __forceinline__ void direct_load_16(const char *ptr, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "global_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds_addr), "v"(ptr)
                 : "memory");
}

__device__ __forceinline__ i32x4_t make_rsrc(const void *base, unsigned bytes)
{
    const unsigned long long a = reinterpret_cast<unsigned long long>(base);
    i32x4_t r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(a & 0xFFFFFFFFull));
    r[1] = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xFFFFull));
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = 0x00020000;
    return r;
}

// Workgroup id -> place in an order that gives each of the eight XCDs a contiguous range.
__device__ __forceinline__ int xcd_remap(int id, int total)
{
    const int q = total >> 3, rem = total & 7, xcd = id & 7;
    return xcd * q + (xcd < rem ? xcd : rem) + (id >> 3);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// LDS stages per wave: as many as fit, at most four
template <int MF, int NC, int NW>
constexpr int D_ = 160 / (NW * 2 * (MF + NC)) < 4 ? 160 / (NW * 2 * (MF + NC)) : 4;

template <bool BF16, bool KN, int MF, int NC, bool OUT_BF16, int NW, int SEG>
__global__ __launch_bounds__(64 * NW) void gemm_rows_kernel(RowsParams<SEG> P)
{
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int KSL = 128 / ES;                                    // k values of a slice
    constexpr int TN = 16 * NC, TR = 16 * MF;
    constexpr int PITCH = TN + 4;                                    // floats per row of a wave's partial tile
    constexpr int KPL = 16 / ES;                                     // k values in a 16-byte chunk
    constexpr int Q = TR * TN / 4;                                   // 16-byte pieces of the output tile
    constexpr int QT = (Q + 64 * NW - 1) / (64 * NW);                // ... per thread
    constexpr int LPS = 2 * (MF + NC);                               // direct loads per slice and wave
    constexpr int STAGE = 2048 * (MF + NC);
    constexpr int D = D_<MF, NC, NW>;                                // stages per wave
    constexpr int RING = D * STAGE;
    static_assert(D >= 2 && D <= 4 && NW * RING <= 160 * 1024, "stages fit in LDS");
    static_assert(TR * PITCH * 4 <= RING, "a partial tile fits in its wave's stages");

    __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * RING];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int R = P.seg_rows * (SEG == 1 ? 1 : P.n_seg);
    auto seg_of = [&](int r) { return SEG == 1 ? 0 : r / P.seg_rows; };
    const int tiles = P.tiles_n * P.tiles_r;

    // extra workgroups: the slices of an all-gather on their way to the landing buffers
    if (const int c0 = (int)blockIdx.x - tiles * P.ksplit; c0 >= 0) {
        const int row16 = P.K * ES / 16;                             // 16-byte chunks per row
        const int64_t per_seg = (int64_t)P.seg_rows * row16;
        for (int64_t i = (int64_t)c0 * (64 * NW) + tid; i < per_seg * P.n_seg; i += (int64_t)P.copy_wgs * (64 * NW)) {
            const int s = SEG == 1 ? 0 : (int)(i / per_seg);
            const int64_t in = i - s * per_seg;
            const int64_t row = in / row16, off = row * P.lda * ES + (in - row * row16) * 16;
            if (P.land[s] != nullptr)
                *reinterpret_cast<u32x4_t *>(reinterpret_cast<char *>(P.land[s]) + off) =
                    *reinterpret_cast<const u32x4_t *>(static_cast<const char *>(P.A[s]) + off);
        }
        return;
    }
    // Every XCD (workgroups x, x + 8, ...: an L2 of its own) takes a band of neighbouring tile columns, the row tiles of a column
    // next to each other: they walk k side by side and read the weights once through that L2, and so do the launches of
    // successive steps.  (With the columns dealt out one by one, the columns' row tiles landed on different XCDs and rounds:
    // us per call, columns one by one / in bands: all-gather step 30 x 4080 x 4984 16.9 / 12.6, reduce-scatter step 685 x 1384 x
    // 5168 32.2 / 28.6, all-gather rank step 4 x 34 x 1800 x 2600 16.5 / 13.5, 8 x 8 x 1536 x 4096 11.8 / 10.8, where two tiles share
    // a 128-byte line of W.)
    // One by one, tile column c on XCD c % 8, where that keeps a column's row tiles on one XCD as well and no line is shared: the
    // rows of [k x n] weights are then read in pieces of a line each by all XCDs at once, not a piece of 512 bytes and more by one.
    // us, one by one / in bands: steps 64 x 4096 x 8192 19.5 / 21.2, 128 x 4096 x 8192 22.2 / 24.2, 128 x 8192 x 3584 15.7 / 16.5,
    // 256 x 2048 x 8192 21.4 / 22.6, 100 x 5120 x 640 6.0 / 6.5; reduce-scatter rank steps 8 x 16 x 8192 x 3584 20.8 / 21.6, 4 x 16 x
    // 6144 x 2048 11.4 / 11.7.  More tiles than compute units (256): a column's row tiles would fall into two rounds, 384 x 4096 x 8192
    // 54.1 / 46.6, 512 x 4096 x 4096 32.8 / 30.1.  Narrower matrices and launches that land the slices of an all-gather beside the tiles are faster in
    // bands: 512 x 1024 x 4096 13.5 / 12.6, reduce-scatter 8 x 32 x 2048 x 4096 15.6 / 14.7, all-gather 8 x 8 x 4096 x 4096 15.6 /
    // 13.2; and so is nearly everything with [n x k] weights (1 x 4096 x 8192 14.8 / 11.5; 131 drawn steps 0.98, but 51 of 6144
    // columns and more over less than 2048 of k 1.02, 48 x 8192 x 1024 5.9 / 6.5: sending those one by one puts a branch in front of
    // every step's first load that costs the others 1 %).
    int tile_n, split = 0, tile_r = 0;
    if (BF16 && KN && NC == 4 && P.tiles_n % 8 == 0 && P.tiles_n > (SEG == 1 ? 16 : 32) && P.ldw % 64 == 0 && P.copy_wgs == 0 &&
        tiles <= 256) {
        tile_r = (int)blockIdx.x / P.tiles_n;
        tile_n = (int)blockIdx.x - tile_r * P.tiles_n;
        if (P.ksplit > 1) {
            split = tile_r % P.ksplit;
            tile_r /= P.ksplit;
        }
    } else {
        const int unit = xcd_remap((int)blockIdx.x, tiles * P.ksplit);
        tile_n = unit;
        if (const int per_col = P.tiles_r * P.ksplit; per_col > 1) {
            tile_n = unit / per_col;
            const int in = unit - tile_n * per_col;
            split = in / P.tiles_r;
            tile_r = in - split * P.tiles_r;
        }
    }
    const int tile = tile_r * P.tiles_n + tile_n;
    const int n0 = tile_n * TN, r0 = tile_r * TR;

    // (segment, row) of the output pieces this thread finishes, and their B_in, requested before anything else
    int64_t ooff[QT];
    int oseg[QT];                                                    // -1: nothing to finish
    const float *orecv[QT];
    f32x4_t rv[QT];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int q = tid + u * 64 * NW;
        const int r = r0 + q / (TN / 4), n = n0 + (q % (TN / 4)) * 4;
        oseg[u] = -1;
        ooff[u] = 0;
        orecv[u] = nullptr;
        rv[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (q < Q && r < R && n < P.N) {
            const int s = seg_of(r);
            oseg[u] = s;
            ooff[u] = (int64_t)(r - s * P.seg_rows) * P.ldo + n;
            orecv[u] = pick(P.recv, s);
            if (orecv[u] != nullptr)
                rv[u] = *reinterpret_cast<const f32x4_t *>(orecv[u] + ooff[u]);
        }
    }

    // A k slice is 128 bytes of k (64 bf16, 32 fp32).  Blocks in LDS, 2 KiB each, per stage: MF of the activations, NC of the
    // weights.  k-contiguous operands: 16 rows of eight 16-byte chunks, chunk c of row r in place c ^ (r / 2): the sixteen
    // rows of a fragment read then lie in sixteen different bank groups.
    const int b = lane >> 4, l16 = lane & 15;
    const char *arow[MF][2];                                         // this lane's pieces of the activation blocks at k0 = 0
    int achunk[2];                                                   // ... and which chunk of the slice they are
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = i * 8 + (lane >> 3);
        achunk[i] = (lane & 7) ^ (row >> 1);
#pragma unroll
        for (int f = 0; f < MF; ++f) {
            int r = r0 + f * 16 + row;
            r = r < R ? r : R - 1;                                   // (a row beyond the last only feeds sums nobody stores)
            const int s = seg_of(r);
            arow[f][i] = static_cast<const char *>(pick(P.A, s)) + (int64_t)(r - s * P.seg_rows) * P.lda * ES;
        }
    }
    const unsigned w_bytes = (unsigned)((KN ? (int64_t)(P.K - 1) * P.ldw + P.N : (int64_t)(P.N - 1) * P.ldw + P.K) * ES);
    const i32x4_t w_rsrc = make_rsrc(P.W, w_bytes);
    // [k x n] weights: KSL rows of 16 NC columns.  bf16: the 32-byte piece (16 columns) t of row k lies in place t ^ (k / 8);
    // fp32: k-row 4 c + e of sixteen lies in row 4 e + c, its 64-byte piece t in place t ^ c (NC = 2: t ^ (c / 2)): the four
    // lane blocks of a fragment read, c = 0 .. 3, then hit different banks.
    constexpr int W_ROWB = TN * ES;
    unsigned woff[2 * NC];                                           // byte offsets of this lane's weight pieces at k0 = 0
    int wk[2 * NC];                                                  // ... and their k inside the slice
#pragma unroll
    for (int i = 0; i < 2 * NC; ++i) {
        if constexpr (KN) {
            const int pos = i * 1024 + lane * 16, q = pos / W_ROWB, in = pos % W_ROWB;
            int piece = in / (16 * ES);
            if constexpr (BF16) {
                wk[i] = q;
                piece ^= (q >> 3) & (NC - 1);
            } else {
                wk[i] = (q & ~15) + (q & 3) * 4 + ((q >> 2) & 3);
                piece ^= (NC == 4 ? q & 3 : NC == 2 ? (q >> 1) & 1 : 0);
            }
            const int n = n0 + piece * 16 + (in % (16 * ES)) / ES;
            woff[i] = n < P.N ? (unsigned)(((int64_t)wk[i] * P.ldw + n) * ES) : OOB;
        } else {
            const int row = (i & 1) * 8 + (lane >> 3), n = n0 + (i >> 1) * 16 + row;
            wk[i] = ((lane & 7) ^ (row >> 1)) * KPL;
            woff[i] = n < P.N ? (unsigned)(((int64_t)n * P.ldw + wk[i]) * ES) : OOB;
        }
    }
    unsigned char *const ring = smem + wave * RING;                  // this wave's own stages: no barrier in the k loop
    const unsigned ring_lds = __builtin_amdgcn_readfirstlane(
        (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)smem) + wave * RING;

    auto issue = [&](int s, int stage) __attribute__((always_inline)) {
        const int k0 = s * KSL;
        const int soff = (int)((KN ? (int64_t)k0 * P.ldw : (int64_t)k0) * ES);
        const unsigned la = ring_lds + stage * STAGE, lw = la + MF * 2048;
        if (k0 + KSL <= P.K) {
#pragma unroll
            for (int i = 0; i < 2 * NC; ++i)
                direct_load_16(w_rsrc, woff[i], soff, lw + i * 1024);
#pragma unroll
            for (int f = 0; f < MF; ++f)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    direct_load_16(arow[f][i] + (k0 + achunk[i] * KPL) * ES, la + f * 2048 + i * 1024);
        } else {                                                     // the ragged tail: weights beyond the range read as zero
#pragma unroll
            for (int i = 0; i < 2 * NC; ++i)
                direct_load_16(w_rsrc, k0 + wk[i] < P.K ? woff[i] : OOB, soff, lw + i * 1024);
#pragma unroll
            for (int f = 0; f < MF; ++f)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int k = k0 + achunk[i] * KPL;
                    direct_load_16(arow[f][i] + (k < P.K ? k : 0) * ES, la + f * 2048 + i * 1024);
                }
        }
    };

    f32x4_t acc[MF][NC];
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
        for (int t = 0; t < NC; ++t)
            acc[f][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // fragments of half h of the slice in `stage`: lane (l16, b) holds row / column l16, chunk 4 h + b
    u32x4_t af[2][MF], wf[2][NC];
    auto read = [&](int s, int stage) __attribute__((always_inline)) {
        const unsigned char *sa = ring + stage * STAGE, *sw = sa + MF * 2048;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int in_block = l16 * 128 + (((4 * h + b) ^ (l16 >> 1)) << 4);
#pragma unroll
            for (int f = 0; f < MF; ++f)
                af[h][f] = *reinterpret_cast<const u32x4_t *>(sa + f * 2048 + in_block);
#pragma unroll
            for (int t = 0; t < NC; ++t) {
                if constexpr (!KN) {
                    wf[h][t] = *reinterpret_cast<const u32x4_t *>(sw + t * 2048 + in_block);
                } else if constexpr (BF16) {
                    const int k = 32 * h + 8 * b + (l16 >> 2);
                    const unsigned char *pw = sw + k * W_ROWB + ((t ^ (b & (NC - 1))) << 5) + (l16 & 3) * 8;
                    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pw));
                    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pw + 4 * W_ROWB));
                    wf[h][t] = __builtin_bit_cast(u32x4_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        wf[h][t][e] = *reinterpret_cast<const unsigned *>(
                            sw + (16 * h + 4 * e + b) * W_ROWB + ((t ^ (NC == 4 ? b : NC == 2 ? b >> 1 : 0)) << 6) + l16 * 4);
                }
            }
        }
        if ((s + 1) * KSL > P.K) {                                   // (what stands for the activations there is anything)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int f = 0; f < MF; ++f)
                    if (s * KSL + (4 * h + b) * KPL >= P.K)
                        af[h][f] = u32x4_t{0u, 0u, 0u, 0u};
        }
    };
    auto multiply = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (BF16) {
#pragma unroll
                for (int t = 0; t < NC; ++t)
#pragma unroll
                    for (int f = 0; f < MF; ++f)
                        acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wf[h][t]),
                                                                           __builtin_bit_cast(bf16x8_t, af[h][f]), acc[f][t], 0, 0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int t = 0; t < NC; ++t)
#pragma unroll
                        for (int f = 0; f < MF; ++f) {
                            const unsigned w = wf[h][t][e], a = af[h][f][e];   // (a bit cast of the element itself takes element 0)
                            acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, w), __builtin_bit_cast(float, a),
                                                                            acc[f][t], 0, 0, 0);
                        }
            }
        }
    };

    // this workgroup's slices [s0, s1), this wave's: s0 + wave, + NW, ...
    const int ns = (P.K + KSL - 1) / KSL;
    const int s0 = (int)(((int64_t)ns * split) / P.ksplit), s1 = (int)(((int64_t)ns * (split + 1)) / P.ksplit);
    const int first = s0 + wave;
    const int count = first < s1 ? (s1 - first + NW - 1) / NW : 0;
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < count)
            issue(first + d * NW, d);
    int stage = 0;
    for (int j = 0; j < count; ++j) {
        const int later = count - 1 - j < D - 1 ? count - 1 - j : D - 1;   // slices still in flight behind this one
        if (later >= 3)
            wait_vmcnt<3 * LPS>();
        else if (later == 2)
            wait_vmcnt<2 * LPS>();
        else if (later == 1)
            wait_vmcnt<LPS>();
        else
            wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
        read(first + j * NW, stage);
        if (j + D < count) {
            __builtin_amdgcn_s_waitcnt(0xC07F);                      // lgkmcnt(0): the fragments have left the stage
            __builtin_amdgcn_sched_barrier(0);
            issue(first + (j + D) * NW, stage);
        }
        multiply();
        stage = stage + 1 == D ? 0 : stage + 1;
    }

    // the waves' partial tiles, row by row, each in its wave's own ring (the last slice has been read)
    {
        float *mine = reinterpret_cast<float *>(ring);
#pragma unroll
        for (int f = 0; f < MF; ++f)
#pragma unroll
            for (int t = 0; t < NC; ++t)                             // lane: row l16, columns 16 t + 4 b .. + 3
                *reinterpret_cast<f32x4_t *>(mine + (f * 16 + l16) * PITCH + t * 16 + b * 4) = acc[f][t];
    }
    __syncthreads();
    f32x4_t sum[QT];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int q = tid + u * 64 * NW;
        sum[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (q < Q) {
            const unsigned char *src = smem + ((q / (TN / 4)) * PITCH + (q % (TN / 4)) * 4) * 4;
#pragma unroll
            for (int w = 0; w < NW; ++w)
                sum[u] += *reinterpret_cast<const f32x4_t *>(src + w * RING);
        }
    }

    if (P.ksplit > 1) {
        constexpr int PART_BYTES = TR * TN * 4;
        auto part_rsrc = [&](int sp) {
            return __builtin_amdgcn_make_buffer_rsrc(P.ws + ((size_t)tile * P.ksplit + sp) * (TR * TN), 0, PART_BYTES, 0x00020000);
        };
        __amdgpu_buffer_rsrc_t rs = part_rsrc(split);
#pragma unroll
        for (int u = 0; u < QT; ++u) {
            const int q = tid + u * 64 * NW;                         // (q >= Q lies beyond num_records: dropped)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, sum[u]), rs, q * 16, 0, COHERENT);
        }
        __builtin_amdgcn_s_waitcnt(0);                               // this wave's stores are acknowledged
        __syncthreads();                                             // ... and every wave's; the LDS tiles are read
        unsigned *arrived = reinterpret_cast<unsigned *>(smem);
        if (tid == 0)
            *arrived = __hip_atomic_fetch_add(&P.counters[tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*arrived != (unsigned)(P.ksplit - 1))
            return;
        if (tid == 0)                                                // ready for the next launch
            __hip_atomic_store(&P.counters[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < QT; ++u)
            sum[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int sp = 0; sp < P.ksplit; ++sp) {
            __amdgpu_buffer_rsrc_t rp = part_rsrc(sp);
#pragma unroll
            for (int u = 0; u < QT; ++u)
                sum[u] += __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rp, (tid + u * 64 * NW) * 16, 0, COHERENT));
        }
    }

#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int s = oseg[u];
        if (s < 0)
            continue;
        if (orecv[u] != nullptr) {
            if (P.copy_wgs == 0)
                if (float *const land = pick(P.land, s))
                    *reinterpret_cast<f32x4_t *>(land + ooff[u]) = rv[u];
            if (P.n_more > 0 && s == P.n_seg - 1)                    // the pairwise schedule's arrivals, in round order
                for (int i = 0; i < P.n_more; ++i) {
                    const f32x4_t t = *reinterpret_cast<const f32x4_t *>(P.more[i] + ooff[u]);
                    if (P.more_land[i] != nullptr)
                        *reinterpret_cast<f32x4_t *>(P.more_land[i] + ooff[u]) = t;
                    rv[u] = rv[u] + t;
                }
            sum[u] = rv[u] + sum[u];                                 // "O <- B_in + O"
        }
        if constexpr (OUT_BF16) {
            bf16x4_t h;
#pragma unroll
            for (int x = 0; x < 4; ++x)
                h[x] = static_cast<__bf16>(sum[u][x]);
            *reinterpret_cast<bf16x4_t *>(static_cast<__bf16 *>(pick(P.out, s)) + ooff[u]) = h;
        } else {
            *reinterpret_cast<f32x4_t *>(static_cast<float *>(pick(P.out, s)) + ooff[u]) = sum[u];
        }
    }
}

template <bool BF16, bool KN, int MF, int NC, bool OUT_BF16, int NW, int SEG>
hipError_t launch_shape(const RowsParams<SEG> &p, hipStream_t s)
{
    const dim3 grid((unsigned)(p.tiles_n * p.tiles_r * p.ksplit + p.copy_wgs)), block(64 * NW);
    hipLaunchKernelGGL((gemm_rows_kernel<BF16, KN, MF, NC, OUT_BF16, NW, SEG>), grid, block, 0, s, p);
    return hipGetLastError();
}

struct RowsShape {
    int mf = 0, nc = 0, ks = 1;                      // mf == 0: not for this kernel
};

template <bool BF16, bool OUT_BF16, int SEG>
hipError_t launch_any(const RowsParams<SEG> &p, bool w_kn, RowsShape t, hipStream_t s)
{
#define CF_ROWS(MF_, NC_, NW_)                                                                                      \
    if (t.mf == MF_ && t.nc == NC_) {                                                                               \
        if constexpr (!(BF16 && NC_ == 1))                                                                          \
            if (w_kn)                                                                                               \
                return launch_shape<BF16, true, MF_, NC_, OUT_BF16, NW_>(p, s);                                     \
        if (!w_kn)                                                                                                  \
            return launch_shape<BF16, false, MF_, NC_, OUT_BF16, NW_>(p, s);                                        \
    }
    CF_ROWS(1, 1, 8) CF_ROWS(1, 2, 8) CF_ROWS(1, 4, 8) CF_ROWS(2, 1, 8) CF_ROWS(2, 2, 8)
    CF_ROWS(2, 4, 4) CF_ROWS(4, 2, 4) CF_ROWS(4, 4, 4)
#undef CF_ROWS
    return hipErrorInvalidValue;
}

// Shape of a launch: the smallest tile (fewest loads in a wave's chain, most compute units at work) whose grid is still one
// round over the chip; 64 x 64 where none is.  bf16 [k x n] weights take at least two column groups (a 32-byte piece of
// every k-row is a quarter of a line).  Measured, us (rows x n x k, [k x n] / [n x k] weights): 8 x 4096 x 1376 32-column tiles
// 4.8 / 4.5, 64-column 5.6 / 5.4; 64 x 8192 x 3584 32 x 64 tiles 15.2 / 14.6, 64 x 64 18.1 / 17.5, 16 x 64 24.5 / -.
// A k range of [k x n] weights on a small part of the chip is split: over four workgroups from 48 slices where a quarter of the
// chip has a tile or less, over two from 64 where half has (us whole / split, bf16: 20 x 136 x 7824 17.4 / 8.5, 28 x 1008 x 7016
// 14.2 / 9.2, 44 x 272 x 5568 11.8 / 8.0; in two 54 x 632 x 4480 10.3 / 8.7, 20 x 1176 x 7224 16.9 / 11.4; at 40 slices 57 x 400 x
// 2512 6.7 / 6.9).  bf16 [n x k] tiles stream as fast unsplit (84 x 160 x 4096 5.9 / 6.8).  Single bf16 steps only: fp32 steps and
// rank steps in one launch take no workspace, so that several of them may be in flight on streams that share one.
RowsShape choose_shape(int64_t rows, int N, int K, bool bf16, bool w_kn, int num_cu)
{
    const Tuning tn = tuning();
    if (tn.rows_mf > 0)
        return RowsShape{tn.rows_mf, w_kn && bf16 && tn.rows_nc == 1 ? 2 : tn.rows_nc, tn.rows_ks};
    static constexpr struct { int mf, nc; } order[] = {{1, 1}, {1, 2}, {2, 1}, {1, 4}, {2, 2}, {2, 4}, {4, 2}, {4, 4}};
    RowsShape t;
    int64_t wgs = 0;
    for (const auto &c : order) {
        if (w_kn && bf16 && c.nc == 1)
            continue;
        t.mf = c.mf;
        t.nc = c.nc;
        wgs = ((rows + 16 * c.mf - 1) / (16 * c.mf)) * ((N + 16 * c.nc - 1) / (16 * c.nc));
        if (wgs <= num_cu)
            break;
    }
    const int slices = (K + (bf16 ? 63 : 31)) / (bf16 ? 64 : 32);
    if (w_kn && bf16 && t.mf * t.nc <= 4)
        t.ks = slices >= 48 && wgs * 4 <= num_cu ? 4 : slices >= 64 && wgs * 2 <= num_cu ? 2 : 1;
    return t;
}

}  // namespace

// Rule between this kernel and the tile kernels, whose cost is theirs to say (gemm_bf16_tile_us, gemm_f32_tile_us).
// fp32: always with tiles under 64 x 64 (one round over the chip: 512 x 1024 x 4096 42 us, the tile kernel 141).  64 x 64 tiles take
// 3.1 us and 4.8 us + 0.0158 us per k a round, which wins over long k ranges (bound by the fp32 MFMAs: 1024 x 1024 x 4096 73 us, 143;
// 512 x 4096 x 4096 142, 175) and not over short ones (2048 x 8192 x 512 206, 153; 768 x 4096 x 256 27, 22; 335 x 2328 x 160 9.6, 9.0)
// nor over grids that the 128 x 128 tiles fill (4096 x 8192 x 4096 2222, 2076).
// bf16: half a round over the chip and less always.  Rows that do not start on a 128-byte line put every slice of theirs on two.
//  * Single steps: 4.6 us, what 64 k cost a round of tiles (by their area, a 64 x 64 tile being 1; 1.12 times that where
//    k-contiguous rows do not start on 128-byte lines) and the megabytes of fp32 output (fitted to 326 steps, rms 0.12).  Of 350 drawn steps of 16 to 1024 rows x 128..8192 x
//    128..8192, each timed on both kernels, 3 are 10 % and more behind the faster one by this rule, 0.2 % on average.  us, this
//    kernel / the tile kernel: 319 x 1688 x 4528 [k x n] 23 / 32 (now in six splits), 213 x 3496 x 6448 33 / 28 (in four),
//    165 x 3472 x 168 [n x k] 5.1 / 6.5, 474 x 1072 x 7768 28.7 / 25.9, 584 x 6456 x 2232 48 / 26.
//  * The steps of a rank step in one launch: a constant, what a round of tiles costs (by their area, a 64 x 64 tile being 1), what
//    64 k cost a round (1.15 times that where the rows of [k x n] weights do not start on 128-byte lines, 1.12 times for [n x k]
//    weights, 1.06 times for the activations alone), and the megabytes of fp32 output with the deliveries that go with it; taken
//    where 0.97 of that is less than the tile kernels' figure.  Fitted (relative error, rms 0.10) to 238 of 500 carried rank steps
//    of 2 x 16 to 8 x 312 rows x 128..8192 x 128..8184, those of 9 us and more.  Of the 500 one is 10 % and more behind the faster
//    kernel by this rule, 0.1 % on average.  us, this kernel / the tile kernel: reduce-scatter 8 x 32 x 5272 x 816 [k x n] 27 / 18,
//    8 x 192 x 512 x 192 [k x n] 10.3 / 7.7, 2 x 192 x 2816 x 5760 [n x k] 47 / 38, 2 x 80 x 4864 x 3712 [k x n] 22 / 30, 2 x 272 x
//    1152 x 2368 [n x k] 16 / 20; all-gather 4 x 302 x 384 x 704 [n x k] 10.7 / 9.4, 2 x 373 x 520 x 3824 [k x n] 21 / 37, 8 x 215 x
//    1088 x 6336 [k x n] 81 / 50.
//  * ... over k ranges of 8192 and more, and under the pairwise schedule of more than two ranks, which that fit has not seen: 1.5 us,
//    7.3 us + 0.235 us per 64 k a round, and 0.02 us per megabyte of W (2 x 96 x 8192 x 8192, 134 MB: 62, the tile kernel 57;
//    4 x 128 x 4096 x 8192 61, 57).
bool gemm_rows_takes(const GemmParams &p, bool bf16, bool w_kn, int num_cu)
{
    const Tuning tn = tuning();
    if (tn.rows == 0 || tn.tile_bm > 0 || tn.tile_f32_bm > 0 || tn.splitk > 0 || tn.staged || tn.deep >= 0 || tn.prefetch >= 0 ||
        tn.xcd_steps >= 0 || tn.k_rotate >= 0 || tn.xcd_bands > 0 || tn.stream_recv >= 0 || tn.mfma16 >= 0 || tn.persist_wgs > 0)
        return false;                                // an override asks for one of the tile kernels
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || p.a_t || p.wait_flag != nullptr || p.cp_bytes != 0)
        return false;
    const int64_t es = bf16 ? 2 : 4, lim = (int64_t)1 << 31;
    if ((int64_t)(w_kn ? p.K : p.N) * p.ldw * es >= lim)
        return false;
    const int64_t rows = (int64_t)p.M * (p.n_steps > 0 ? p.n_steps : 1);
    const RowsShape t = choose_shape(rows, p.N, p.K, bf16, w_kn, num_cu);
    const int64_t wgs = ((rows + 16 * t.mf - 1) / (16 * t.mf)) * ((p.N + 16 * t.nc - 1) / (16 * t.nc));
    if (wgs >= ((int64_t)1 << 24))
        return false;
    if (tn.rows_mf > 0 || (bf16 ? wgs * 2 <= num_cu : t.mf * t.nc < 16))
        return true;
    const int64_t rounds = (wgs + num_cu - 1) / num_cu;
    if (!bf16)
        return 3.1 + rounds * (4.8 + 0.0158 * p.K) < gemm_f32_tile_us(p, num_cu);
    const double kt = (p.K + 63) / 64, adds = gemm_share_with_recv(p), area = t.mf * t.nc / 16.0, mo = 4e-6 * rows * p.N;
    const bool off_lines = p.lda % 64 != 0 || (!w_kn && p.ldw % 64 != 0);
    if (p.n_steps > 0 && p.K < 8192 && (adds == 0.0 || adds >= 0.5)) {
        const double slices = kt * (w_kn && p.ldw % 64 != 0 ? 1.15 : !w_kn && p.ldw % 64 != 0 ? 1.12 : p.lda % 64 != 0 ? 1.06 : 1.0);
        return 0.97 * (3.9 + rounds * (2.2 * area + slices * (0.067 + 0.148 * area)) + (0.79 + 0.4 * adds) * mo) < gemm_bf16_rank_step_us(p, num_cu);
    }
    const double slices = kt * (off_lines ? 1.12 : 1.0);
    const double us = p.n_steps > 0 ? 1.5 + rounds * (3.6 + 3.7 * area + 0.235 * slices) + 0.02e-6 * 2.0 * p.N * p.K
                                    : 4.6 + rounds * slices * (0.035 + 0.177 * area) + (0.38 + 0.2 * adds) * mo;
    return us < gemm_bf16_tile_us(p, num_cu);
}

size_t gemm_rows_ws_bytes(const GemmParams &p, bool bf16, bool w_kn, int num_cu)
{
    if (!bf16 || p.n_steps > 0 || !gemm_rows_takes(p, bf16, w_kn, num_cu))
        return 0;
    const RowsShape t = choose_shape(p.M, p.N, p.K, bf16, w_kn, num_cu);
    const size_t tiles = (size_t)((p.N + 16 * t.nc - 1) / (16 * t.nc)) * (size_t)((p.M + 16 * t.mf - 1) / (16 * t.mf));
    return t.ks > 1 ? tiles * t.ks * (256 * t.mf * t.nc) * sizeof(float) : 0;
}

template <int SEG>
static hipError_t launch_segments(const GemmParams &g, bool bf16, bool w_kn, bool out_bf16, hipStream_t s, int num_cu)
{
    RowsParams<SEG> p;
    p.W = g.W;
    p.lda = g.lda;
    p.ldw = g.ldw;
    p.ldo = g.ldo;
    p.seg_rows = g.M;
    p.n_seg = g.n_steps > 0 ? g.n_steps : 1;
    p.N = g.N;
    p.K = g.K;
    bool lands_slice = false;
    for (int j = 0; j < SEG; ++j) {
        const bool in = j < p.n_seg;
        p.A[j] = !in ? nullptr : g.n_steps > 0 ? g.A_step[j] : g.A;
        p.recv[j] = !in ? nullptr : g.n_steps > 0 ? g.recv_step[j] : g.recv;
        p.out[j] = !in ? nullptr : g.n_steps > 0 ? g.out_step[j] : g.out;
        p.land[j] = in && g.n_steps > 0 ? static_cast<float *>(g.land_step[j]) : nullptr;
        lands_slice = lands_slice || (p.land[j] != nullptr && p.recv[j] == nullptr);
    }
    p.n_more = g.n_recv_more;
    for (int i = 0; i < RowsParams<SEG>::MORE; ++i) {
        p.more[i] = i < p.n_more ? g.recv_more[i] : nullptr;
        p.more_land[i] = i < p.n_more ? g.land_more[i] : nullptr;
    }
    const int64_t rows = (int64_t)p.seg_rows * p.n_seg;
    const RowsShape t = choose_shape(rows, p.N, p.K, bf16, w_kn, num_cu);
    p.tiles_n = (p.N + 16 * t.nc - 1) / (16 * t.nc);
    p.tiles_r = (int)((rows + 16 * t.mf - 1) / (16 * t.mf));
    const size_t tiles = (size_t)p.tiles_n * p.tiles_r;
    p.ksplit = t.ks;
    if (p.ksplit > 1 && (!bf16 || g.ws == nullptr || g.counters == nullptr || tiles > (size_t)g.max_tiles ||
                         tiles * p.ksplit * (256 * t.mf * t.nc) * sizeof(float) > g.ws_bytes))
        p.ksplit = 1;
    p.ws = g.ws;
    p.counters = g.counters;
    p.copy_wgs = 0;
    if (lands_slice) {
        const int64_t chunks = rows * p.K * (bf16 ? 2 : 4) / 16;
        const int64_t want = (chunks + 2047) / 2048;
        p.copy_wgs = (int)(want < 1 ? 1 : (want < num_cu ? want : num_cu));
    }
    if (!bf16)
        return launch_any<false, false>(p, w_kn, t, s);
    return out_bf16 ? launch_any<true, true>(p, w_kn, t, s) : launch_any<true, false>(p, w_kn, t, s);
}

hipError_t launch_gemm_rows(const GemmParams &g, bool bf16, bool w_kn, bool out_bf16, hipStream_t s, int num_cu)
{
    if (g.n_steps == 0 && g.n_recv_more <= RowsParams<1>::MORE)
        return launch_segments<1>(g, bf16, w_kn, out_bf16, s, num_cu);
    return launch_segments<GemmParams::MAX_STEPS>(g, bf16, w_kn, out_bf16, s, num_cu);
}

}  // namespace cf
