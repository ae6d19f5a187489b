// bf16 x bf16 -> fp32 chunk GEMM for gfx950, direct-to-LDS variant.
//
//  * Operand tiles go from global memory straight into LDS (buffer_load ... lds,
//    16 bytes per lane) without passing through registers.
//  * A [k x n] weight tile stays in its natural order in LDS and is read back
//    with the transposing LDS read (ds_read_b64_tr_b16); a [n x k] weight tile
//    and the activations are read with plain 16-byte reads.
//  * k-tiles of 64 (full 128-byte lines of the k-contiguous operands) in NS = 2..4
//    LDS stages (as many as the tile shape leaves room for in 160 KiB).  A k-tile is consumed in four 16-wide slices; fragments are
//    double-buffered in registers and the LDS reads of slice s+1 are issued under
//    the first MFMAs of slice s.  The one barrier per k-tile sits before the last
//    slice: by then every wave has read all of the tile, so the freed stage's
//    next tile can be requested, and the next tile (requested NS-1 barriers
//    earlier) is published; its first fragments are fetched under the MFMAs of
//    the last slice, so the matrix pipe does not drain at tile boundaries.
//  * The direct loads of a tile are not issued as one burst: each wave issues one
//    after every few MFMAs.  A burst fills the address queue of the texture unit
//    and the wave -- which issues in order -- then cannot feed the matrix pipe
//    until its last load has been accepted.
//  * Fused epilogue: Alg. 2 "O <- B_in + O", "B_out <- O", or Alg. 1's in-place
//    slice store, with bounds-checked buffer loads/stores in whole 128-byte lines;
//    B_in, read once, goes on to the landing buffer from the same registers.
//
// Layout in LDS (per stage):
//   activations / [n x k] weights: 128-byte rows (64 k) of eight 16-byte chunks,
//     two rows per 256-byte line; chunk index and line half are XOR-ed with row
//     bits 1..3 so that the 16-byte fragment reads of 16 consecutive rows hit 16
//     different bank groups.  A wave-wide direct load fills 1 KiB of contiguous
//     LDS (8 rows); the swizzle is applied by choosing which global chunk each
//     lane fetches.
//   [k x n] weights: one k-row of BN bf16 after the other; the 64-byte groups of
//     a row are XOR-ed with (k & 3) so that the four rows a transposing read
//     touches fall into different banks.
// Rows / columns beyond the matrix and the k tail read as zero through the
// buffer bounds check (such a lane is given an offset beyond num_records).
#include "cf_internal.h"

#include <cstdio>
#include <cstdlib>
#include <type_traits>
namespace cf {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

constexpr int BK = 64;                    // k extent of one LDS stage
constexpr int KS = BK / 16;               // 16-wide k-slices (one MFMA deep) per stage
constexpr unsigned OOB = 0x80000000u;     // byte offset beyond any buffer this kernel accepts

// Byte offset of 16-byte chunk kc (0..7) of tile row `row` (128-byte rows).  Only row bits
// 0..3 enter the swizzle, so rows 32 apart differ by a constant 4096 bytes, and the chunk
// pair of k-slice ks is reached by XOR-ing (ks << 5) into the offset of slice 0.
__device__ __forceinline__ int swz_row(int row, int kc)
{
    const int r0 = row & 1, r1 = (row >> 1) & 1, r2 = (row >> 2) & 1, r3 = (row >> 3) & 1;
    const int half = r0 ^ r3;
    const int kcp = kc ^ ((r1 << 2) | (r2 << 1) | r3);
    return ((row >> 1) << 8) + (half << 7) + (kcp << 4);
}

// Inverse: which (row, kc) lives at bytes [pos, pos+16) of a tile.
__device__ __forceinline__ void unswz_row(int pos, int &row, int &kc)
{
    const int rp = pos >> 8, half = (pos >> 7) & 1, kcp = (pos >> 4) & 7;
    const int r1 = rp & 1, r2 = (rp >> 1) & 1, r3 = (rp >> 2) & 1;
    row = (rp << 1) | (half ^ r3);
    kc = kcp ^ ((r1 << 2) | (r2 << 1) | r3);
}

// Raw buffer descriptor: base, stride 0, num_records bytes, 32-bit raw data format.
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

// One wave-wide 16-byte-per-lane load from global memory straight into LDS:
// lane L's 16 bytes land at LDS byte address lds_addr + 16 L.  Issued as inline
// assembly so that the compiler does not order later LDS reads of OTHER stages
// behind it; completion is awaited explicitly (vmcnt) before the barrier that
// publishes the stage.
__device__ __forceinline__ void direct_load_16(i32x4_t rsrc, unsigned voffset, int soffset, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voffset), "s"(rsrc), "s"(soffset)
                 : "memory");   // M0 is written here and used by nothing else in this kernel
}

// s_waitcnt on the vector-memory counter only (gfx9 encoding: vmcnt in bits 3:0 and 15:14).
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// Scheduling hint for one slice phase: after each MFMA up to RPM LDS reads, until REMAIN reads are placed.
template <int REMAIN, int RPM>
__device__ __forceinline__ void interleave_mfma_reads()
{
    if constexpr (REMAIN > 0) {
        constexpr int now = REMAIN < RPM ? REMAIN : RPM;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, now, 0);   // `now` LDS reads
        interleave_mfma_reads<REMAIN - now, RPM>();
    }
}

__device__ __forceinline__ int xcd_remap(int pid, int total)
{
    constexpr int NXCD = 8;
    const int q = total / NXCD, rem = total % NXCD;
    const int xcd = pid % NXCD, idx = pid / NXCD;
    return xcd * q + (xcd < rem ? xcd : rem) + idx;
}

// A_T: the left operand is stored [K x M] (see GemmParams::a_t); its tile then lives in LDS like a
// [k x n] weight tile and is read with the transposing LDS read as well.
// PERSIST: one launch runs all steps of a rank step (GemmParams::n_steps, see the work-item loop below).
// RECV: a step of the launch adds a received partial (fp32 output only).
// NT: B_in, its landed copy and the output pass the caches by (GemmParams::non_temporal, set by the launcher).
// MF16: the 256x256 tile's main loop on v_mfma_f32_16x16x32_bf16 instead of v_mfma_f32_32x32x16_bf16 -- the same
// flops from twice as many instructions that each write a quarter of the accumulator registers, which costs the chip
// less power per flop (measured) and, where the launch is paced by the power limit, time.  A 32x32 sub-tile of the
// accumulators is then four 16x16 tiles: registers 4g .. 4g+3 with g = 2x + y hold rows 16x + (lane & 15), columns
// 16y + 4 (lane >> 4) .. + 3.  A k-tile is two 32-wide slices, each consumed in four quarter phases (one 32-row block
// of the wave tile per phase).
template <int BM, int BN, int WGM, int WGN, int NS, bool SPREAD, bool W_KN, bool OUT_BF16, bool RECV, bool A_T = false,
          bool PERSIST = false, bool MF16 = false, int HOPS = 0, bool NT = false>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_dl_kernel(GemmParams P, int tiles_m, int tiles_n)
{
    static_assert(!MF16 || (SPREAD && NS == 2), "16x16x32 main loop: 256x256 tile");
    static_assert(!RECV || !OUT_BF16, "received partials are fp32, and so is their sum");
    static_assert(!A_T || (W_KN && !OUT_BF16), "the transposed left operand comes with [k x n] weights and fp32 output");
    constexpr int NW = WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
    constexpr int A_LD = (A_BYTES / 1024) / NW;     // 1 KiB wave-loads of the A tile per wave
    constexpr int B_LD = (B_BYTES / 1024) / NW;
    constexpr int LPT = A_LD + B_LD;                // direct loads per wave per k-tile
    static_assert(A_LD >= 1 && B_LD >= 1 && (A_BYTES / 1024) % NW == 0 && (B_BYTES / 1024) % NW == 0, "tile vs waves");
    // LDS: NSA stages of the left-operand tile, then NS stages of the weight tile.  The 256x256 tile (SPREAD)
    // fills the 160 KiB with THREE left-operand stages and two weight stages: its weight loads go out first
    // after the barrier that frees their stage and its left-operand loads one k-tile further ahead (see the
    // steady state below), which lengthens the time every load has to arrive.
    constexpr int NSA = SPREAD ? NS + 1 : NS;
    constexpr int W_BASE = NSA * A_BYTES;
    // wave-private scratch of the epilogue's stores (4 KiB per wave): a left-operand stage that no load targets any
    // more (after a barrier: every wave is done reading the stages) -- the third stage of the 256x256 tile, else the first
    constexpr int E_SCR_BYTES = 4096;
    static_assert(NW * E_SCR_BYTES <= A_BYTES || !SPREAD, "epilogue scratch inside one left-operand stage");
    static_assert(NW * E_SCR_BYTES <= NSA * A_BYTES + NS * B_BYTES, "epilogue scratch inside the stages");
    static_assert(NS >= 2 && NS <= 4 && NSA * A_BYTES + NS * B_BYTES <= 160 * 1024, "LDS budget");
    static_assert(KS == 4, "the slice schedule below is written for four slices per stage");
    constexpr int W_ROWB = BN * 2;                   // bytes of one k-row of a [k x n] weight tile
    constexpr int A_ROWB = BM * 2;                   // bytes of one k-row of a [k x m] left-operand tile

    __shared__ __attribute__((aligned(1024))) unsigned char smem[NSA * A_BYTES + NS * B_BYTES];

    const int tid0 = threadIdx.x;

    // Workgroups beyond the GEMM's own grid carry the emulated delivery of the NEXT step (what the ring
    // neighbour sends while this step computes): a streaming copy that shares the launch with the GEMM,
    // so that no second stream, event or inter-queue wait sits between two step kernels.
    const int gemm_wgs = tiles_m * tiles_n * P.splits;
    if (!PERSIST && (int)blockIdx.x >= gemm_wgs) {
        const u32x4_t *src = static_cast<const u32x4_t *>(P.cp_src);
        u32x4_t *dst = static_cast<u32x4_t *>(P.cp_dst);
        const size_t n16 = P.cp_bytes / 16;
        const size_t stride = (size_t)P.cp_wgs * (64 * NW);
        size_t i = (size_t)((int)blockIdx.x - gemm_wgs) * (64 * NW) + tid0;
        for (; i + 3 * stride < n16; i += 4 * stride) {
            const u32x4_t v0 = __builtin_nontemporal_load(&src[i]);
            const u32x4_t v1 = __builtin_nontemporal_load(&src[i + stride]);
            const u32x4_t v2 = __builtin_nontemporal_load(&src[i + 2 * stride]);
            const u32x4_t v3 = __builtin_nontemporal_load(&src[i + 3 * stride]);
            __builtin_nontemporal_store(v0, &dst[i]);
            __builtin_nontemporal_store(v1, &dst[i + stride]);
            __builtin_nontemporal_store(v2, &dst[i + 2 * stride]);
            __builtin_nontemporal_store(v3, &dst[i + 3 * stride]);
        }
        for (; i < n16; i += stride)
            __builtin_nontemporal_store(__builtin_nontemporal_load(&src[i]), &dst[i]);
        return;
    }

    // Persistent mode (GemmParams::n_steps > 0): one launch runs ALL steps of a rank step.  The work items
    // (step, output tile) are dealt out round robin, step-major, to the workgroups of a grid that fills the
    // chip once; a workgroup goes on to its next item as soon as it is done with the last one, so tiles of
    // different steps run side by side (the chunk GEMMs of Alg. 1 / Alg. 2 do not depend on each other; only
    // the add of B_in / the arrival of the slice does, and both are there before the launch) and nothing
    // is launched, drained or refilled between steps.  Every workgroup's loop is finite: the kernel exits.
    // (The k range of a persistent launch is never split, and the kernel has no code for it: a path on which the splits that
    // finish first leave with requests of B_in outstanding made the compiler drain the request queue on every trip of six
    // main loops.  us with / without that path: reduce-scatter step 1408 x 6400 x 8128 236 / 193, rank steps 8 x 700 x 8192 x
    // 3584 307 / 295, 8 x 960 x 4096 x 2048 140 / 133.)
    const int tiles_per_step = tiles_m * tiles_n * (PERSIST ? 1 : P.splits);
    // XCD-per-step mapping (GemmParams::xcd_steps): XCD x (workgroups x, x+8, ...) runs the steps x, x+8, ...
    // whole, so a step's own operand (A of the step) passes through one L2 only, instead of through all
    // eight when every XCD holds a band of every step's tiles.  With GemmParams::xcd_bands = NB > 1 the XCDs form
    // 8 / NB step groups x NB column bands instead: XCD x runs the steps x / NB, x / NB + 8 / NB, ... on the tile
    // columns of band x % NB only -- fewer weight bands and more left-operand bands per L2, which is less traffic
    // where a step has few tile rows and many tile columns.
    const bool by_xcd = PERSIST && P.xcd_steps;
    const int xcd_nb = by_xcd ? P.xcd_bands : 1, xcd_groups = 8 / xcd_nb;
    const int xcd_grp = (int)(blockIdx.x & 7) / xcd_nb, xcd_band = (int)(blockIdx.x & 7) % xcd_nb;
    const int item_stride = by_xcd ? (int)(gridDim.x >> 3) : (int)gridDim.x;
    const int n_items = PERSIST ? (by_xcd ? (tiles_per_step * P.n_steps) >> 3 : tiles_per_step * P.n_steps) : 0;
    int item = by_xcd ? (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    do {
    // Lane and wave indices are taken anew for every work item: what is derived from them then lives
    // from its first use in this item, not across the whole loop.
    int tid = tid0;
    if constexpr (PERSIST)
        asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WGM, wn = wave / WGM;
    // the XCD's items: all (step, tile row) pairs of one tile column, then the next column of its band
    const int rows_x = by_xcd ? (P.n_steps / xcd_groups) * tiles_m : 1;       // (step, tile row) pairs of this XCD
    const int step_i = PERSIST ? (by_xcd ? xcd_grp + xcd_groups * ((item % rows_x) / tiles_m) : item / tiles_per_step) : 0;
    const void *const cA = PERSIST ? P.A_step[step_i] : P.A;
    const float *const cRecv = PERSIST ? P.recv_step[step_i] : P.recv;
    void *const cLand = PERSIST ? P.land_step[step_i] : nullptr;   // where the delivery is to land, if this kernel carries it
    void *const cOut = PERSIST ? P.out_step[step_i] : P.out;
    const unsigned *const cFlag = PERSIST ? nullptr : P.wait_flag;
    // further received partials (GemmParams::recv_more): in a persistent launch they belong to the last step only
    const int n_more = (!PERSIST || step_i == P.n_steps - 1) ? P.n_recv_more : 0;

    // Work item = (output tile, k-split); the splits of a tile are neighbours in the remapped order.
    const int splits = PERSIST ? 1 : P.splits;
    const int work = by_xcd ? (xcd_band * (tiles_n / xcd_nb) + item / rows_x) * tiles_m + (item % rows_x) % tiles_m
                            : xcd_remap(PERSIST ? item % tiles_per_step : (int)blockIdx.x, tiles_per_step);
    const int tile = work / splits, split = work % splits;
    const int m0 = (tile % tiles_m) * BM;
    const int n0 = (tile / tiles_m) * BN;
    const int M = P.M, N = P.N, K = P.K;
    const int nk_all = (K + BK - 1) / BK;
    const int ktb = (int)(((long long)nk_all * split) / splits);          // first k-tile of this split
    const int nk = (int)(((long long)nk_all * (split + 1)) / splits) - ktb; // its number of k-tiles

    // Device-side wait for an emulated delivery: one lane polls the flag with device-coherent loads,
    // sleeping between polls, for at most spin_limit polls (every wave reaches the barrier either way).
    // The delivery was written by another kernel while this one was already running, possibly through
    // the L2 of another XCD: the caches this kernel reads through may hold older contents of those
    // addresses.  So what follows the wait is either an agent-scope acquire (operand loads: L1 and the
    // non-local L2 lines are invalidated once per workgroup) or loads with the device-coherent cache
    // policy (the B_in loads of the epilogue, which are read once anyway).
    auto wait_delivery = [&](bool acquire) __attribute__((always_inline)) {
        if (cFlag != nullptr) {
            if (tid == 0) {
                unsigned n = 0;
                while (__hip_atomic_load(cFlag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == 0u) {
                    if (++n >= P.spin_limit) {
                        __hip_atomic_fetch_or(P.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(32);
                }
            }
            __syncthreads();
            if (acquire)
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
    };
    if (P.wait_at_start)
        wait_delivery(true);

    // Buffer resources; all byte extents are below 2^31 (host-checked).
    const unsigned a_bytes = (unsigned)((A_T ? ((int64_t)(K - 1) * P.lda + M) : ((int64_t)(M - 1) * P.lda + K)) * 2);
    const unsigned w_bytes = (unsigned)((W_KN ? ((int64_t)(K - 1) * P.ldw + N) : ((int64_t)(N - 1) * P.ldw + K)) * 2);
    i32x4_t a_rsrc = make_rsrc(cA, a_bytes);
    i32x4_t w_rsrc = make_rsrc(P.W, w_bytes);
    const unsigned lds_base = __builtin_amdgcn_readfirstlane(
        (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)smem);

    // Per-lane global byte offsets (k0 = 0) of every wave-load, and the k index of its chunk for the tail test.
    unsigned a_off[A_LD], b_off[B_LD];
#pragma unroll
    for (int j = 0; j < A_LD; ++j) {
        const int pos = (j * NW + wave) * 1024 + lane * 16;
        if constexpr (A_T) {
            const int k = pos / A_ROWB, inrow = pos % A_ROWB;
            const int q = (inrow >> 6) ^ (k & 3);
            const int c4 = ((inrow >> 4) & 3) ^ (MF16 ? ((k >> 4) & 1) << 1 : 0);    // (as the [k x n] weights, below)
            const int gm = m0 + q * 32 + c4 * 8;
            a_off[j] = gm < M ? (unsigned)(((int64_t)k * P.lda + gm) * 2) : OOB;
        } else {
            int row, kc;
            unswz_row(pos, row, kc);
            const int gm = m0 + row;
            a_off[j] = gm < M ? (unsigned)(((int64_t)gm * P.lda + kc * 8) * 2) : OOB;
        }
    }
#pragma unroll
    for (int j = 0; j < B_LD; ++j) {
        const int pos = (j * NW + wave) * 1024 + lane * 16;
        if constexpr (W_KN) {
            const int k = pos / W_ROWB, inrow = pos % W_ROWB;
            const int q = (inrow >> 6) ^ (k & 3);
            // (MF16: the two 32-byte halves of a 64-byte group change places in the rows with odd k / 16: the sixteen-lane
            // blocks of a transposing read then hold different 8-row groups of k for the SAME columns, and the two
            // blocks that are served together -- lanes 0..15 and 16..31: k / 8 = 0 and 2, or 1 and 3, see the
            // fragment addressing -- must not fall into the same banks)
            const int c4 = ((inrow >> 4) & 3) ^ (MF16 ? ((k >> 4) & 1) << 1 : 0);
            const int gn = n0 + q * 32 + c4 * 8;
            b_off[j] = gn < N ? (unsigned)(((int64_t)k * P.ldw + gn) * 2) : OOB;
        } else {
            int row, kc;
            unswz_row(pos, row, kc);
            const int gn = n0 + row;
            b_off[j] = gn < N ? (unsigned)(((int64_t)gn * P.ldw + kc * 8) * 2) : OOB;
        }
    }
    // k index (inside a k-tile) of the chunk wave-load j of a tile fetches for this lane: needed only where a
    // k-tile is ragged or beyond the range, so it is recomputed there (from an opaque copy of the lane index:
    // kept in registers across the main loop it costs eight of them)
    auto chunk_k = [&](int j, bool k_major, int rowb) __attribute__((always_inline)) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int pos = (j * NW + wave) * 1024 + ln * 16;
        if (k_major)
            return pos / rowb;
        int row, kc;
        unswz_row(pos, row, kc);
        return kc * 8;
    };
    const int w_kstep = W_KN ? (int)(P.ldw * 2) : 2;   // bytes per unit of k along W
    const int a_kstep = A_T ? (int)(P.lda * 2) : 2;    // ... and along the left operand
    // MF16 (whole tiles only: no lane is out of range): wave-load j of a tile fetches, lane by lane, what wave-load 0
    // fetches 64 rows further on (a tile stored by k-rows: what wave-load j - 2 fetches 32 k-rows further on -- the
    // 32-byte halves change places every 16 k-rows), so one per-lane offset per operand (two if stored by k-rows) is
    // kept and the distance goes into the scalar part of the address
    constexpr int A_JP = (MF16 && A_T) ? 2 : 1;      // wave-loads of a left-operand tile with an offset register of their own
    constexpr int W_JP = (MF16 && W_KN) ? 2 : 1;     // ... of a weight tile
    const int a_jstep = MF16 ? (int)((A_T ? 16 : 64) * P.lda * 2) : 0;
    const int w_jstep = MF16 ? (int)((W_KN ? 16 : 64) * P.ldw * 2) : 0;
    // per-lane offset register and scalar distance of wave-load j of an operand
    auto a_reg = [](int j) { return MF16 ? j % A_JP : j; };
    auto a_dist = [&](int j) __attribute__((always_inline)) { return (j - j % A_JP) * a_jstep; };
    auto w_reg = [](int j) { return MF16 ? j % W_JP : j; };
    auto w_dist = [&](int j) __attribute__((always_inline)) { return (j - j % W_JP) * w_jstep; };

    // Direct load number `idx` (0 .. LPT-1: the A wave-loads, then the W wave-loads) of local k-tile
    // kt into `stage`.  Where the waits count on it -- in the prologue, and in the loops that test their loads -- a tile beyond
    // the end of this split's k range is requested all the same, with every lane out of range: it reads zeros and moves no
    // data.
    // Persistent mode: the workgroups of step group g of G (XCD x of 8 without column bands) walk the k range
    // starting g/G of the way in and wrap around, so that the XCDs that read the same weight tiles -- and would ask
    // for the same lines at the same moment -- are spread over the k range (measured: 1 % of the pair's rank step).
    // The sum over k is taken in that rotated order: deterministic for a given launch, last-bit different between
    // step groups.
    const int rot = (PERSIST && P.k_rotate) ? (xcd_grp * nk_all) / xcd_groups : 0;
    auto ktile = [&](int kt) __attribute__((always_inline)) {                           // global k-tile of this item's local k-tile kt
        const int kk = ktb + kt + rot;
        return kk >= nk_all ? kk - nk_all : kk;
    };
    // With WHOLE_K (a k-tile known to be whole, and inside the range) the load is issued without any test: a
    // branch after every MFMA segment of the main loop costs more than it looks (measured: 4 - 6 % of the launch,
    // and a select on the offset still 1 %).
    auto issue_load = [&](int kt, int stage_a, int stage_w, auto idx_tag, auto whole_k_tag) __attribute__((always_inline)) {
        constexpr int idx = decltype(idx_tag)::value;
        constexpr bool WHOLE_K = decltype(whole_k_tag)::value;
        const int k0 = ktile(kt) * BK;
        const unsigned sa = lds_base + stage_a * A_BYTES + wave * 1024;
        const unsigned sw = lds_base + W_BASE + stage_w * B_BYTES + wave * 1024;
        if constexpr (WHOLE_K) {
            if constexpr (idx < A_LD)
                direct_load_16(a_rsrc, a_off[a_reg(idx)], k0 * a_kstep + a_dist(idx), sa + idx * NW * 1024);
            else
                direct_load_16(w_rsrc, b_off[w_reg(idx - A_LD)], k0 * w_kstep + w_dist(idx - A_LD), sw + (idx - A_LD) * NW * 1024);
            return;
        }
        const bool full = kt < nk && (k0 + BK) <= K;     // uniform: the common case needs no per-lane test
        if (full) {
            if constexpr (idx < A_LD)
                direct_load_16(a_rsrc, a_off[a_reg(idx)], k0 * a_kstep + a_dist(idx), sa + idx * NW * 1024);
            else
                direct_load_16(w_rsrc, b_off[w_reg(idx - A_LD)], k0 * w_kstep + w_dist(idx - A_LD), sw + (idx - A_LD) * NW * 1024);
        } else {
            const bool none = kt >= nk;
            const int klim = none ? -1 : K;              // chunks at k >= klim read as zero
            const int ks0 = none ? 0 : k0;
            if constexpr (idx < A_LD) {
                const unsigned off = (k0 + chunk_k(idx, A_T, A_ROWB)) >= klim ? OOB : a_off[a_reg(idx)];
                direct_load_16(a_rsrc, off, ks0 * a_kstep + a_dist(idx), sa + idx * NW * 1024);
            } else {
                constexpr int j = idx - A_LD;
                const unsigned off = (k0 + chunk_k(j, W_KN, W_ROWB)) >= klim ? OOB : b_off[w_reg(j)];
                direct_load_16(w_rsrc, off, ks0 * w_kstep + w_dist(j), sw + j * NW * 1024);
            }
        }
    };
    auto issue_range = [&](int kt, int stage_a, int stage_w, auto lo_tag, auto hi_tag) __attribute__((always_inline)) {   // loads [lo, hi) of a tile
        constexpr int lo = decltype(lo_tag)::value, hi = decltype(hi_tag)::value;
        static_assert(hi - lo <= 12, "at most twelve direct loads per tile and wave");
        const int k0 = ktile(kt) * BK;
        const unsigned sa = lds_base + stage_a * A_BYTES + wave * 1024;
        const unsigned sw = lds_base + W_BASE + stage_w * B_BYTES + wave * 1024;
        if (kt < nk && (k0 + BK) <= K) {                 // uniform: the common case, no per-lane test
#pragma unroll
            for (int idx = lo; idx < hi; ++idx) {
                if (idx < A_LD)
                    direct_load_16(a_rsrc, a_off[idx < A_LD ? a_reg(idx) : 0], k0 * a_kstep + a_dist(idx), sa + idx * NW * 1024);
                else
                    direct_load_16(w_rsrc, b_off[idx >= A_LD ? w_reg(idx - A_LD) : 0], k0 * w_kstep + w_dist(idx - A_LD),
                                   sw + (idx - A_LD) * NW * 1024);
            }
        } else {
            if constexpr (lo + 0 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 0>{}, std::false_type{});
            if constexpr (lo + 1 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 1>{}, std::false_type{});
            if constexpr (lo + 2 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 2>{}, std::false_type{});
            if constexpr (lo + 3 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 3>{}, std::false_type{});
            if constexpr (lo + 4 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 4>{}, std::false_type{});
            if constexpr (lo + 5 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 5>{}, std::false_type{});
            if constexpr (lo + 6 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 6>{}, std::false_type{});
            if constexpr (lo + 7 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 7>{}, std::false_type{});
            if constexpr (lo + 8 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 8>{}, std::false_type{});
            if constexpr (lo + 9 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 9>{}, std::false_type{});
            if constexpr (lo + 10 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 10>{}, std::false_type{});
            if constexpr (lo + 11 < hi) issue_load(kt, stage_a, stage_w, std::integral_constant<int, lo + 11>{}, std::false_type{});
        }
    };

    // (MF16: the accumulators as the 16x16 tiles the MFMAs write, acc4[i][j][g] = registers 4g .. 4g+3 of sub-tile (i, j))
    f32x16_t acc[MF16 ? 1 : TM][MF16 ? 1 : TN];
    f32x4_t acc4[MF16 ? TM : 1][MF16 ? TN : 1][4];
    if constexpr (MF16) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    acc4[i][j][g] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    acc[i][j][e] = 0.0f;
    }
    // registers 4g .. 4g+3 of sub-tile (i, j)
    auto acc_get = [&](int i, int j, int g) __attribute__((always_inline)) {
        if constexpr (MF16) {
            return acc4[i][j][g];
        } else {
            f32x4_t o;
            o[0] = acc[i][j][4 * g + 0];
            o[1] = acc[i][j][4 * g + 1];
            o[2] = acc[i][j][4 * g + 2];
            o[3] = acc[i][j][4 * g + 3];
            return o;
        }
    };
    auto acc_set = [&](int i, int j, int g, f32x4_t v) __attribute__((always_inline)) {
        if constexpr (MF16) {
            acc4[i][j][g] = v;
        } else {
            acc[i][j][4 * g + 0] = v[0];
            acc[i][j][4 * g + 1] = v[1];
            acc[i][j][4 * g + 2] = v[2];
            acc[i][j][4 * g + 3] = v[3];
        }
    };

    // All-gather with the delivery carried by the consumer (GemmParams::land_step): the left operand comes in from the
    // neighbour's buffer, and each of its k-tiles is stored on to the landing buffer by ONE of the workgroups that
    // load it: the work item of tile column c takes the local k-tiles c, c + tiles_n, c + 2 tiles_n, ...  (All
    // items of a step and tile row walk k in the same order: the k rotation comes with whole steps per XCD.)
    // Every wave stores the 4 KiB it loaded itself -- it reads them back from the stage, whole 128-byte rows per
    // eight lanes, at the global offsets it fetched them from -- so its own vmcnt wait is all the ordering needed.
    constexpr bool CARRY_A = PERSIST && !A_T;
    // Weight gradient likewise (GemmParams::hop_tiles): the operand that travels is either one, and comes in from one buffer per
    // block of rows, to whose descriptor the loads go over with the first k-tile of the block (one test per k-tile).  An
    // instance of its own: in the plain one the tests cost weight-gradient steps 1.5 % (8192 rows into 8192 x 3584 381 / 387 us).
    // HOPS: 1 the left one, 2 the right one.
    static_assert(HOPS == 0 || (PERSIST && A_T && MF16 && !RECV), "a weight gradient on whole tiles, written once");
    constexpr bool hop_right = HOPS == 2;
    int carry_at = (CARRY_A && cLand != nullptr && cRecv == nullptr) ? tile / tiles_m : 0x7fffffff;
    int hop_at = 0x7fffffff;                             // the k-tile with which the next block of rows begins
    if (HOPS != 0) {
        carry_at = hop_right ? tile % tiles_m : tile / tiles_m;
        hop_at = P.hop_tiles;
    }
    const int carry_step = hop_right ? tiles_m : tiles_n;
    __amdgpu_buffer_rsrc_t la_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        cLand, 0, ((CARRY_A || HOPS != 0) && cLand != nullptr) ? (int)(hop_right ? w_bytes : a_bytes) : 0, 0x00020000);
    // k-tile kt is about to be requested: the first of a block of rows takes the loads to that block's buffer
    auto next_hop = [&](int kt) __attribute__((always_inline)) {
        if (HOPS != 0 && kt == hop_at && kt < nk) {
            const i32x4_t r = make_rsrc(P.A_step[1 + kt / P.hop_tiles], hop_right ? w_bytes : a_bytes);
            if (hop_right)
                w_rsrc = r;
            else
                a_rsrc = r;
            hop_at += P.hop_tiles;
        }
    };
    // (A ragged k-tile is the last of a work item, LAST: its lanes beyond the k range store nothing.)
    auto carry_tile = [&](int kt, int stage_a, int stage_w, auto last_tag) __attribute__((always_inline)) {
        const int k0 = ktile(kt) * BK;
        if constexpr (HOPS != 0) {
            static_assert(HOPS == 0 || A_LD == B_LD, "the waits count the same stores for either operand");
            const unsigned own = (unsigned)(kt - P.hop_own * P.hop_tiles) < (unsigned)P.hop_tiles ? OOB : 0;   // nothing to land
#pragma unroll
            for (int j = 0; j < A_LD; ++j) {
                const int at = (hop_right ? W_BASE + stage_w * B_BYTES : stage_a * A_BYTES) + (j * NW + wave) * 1024 + lane * 16;
                const u32x4_t t = *reinterpret_cast<const u32x4_t *>(smem + at);
                const unsigned off = hop_right ? b_off[w_reg(j)] : a_off[a_reg(j)];
                const int dist = hop_right ? k0 * w_kstep + w_dist(j) : k0 * a_kstep + a_dist(j);
                __builtin_amdgcn_raw_buffer_store_b128(t, la_rsrc, (int)(off | own), dist, 0);
            }
            carry_at += carry_step;
            return;
        }
        const bool ragged = decltype(last_tag)::value && k0 + BK > K;
#pragma unroll
        for (int j = 0; j < A_LD; ++j) {
            const u32x4_t t = *reinterpret_cast<const u32x4_t *>(smem + stage_a * A_BYTES + (j * NW + wave) * 1024 + lane * 16);
            unsigned off = a_off[MF16 ? 0 : j];
            if (ragged)
                off = k0 + chunk_k(j, false, 0) < K ? off : OOB;
            __builtin_amdgcn_raw_buffer_store_b128(t, la_rsrc, (int)off, k0 * 2 + j * a_jstep, 0);
        }
        carry_at += tiles_n;
    };

    // Fragment addressing (byte offsets inside a stage), fixed for the whole loop.  The swizzle
    // uses row bits 0..3 only, so the 32-row MFMA tiles of a wave differ by constants, and the
    // 16-wide k-slice ks is reached by XOR-ing (ks << 5) into the offset of slice 0.
    const int frow = lane & 31, fkc = lane >> 5;
    const int a_addr = swz_row(wm * WTM + frow, fkc);
    int a_addr_t[A_T ? TM : 1];
    if constexpr (A_T) {
        const int blk = lane >> 4, i16 = lane & 15;
        const int kl = (blk >> 1) * 8 + (i16 >> 2);
        const int ml = wm * WTM + (blk & 1) * 16 + (i16 & 3) * 4;        // row of tile i = 0
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int q = ((ml >> 5) + i) ^ (kl & 3);
            a_addr_t[i] = kl * A_ROWB + (q << 6) + (ml & 31) * 2;
        }
    } else {
        a_addr_t[0] = 0;
    }
    int w_addr[W_KN ? TN : 1];
    if constexpr (W_KN) {
        const int blk = lane >> 4, i16 = lane & 15;
        const int kl = (blk >> 1) * 8 + (i16 >> 2);                      // k of (ks = 0, h = 0)
        const int nl = wn * WTN + (blk & 1) * 16 + (i16 & 3) * 4;        // column of tile j = 0
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int q = ((nl >> 5) + j) ^ (kl & 3);
            w_addr[j] = W_BASE + kl * W_ROWB + (q << 6) + (nl & 31) * 2;
        }
    } else {
        w_addr[0] = W_BASE + swz_row(wn * WTN + frow, fkc);
    }

    // MF16: a fragment is 16 rows x 32 k: lane L holds row (L & 15) and one 16-byte chunk (8 k) of the 32-wide slice --
    // chunk 0, 2, 1, 3 for the lane blocks L >> 4 = 0, 1, 2, 3 (which eight k values sit in which slots of the
    // contraction is free as long as both operands agree; with this order the lanes L and L + 32 read an even and an
    // odd chunk, as they do in the 32x32x16 layout).  The second slice of a k-tile is reached by XOR-ing 64 into the
    // offset, 16-row tiles lie 2 KiB apart.  (The LDS bank-conflict counter shows 64 cycles per wave and k-tile for this
    // loop with either chunk order -- 2.5 % of a k-tile's time -- and none for the 32x32x16 loop.)
    constexpr int TN16 = WTN / 16;
    int a_addr16 = 0;
    // ([k x n] weights: one address per pair of 16-column tiles; the odd tile of a pair lies at that address ^ 32)
    int w_addr16[(MF16 && W_KN) ? TN16 / 2 : 1];
    if constexpr (MF16) {
        static_assert(!MF16 || (TM == 4 && TN == 2), "quarter phases are written for the 128x64 wave tile");
        const int kch = (((lane >> 4) & 1) << 1) | (lane >> 5);          // this lane's chunk of a slice
        const int i16 = lane & 15;
        const int kl = kch * 8 + (i16 >> 2);                                 // k of (slice 0, first half), tiles stored by k-rows
        if constexpr (A_T) {
            // (16-row tile t of the wave's rows lies at this address ^ 32 t: the swizzle touches those bits alone)
            static_assert(!A_T || WTM == 128, "four 64-byte groups to a wave's rows");
            a_addr16 = kl * A_ROWB + (((wm * WTM) >> 5 | (kl & 3)) << 6) + (((i16 & 3) * 8) ^ (((kl >> 4) & 1) << 5));
        } else {
            a_addr16 = swz_row(wm * WTM + (lane & 15), kch);
        }
        if constexpr (W_KN) {
#pragma unroll
            for (int t = 0; t < TN16; t += 2) {
                const int nl = wn * WTN + t * 16 + (i16 & 3) * 4;
                const int q = (nl >> 5) ^ (kl & 3);
                w_addr16[t / 2] = W_BASE + kl * W_ROWB + (q << 6) + (((nl & 31) * 2) ^ (((kl >> 4) & 1) << 5));
            }
        } else {
            w_addr16[0] = W_BASE + swz_row(wn * WTN + (lane & 15), kch);
        }
    } else {
        w_addr16[0] = 0;
    }
    auto read_frags = [&](int stage_a, int stage_w, int ks, bf16x8_t (&af)[TM], bf16x8_t (&wf)[TN]) __attribute__((always_inline)) {
        const unsigned char *st = smem + stage_a * A_BYTES;
        const unsigned char *stw = smem + stage_w * B_BYTES;     // (w_addr holds the weight region's base)
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if constexpr (A_T) {
                const unsigned char *pa = st + a_addr_t[i] + ks * 16 * A_ROWB;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4_t *)(pa));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4_t *)(pa + 4 * A_ROWB));
                const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                af[i] = __builtin_bit_cast(bf16x8_t, both);
            } else {
                af[i] = *reinterpret_cast<const bf16x8_t *>(st + (a_addr ^ (ks << 5)) + i * 32 * 128);
            }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if constexpr (W_KN) {
                const unsigned char *pw = stw + w_addr[j] + ks * 16 * W_ROWB;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4_t *)(pw));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4_t *)(pw + 4 * W_ROWB));
                const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                wf[j] = __builtin_bit_cast(bf16x8_t, both);
            } else {
                wf[j] = *reinterpret_cast<const bf16x8_t *>(stw + (w_addr[0] ^ (ks << 5)) + j * 32 * 128);
            }
        }
    };
    auto mfma_block = [&](const bf16x8_t (&af)[TM], const bf16x8_t (&wf)[TN]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[j], af[i], acc[i][j], 0, 0, 0);
    };

    // One slice phase: the LDS reads of the NEXT slice's fragments (into afn, wfn), then the MFMAs of
    // the fragments in (afc, wfc) in NSEG segments.  The reads are interleaved with the MFMAs of the
    // first segment; after each segment one direct load of a later k-tile may be issued (load slots
    // LO .. LO+NSEG-1 of tile kt_l into stage_l), so that the wave never queues a burst of loads
    // behind which its MFMAs would wait.
    constexpr int NREAD = (A_T ? 2 * TM : TM) + (W_KN ? 2 * TN : TN);
    constexpr int NMFMA = TM * TN;
    constexpr int NSEG = NMFMA < 4 ? NMFMA : 4;
    constexpr int MPS = NMFMA / NSEG;                       // MFMAs per segment
    constexpr int LH = LPT < NSEG ? LPT : NSEG;             // loads issued in the first load phase
    static_assert(NMFMA % NSEG == 0 && (!SPREAD || LPT - LH <= NSEG), "segmenting");
    auto mfma_seg = [&](const bf16x8_t (&af)[TM], const bf16x8_t (&wf)[TN], auto seg_tag) __attribute__((always_inline)) {
        constexpr int seg = decltype(seg_tag)::value;
#pragma unroll
        for (int q = seg * MPS; q < (seg + 1) * MPS; ++q)
            acc[q / TN][q % TN] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q % TN], af[q / TN], acc[q / TN][q % TN], 0, 0, 0);
    };
    auto phase = [&](const bf16x8_t (&afc)[TM], const bf16x8_t (&wfc)[TN], bool do_read, int sa_n, int sw_n, int ks_n,
                     bf16x8_t (&afn)[TM], bf16x8_t (&wfn)[TN], int kt_l, int sa_l, int sw_l, auto lo_tag, auto n_tag,
                     auto whole_k_tag) __attribute__((always_inline)) {
        constexpr int LO = decltype(lo_tag)::value, NL = decltype(n_tag)::value;   // load slots of this phase
        if (do_read)
            read_frags(sa_n, sw_n, ks_n, afn, wfn);
        mfma_seg(afc, wfc, std::integral_constant<int, 0>{});
        interleave_mfma_reads<NREAD, (NREAD + MPS - 1) / MPS>();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NL > 0) issue_load(kt_l, sa_l, sw_l, std::integral_constant<int, LO>{}, whole_k_tag);
        if constexpr (NSEG > 1) {
            mfma_seg(afc, wfc, std::integral_constant<int, 1>{});
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NL > 1) issue_load(kt_l, sa_l, sw_l, std::integral_constant<int, LO + 1>{}, whole_k_tag);
        }
        if constexpr (NSEG > 2) {
            mfma_seg(afc, wfc, std::integral_constant<int, 2>{});
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NL > 2) issue_load(kt_l, sa_l, sw_l, std::integral_constant<int, LO + 2>{}, whole_k_tag);
        }
        if constexpr (NSEG > 3) {
            mfma_seg(afc, wfc, std::integral_constant<int, 3>{});
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NL > 3) issue_load(kt_l, sa_l, sw_l, std::integral_constant<int, LO + 3>{}, whole_k_tag);
        }
    };
    using c0 = std::integral_constant<int, 0>;
    using cLH = std::integral_constant<int, LH>;
    using cLR = std::integral_constant<int, LPT - LH>;
    using cLPT = std::integral_constant<int, LPT>;

    bf16x8_t af0[TM], wf0[TN], af1[TM], wf1[TN];

    const unsigned r_bytes = (unsigned)(((int64_t)(M - 1) * P.ldo + N) * 4);
    __amdgpu_buffer_rsrc_t r_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(cRecv), 0, cRecv != nullptr ? (int)r_bytes : 0, 0x00020000);
    constexpr int COHERENT_LD = 1 | 16;               // buffer cache-policy bits sc0 | sc1
    constexpr int LINE_AUX = NT ? 2 : 0;              // ... and nt
    // B_in and the fp32 output are read and written as whole 128-byte lines: eight lanes to a row of a 32-column block,
    // eight rows per instruction, four instructions to a 32x32 sub-tile.  The offsets are taken anew from an opaque
    // copy of the lane index where they are needed: the main loop has no registers for them.
    const unsigned rows8 = (unsigned)P.ldo * 32u;     // bytes from one instruction's eight rows to the next's
    auto line_offsets = [&](int i, int j, int (&off)[4]) __attribute__((always_inline)) {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int r = m0 + wm * WTM + i * 32 + (ln >> 3), cl = n0 + wn * WTN + j * 32 + (ln & 7) * 4;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
            off[s4] = (MF16 || (r + 8 * s4 < M && cl < N)) ? (int)(((unsigned)r * (unsigned)P.ldo + cl) * 4u + s4 * rows8) : (int)OOB;
    };
    // Row blocks of B_in held in registers, the one being added and the next; of them EARLY are requested where the k loop has
    // issued its last operand load (a launch that waits for a flag requests nothing ahead).  The 256x256 tile has
    // registers for one only.
    constexpr int LV = RECV ? 2 : 1;
    constexpr int EARLY = !(PERSIST && RECV) ? 0 : (BM == 256 && BN == 256) ? 1 : 2;
    static_assert(LV <= TM, "row blocks in flight");
    constexpr int EARLY_LOADS = EARLY * TN * 4;
    u32x4_t lv[LV][RECV ? TN : 1][4];
    auto load_lines = [&](int i, auto aux_tag) __attribute__((always_inline)) {
        constexpr int AUX = decltype(aux_tag)::value;
#pragma unroll
        for (int j = 0; j < (RECV ? TN : 0); ++j) {
            int lo[4];
            line_offsets(i, j, lo);
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4)
                lv[i % LV][j][s4] = __builtin_amdgcn_raw_buffer_load_b128(r_rsrc, lo[s4], 0, AUX);
        }
    };
    // (a launch that waited for its delivery's flag reads it with the device-coherent cache policy, see wait_delivery)
    const bool recv_coherent = cFlag != nullptr && !P.wait_at_start;
    auto load_recv = [&](int i) __attribute__((always_inline)) {
        if (recv_coherent)
            load_lines(i, std::integral_constant<int, COHERENT_LD>{});
        else
            load_lines(i, std::integral_constant<int, LINE_AUX>{});
    };

    // The delivery landed in front of the main loop (GemmParams::land_first): every other workgroup of an XCD copies its
    // tile's part of B_in from the sender's to the landing buffer before it multiplies (its first operand tiles arrive
    // meanwhile), the others behind it, in the epilogue.  The work items of a round start together and are equally long:
    // otherwise all compute units multiply while the memory idles and then all move their tiles.  B_in itself is added in
    // the epilogue in either case: a sum that starts at B_in saves the second read of it (8 x 1024 x 8192 x 1024: 202
    // instead of 209 us) but rounds every k step at B_in's magnitude, which doubles the error against 64 bits.
    const bool lands_first = PERSIST && RECV && P.land_first && cLand != nullptr && cRecv != nullptr && (((int)blockIdx.x >> 3) & 1) != 0;
    auto land_in_front = [&]() __attribute__((always_inline)) {
        if constexpr (PERSIST && RECV) {
            if (lands_first) {
                __amdgpu_buffer_rsrc_t l_rsrc = __builtin_amdgcn_make_buffer_rsrc(cLand, 0, (int)r_bytes, 0x00020000);
                u32x4_t v[TM][TN][4];                // (the accumulators are not in use yet)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        int lo[4];
                        line_offsets(i, j, lo);
#pragma unroll
                        for (int s4 = 0; s4 < 4; ++s4)   // (through the caches: the epilogue reads it again)
                            v[i][j][s4] = __builtin_amdgcn_raw_buffer_load_b128(r_rsrc, lo[s4], 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        int lo[4];
                        line_offsets(i, j, lo);
#pragma unroll
                        for (int s4 = 0; s4 < 4; ++s4)
                            __builtin_amdgcn_raw_buffer_store_b128(v[i][j][s4], l_rsrc, lo[s4], 0, LINE_AUX);
                        __builtin_amdgcn_sched_barrier(0);
                    }
            }
        }
    };
    auto request_early = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < EARLY; ++i)
            load_lines(i, std::integral_constant<int, LINE_AUX>{});
    };
    // the left-operand stage whose memory serves as the wave-private scratch of the epilogue's stores
    constexpr int land_stage = SPREAD ? NSA - 1 : 0;
    if constexpr (SPREAD && MF16) {
        // The schedule of the 256x256 tile (see the variant below for its reasoning) on 16x16x32 MFMAs.  A k-tile is two
        // 32-wide slices; a slice is consumed in four quarter phases, phase p = the wave tile's 32-row block p:
        // 2 left-operand fragments (16-row tiles x = 0, 1) x 4 weight fragments = 8 MFMAs, in four segments of two
        // (segments 0, 1: x = 0; segments 2, 3: x = 1).  A phase is short (128 cycles of MFMA issue), so LDS reads and
        // direct loads are dealt out thinly -- at most one fragment read and one direct load per segment -- and every
        // fragment register is refilled as soon as its last MFMA has issued, a phase and a half before its next use:
        // the left-operand fragments live in two buffers that alternate by phase (afA: even phases), and phase q reads
        //     at segment 0: fragment x = 1 of phase q+1, into the other buffer (its last use was in phase q-1);
        //     at segment 2: fragment x = 0 of phase q+2, into its own buffer;
        // the weight fragments live in two buffers that alternate by slice; those of slice 1 are read one per phase in
        // phases 0 .. 3, those of slice 0 of the next tile two per phase in phases 6 and 7 (segments 1 and 3).
        //   steady state, tile kt (phases 0 .. 7 = slice 0 blocks 0 .. 3, slice 1 blocks 0 .. 3):
        //     phases 0 .. 3: + one left-operand load of tile kt+NS each, into the stage tile kt-1 vacated
        //     phase 6, after segment 0 (the last read of tile kt has been issued):
        //              wait: tile kt+1 complete; barrier: tile kt has been read by all;
        //              then the first reads of tile kt+1, and in phases 6 and 7 + two weight loads of tile kt+NS each
        static_assert(A_LD == 4 && B_LD == 4, "load slots below: four loads per operand, tile and wave");
        using p0_t = std::integral_constant<int, 0>;
        using p1_t = std::integral_constant<int, 1>;
        using p2_t = std::integral_constant<int, 2>;
        using p3_t = std::integral_constant<int, 3>;
        using c1 = std::integral_constant<int, 1>;
        using c2 = std::integral_constant<int, 2>;
        using on_t = std::true_type;
        using off_t = std::false_type;
        bf16x8_t afA[2], afB[2], wfA[4], wfB[4];
        // the two MFMAs of segment seg of a phase on block PB: 16-row tile x = seg / 2, 16-column tiles 2 (seg & 1) + {0, 1}
        auto mfma16_seg = [&](auto pb_tag, const bf16x8_t (&af)[2], const bf16x8_t (&wf)[4], auto seg_tag) __attribute__((always_inline)) {
            constexpr int PB = decltype(pb_tag)::value, seg = decltype(seg_tag)::value;
            constexpr int x = seg >> 1, j = seg & 1;
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const int g = 2 * x + y;
                acc4[MF16 ? PB : 0][MF16 ? j : 0][g] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[2 * j + y], af[x], acc4[MF16 ? PB : 0][MF16 ? j : 0][g], 0, 0, 0);
            }
        };
        auto frag_a16 = [&](int stage_a, int sl, int t16) __attribute__((always_inline)) {
            if constexpr (A_T) {
                const unsigned char *pa = smem + stage_a * A_BYTES + (a_addr16 ^ (t16 << 5)) + sl * 32 * A_ROWB;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pa));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pa + 4 * A_ROWB));
                const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                return __builtin_bit_cast(bf16x8_t, both);
            } else {
                return *reinterpret_cast<const bf16x8_t *>(smem + stage_a * A_BYTES + (a_addr16 ^ (sl << 6)) + t16 * 2048);
            }
        };
        auto frag_w16 = [&](int stage_w, int sl, auto t_tag) __attribute__((always_inline)) {
            constexpr int t = decltype(t_tag)::value;
            const unsigned char *stw = smem + stage_w * B_BYTES;
            if constexpr (W_KN) {
                const unsigned char *pw = stw + (w_addr16[(MF16 && W_KN) ? t / 2 : 0] ^ ((t & 1) << 5)) + sl * 32 * W_ROWB;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pw));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pw + 4 * W_ROWB));
                const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                return __builtin_bit_cast(bf16x8_t, both);
            } else {
                return *reinterpret_cast<const bf16x8_t *>(stw + (w_addr16[0] ^ (sl << 6)) + t * 2048);
            }
        };
        constexpr int NRD_AF = A_T ? 2 : 1, NRD_WF = W_KN ? 2 : 1;   // LDS reads of one fragment
        auto nothing = [&]() __attribute__((always_inline)) {};
        // One quarter phase on block PB with the fragments (afc, wfc).
        //   r1: fragment x = 1 of (stage s1, slice l1, block b1) into afo[1] at segment 0;  mid(): between segments 0 and 1;
        //   nwf weight fragments w0, w0 + 1 of (stage sw, slice lw) into wfn at segments 1 and 3;
        //   r2: fragment x = 0 of (s2, l2, b2) into afc[0] at segment 2;
        //   ld1(), ld3(): direct loads issued at segments 1 and 3.
        auto phase16 = [&](auto pb_tag, bf16x8_t (&afc)[2], const bf16x8_t (&wfc)[4], bf16x8_t (&afo)[2], bf16x8_t (&wfn)[4],
                           auto r1_tag, int s1, int l1, int b1, auto mid, auto nwf_tag, int sw, int lw, auto w0_tag,
                           auto r2_tag, int s2, int l2, int b2, auto ld1, auto ld3) __attribute__((always_inline)) {
            constexpr bool R1 = decltype(r1_tag)::value, R2 = decltype(r2_tag)::value;
            constexpr int NWF = decltype(nwf_tag)::value, W0 = decltype(w0_tag)::value;
            if constexpr (R1)
                afo[1] = frag_a16(s1, l1, 2 * b1 + 1);
            mfma16_seg(pb_tag, afc, wfc, std::integral_constant<int, 0>{});
            interleave_mfma_reads<R1 ? NRD_AF : 0, 1>();
            __builtin_amdgcn_sched_barrier(0);
            mid();
            if constexpr (NWF > 0)
                wfn[W0] = frag_w16(sw, lw, std::integral_constant<int, W0>{});
            ld1();
            mfma16_seg(pb_tag, afc, wfc, std::integral_constant<int, 1>{});
            interleave_mfma_reads<((NWF > 0) ? NRD_WF : 0), 1>();
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (R2)
                afc[0] = frag_a16(s2, l2, 2 * b2);
            mfma16_seg(pb_tag, afc, wfc, std::integral_constant<int, 2>{});
            interleave_mfma_reads<R2 ? NRD_AF : 0, 1>();
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (NWF > 1)
                wfn[W0 + 1] = frag_w16(sw, lw, std::integral_constant<int, W0 + 1>{});
            ld3();
            mfma16_seg(pb_tag, afc, wfc, std::integral_constant<int, 3>{});
            interleave_mfma_reads<((NWF > 1) ? NRD_WF : 0), 1>();
            __builtin_amdgcn_sched_barrier(0);
        };
        // Phases 0 .. 5 of a tile in stages (ca, cw); ldq(q): the direct load phase q (0 .. 3) issues (at its segment 1).
        auto front16 = [&](int ca, int cw, auto ld0, auto ld1_, auto ld2, auto ld3_, auto ph2) __attribute__((always_inline)) {
            phase16(p0_t{}, afA, wfA, afB, wfB, on_t{}, ca, 0, 1, nothing, c1{}, cw, 1, c0{}, on_t{}, ca, 0, 2, ld0, nothing);
            phase16(p1_t{}, afB, wfA, afA, wfB, on_t{}, ca, 0, 2, nothing, c1{}, cw, 1, c1{}, on_t{}, ca, 0, 3, ld1_, nothing);
            ph2(ld2);
            phase16(p3_t{}, afB, wfA, afA, wfB, on_t{}, ca, 1, 0, nothing, c1{}, cw, 1, std::integral_constant<int, 3>{}, on_t{}, ca, 1, 1, ld3_, nothing);
            phase16(p0_t{}, afA, wfB, afB, wfA, on_t{}, ca, 1, 1, nothing, c0{}, 0, 0, c0{}, on_t{}, ca, 1, 2, nothing, nothing);
            phase16(p1_t{}, afB, wfB, afA, wfA, on_t{}, ca, 1, 2, nothing, c0{}, 0, 0, c0{}, on_t{}, ca, 1, 3, nothing, nothing);
        };
        // phase 2 of a tile in stages (ca, cw) as a plain phase
        auto plain_ph2 = [&](int ca, int cw) __attribute__((always_inline)) {
            return [&, ca, cw](auto ld2) __attribute__((always_inline)) {
                phase16(p2_t{}, afA, wfA, afB, wfB, on_t{}, ca, 0, 3, nothing, c1{}, cw, 1, c2{}, on_t{}, ca, 1, 0, ld2, nothing);
            };
        };

    #pragma unroll
        for (int t = 0; t < NS; ++t)
            issue_range(t, t, t, c0{}, cLPT{});
        land_in_front();
        wait_vmcnt<(NS - 1) * LPT>();
        __syncthreads();
        afA[0] = frag_a16(0, 0, 0);
        afA[1] = frag_a16(0, 0, 1);
        afB[0] = frag_a16(0, 0, 2);
        wfA[0] = frag_w16(0, 0, std::integral_constant<int, 0>{});
        wfA[1] = frag_w16(0, 0, std::integral_constant<int, 1>{});
        wfA[2] = frag_w16(0, 0, std::integral_constant<int, 2>{});
        wfA[3] = frag_w16(0, 0, std::integral_constant<int, 3>{});
        __builtin_amdgcn_sched_barrier(0);

        int cur_a = 0, cur_w = 0;                        // stages of tile kt
        int prev_a = NSA - 1;                            // left-operand stage of tile kt-1 (= of tile kt+NS)
        auto body = [&](int kt, int ca, int cw, int pa, int na, int nw_, auto wk) __attribute__((always_inline)) {
            auto la = [&](auto idx_tag) __attribute__((always_inline)) {       // a left-operand load of tile kt+NS
                return [&, kt, pa](/*no args*/) __attribute__((always_inline)) { issue_load(kt + NS, pa, 0, decltype(idx_tag){}, wk); };
            };
            auto lw = [&](auto idx_tag) __attribute__((always_inline)) {       // a weight load of tile kt+NS
                return [&, kt, cw]() __attribute__((always_inline)) { issue_load(kt + NS, 0, cw, decltype(idx_tag){}, wk); };
            };
            next_hop(kt + NS);
            front16(ca, cw, la(std::integral_constant<int, 0>{}), la(std::integral_constant<int, 1>{}),
                    la(std::integral_constant<int, 2>{}), la(std::integral_constant<int, 3>{}), plain_ph2(ca, cw));
            auto publish = [&]() __attribute__((always_inline)) {
                if ((CARRY_A || HOPS != 0) && kt == carry_at) {   // tile kt goes on to the landing buffer: its stores are the
                    carry_tile(kt, ca, cw, std::false_type{});          // youngest requests and need not be awaited here
                    wait_vmcnt<(NS - 2) * LPT + 2 * A_LD>();
                } else {
                    wait_vmcnt<(NS - 2) * LPT + A_LD>();
                }
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            };
            phase16(p2_t{}, afA, wfB, afB, wfA, on_t{}, ca, 1, 3, publish, c2{}, nw_, 0, c0{}, on_t{}, na, 0, 0,
                    lw(std::integral_constant<int, 4>{}), lw(std::integral_constant<int, 5>{}));
            phase16(p3_t{}, afB, wfB, afA, wfA, on_t{}, na, 0, 0, nothing, c2{}, nw_, 0, c2{}, on_t{}, na, 0, 1,
                    lw(std::integral_constant<int, 6>{}), lw(std::integral_constant<int, 7>{}));
        };
        // The iterations that request a whole k-tile do not test their loads; the others (a ragged k-tile, which is the last of
        // the range, or one beyond it, which reads zeros and moves nothing) do.
        const int tested_at = nk - NS - (K % BK != 0 ? 1 : 0);
        int kt = 0;
        for (; kt < tested_at; ++kt) {
            const int nxt_a = (cur_a + 1 == NSA) ? 0 : cur_a + 1;
            const int nxt_w = (cur_w + 1 == NS) ? 0 : cur_w + 1;
            body(kt, cur_a, cur_w, prev_a, nxt_a, nxt_w, std::true_type{});
            prev_a = cur_a;
            cur_a = nxt_a;
            cur_w = nxt_w;
        }
        // the last tile of a work item: nothing follows it
        auto last16 = [&](int ca, int cw) __attribute__((always_inline)) {
            request_early();
            front16(ca, cw, nothing, nothing, nothing, nothing, plain_ph2(ca, cw));
            phase16(p2_t{}, afA, wfB, afB, wfA, on_t{}, ca, 1, 3, nothing, c0{}, 0, 0, c0{}, off_t{}, 0, 0, 0, nothing, nothing);
            if ((CARRY_A || HOPS != 0) && nk - 1 == carry_at)
                carry_tile(nk - 1, ca, cw, std::true_type{});
            phase16(p3_t{}, afB, wfB, afA, wfA, off_t{}, 0, 0, 0, nothing, c0{}, 0, 0, c0{}, off_t{}, 0, 0, 0, nothing, nothing);
        };
        asm volatile("" : "+s"(kt));                     // (keeps the compiler from peeling the loop below: it spills)
        for (; kt + 1 < nk; ++kt) {
            const int nxt_a = (cur_a + 1 == NSA) ? 0 : cur_a + 1;
            const int nxt_w = (cur_w + 1 == NS) ? 0 : cur_w + 1;
            body(kt, cur_a, cur_w, prev_a, nxt_a, nxt_w, std::false_type{});
            prev_a = cur_a;
            cur_a = nxt_a;
            cur_w = nxt_w;
        }
        if (nk > 0)
            last16(cur_a, cur_w);
    } else if constexpr (SPREAD) {
        // The left-operand tile has NS+1 stages, the weight tile NS (tile t lives in stages t mod (NS+1) and
        // t mod NS).  Loads return in issue order, so what is issued first must be what is needed first:
        //   prologue: tiles 0 .. NS-1 whole, in tile order; tile 0 is awaited, its first fragments fetched
        //   steady state, tile kt:
        //     slice 0: + the left-operand loads of tile kt+NS, into the stage tile kt-1 vacated
        //     slice 1, slice 2
        //     wait: tile kt+1 complete -- the loads of NS-2 later whole tiles and the left-operand loads
        //           just issued may be in flight; barrier: tile kt has been read by all
        //     slice 3: + the weight loads of tile kt+NS, into the stage tile kt vacated
        // A weight load thus has 1 to 1.25 k-tiles of MFMA time to arrive and a left-operand load 1.75 to 2
        // (with NS = 2; both NS-2 more otherwise).
        static_assert(A_LD == LH && LPT - LH == B_LD, "one load slot per MFMA segment and operand");
        using cALD = std::integral_constant<int, A_LD>;
    #pragma unroll
        for (int t = 0; t < NS; ++t)
            issue_range(t, t, t, c0{}, cLPT{});
        land_in_front();
        wait_vmcnt<(NS - 1) * LPT>();
        __syncthreads();
        read_frags(0, 0, 0, af0, wf0);
        __builtin_amdgcn_sched_barrier(0);

        // The steady state is branch-free: only the iteration that requests a ragged k-tile (the last of the range: the launcher
        // then leaves the k order unrotated) tests its loads, and the last NS iterations have none to issue.
        int cur_a = 0, cur_w = 0;                        // stages of tile kt
        int prev_a = NSA - 1;                            // left-operand stage of tile kt-1 (= of tile kt+NS)
        // LOADS 2: loads of tile kt+NS, known to be whole; 1: tested; 0: none, R tiles behind tile kt+1 may be in flight
        auto body = [&](int kt, int ca, int cw, int pa, int na, int nw_, auto loads_tag, auto r_tag) __attribute__((always_inline)) {
            constexpr int LOADS = decltype(loads_tag)::value, R = decltype(r_tag)::value;
            using wk = std::integral_constant<bool, LOADS == 2>;
            using nA = std::integral_constant<int, LOADS ? A_LD : 0>;
            using nW = std::integral_constant<int, LOADS ? LPT - LH : 0>;
            constexpr int BEHIND = LOADS ? (NS - 2) * LPT + A_LD : R * LPT + EARLY_LOADS;
            phase(af0, wf0, true, ca, cw, 1, af1, wf1, kt + NS, pa, 0, c0{}, nA{}, wk{});
            phase(af1, wf1, true, ca, cw, 2, af0, wf0, 0, 0, 0, c0{}, c0{}, wk{});
            phase(af0, wf0, true, ca, cw, 3, af1, wf1, 0, 0, 0, c0{}, c0{}, wk{});
            if (CARRY_A && kt == carry_at) {         // tile kt goes on to the landing buffer: its stores are the
                carry_tile(kt, ca, 0, std::false_type{});               // youngest requests and need not be awaited here
                wait_vmcnt<BEHIND + A_LD>();
            } else {
                wait_vmcnt<BEHIND>();
            }
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            phase(af1, wf1, true, na, nw_, 0, af0, wf0, kt + NS, 0, cw, cALD{}, nW{}, wk{});
        };
        int kt = 0;
        auto step = [&](auto loads_tag, auto r_tag) __attribute__((always_inline)) {
            const int nxt_a = (cur_a + 1 == NSA) ? 0 : cur_a + 1;
            const int nxt_w = (cur_w + 1 == NS) ? 0 : cur_w + 1;
            body(kt, cur_a, cur_w, prev_a, nxt_a, nxt_w, loads_tag, r_tag);
            prev_a = cur_a;
            cur_a = nxt_a;
            cur_w = nxt_w;
            ++kt;
        };
        using l0 = std::integral_constant<int, 0>;
        using l1 = std::integral_constant<int, 1>;
        using l2 = std::integral_constant<int, 2>;
        const int whole_end = nk - NS - (K % BK != 0 ? 1 : 0);
        while (kt < whole_end)
            step(l2{}, l0{});
        while (kt < nk - NS)
            step(l1{}, l0{});
        request_early();
        if constexpr (NS > 3) {
            if (nk > 3)
                step(l0{}, l2{});
        }
        if constexpr (NS > 2) {
            if (nk > 2)
                step(l0{}, l1{});
        }
        if (nk > 1)
            step(l0{}, l0{});
        if (nk > 0) {                                    // last tile: nothing follows it
            using wk = std::true_type;
            phase(af0, wf0, true, cur_a, cur_w, 1, af1, wf1, 0, 0, 0, c0{}, c0{}, wk{});
            phase(af1, wf1, true, cur_a, cur_w, 2, af0, wf0, 0, 0, 0, c0{}, c0{}, wk{});
            phase(af0, wf0, true, cur_a, cur_w, 3, af1, wf1, 0, 0, 0, c0{}, c0{}, wk{});
            if (CARRY_A && nk - 1 == carry_at)
                carry_tile(nk - 1, cur_a, 0, std::true_type{});
            phase(af1, wf1, false, 0, 0, 0, af0, wf0, 0, 0, 0, c0{}, c0{}, wk{});
        }
    } else {
        // Variant for two workgroups per CU over long k ranges: a tile's loads go out together right
        // after the barrier that frees their stage, and the LDS reads of the next slice are
        // interleaved with all MFMAs of the current one.
        auto phase_b = [&](const bf16x8_t (&afc)[TM], const bf16x8_t (&wfc)[TN], bool do_read, int stage_n, int ks_n,
                           bf16x8_t (&afn)[TM], bf16x8_t (&wfn)[TN], auto rpm_tag) __attribute__((always_inline)) {
            constexpr int RPM = decltype(rpm_tag)::value;
            if (do_read)
                read_frags(stage_n, stage_n, ks_n, afn, wfn);
#pragma unroll
            for (int q = 0; q < NMFMA; ++q)
                acc[q / TN][q % TN] =
                    __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfc[q % TN], afc[q / TN], acc[q / TN][q % TN], 0, 0, 0);
            interleave_mfma_reads<NREAD, RPM>();
            __builtin_amdgcn_sched_barrier(0);
        };
        constexpr int RPM_N = (NREAD + NMFMA - 1) / NMFMA;      // reads spread over the whole slice
        using rpm1 = std::integral_constant<int, RPM_N>;
        using rpm2 = std::integral_constant<int, 2 * RPM_N>;    // reads packed into its first half
#pragma unroll
        for (int t = 0; t < NS; ++t)
            issue_range(t, t, t, c0{}, cLPT{});
        land_in_front();
        wait_vmcnt<(NS - 1) * LPT>();
        __syncthreads();
        read_frags(0, 0, 0, af0, wf0);
        __builtin_amdgcn_sched_barrier(0);
        int cur = 0;
        for (int kt = 0; kt + 1 < nk; ++kt) {
            const int nxt = (cur + 1 == NS) ? 0 : cur + 1;
            phase_b(af0, wf0, true, cur, 1, af1, wf1, rpm1{});
            phase_b(af1, wf1, true, cur, 2, af0, wf0, rpm1{});
            phase_b(af0, wf0, true, cur, 3, af1, wf1, rpm2{});   // reads early: complete at the barrier
            // tile kt+1 complete, NS-2 later tiles may be in flight
            if (CARRY_A && kt == carry_at) {         // tile kt goes on to the landing buffer (stores not awaited here)
                carry_tile(kt, cur, 0, std::false_type{});
                wait_vmcnt<(NS - 2) * LPT + A_LD>();
            } else {
                wait_vmcnt<(NS - 2) * LPT>();
            }
            __syncthreads();                 // tile kt is read by all, tile kt+1 is published
            issue_range(kt + NS, cur, cur, c0{}, cLPT{});
            __builtin_amdgcn_sched_barrier(0);
            phase_b(af1, wf1, true, nxt, 0, af0, wf0, rpm1{});
            cur = nxt;
        }
        if (nk > 0) {
            request_early();
            phase_b(af0, wf0, true, cur, 1, af1, wf1, rpm1{});
            phase_b(af1, wf1, true, cur, 2, af0, wf0, rpm1{});
            phase_b(af0, wf0, true, cur, 3, af1, wf1, rpm1{});
            if (CARRY_A && nk - 1 == carry_at)
                carry_tile(nk - 1, cur, 0, std::true_type{});
            phase_b(af1, wf1, false, 0, 0, af0, wf0, rpm1{});
        }
    }
    // no direct load may outlive its LDS allocation (the early requests of B_in are younger than all of them)
    wait_vmcnt<EARLY_LOADS>();

    // Split-K: every split parks its fp32 partial tile in the workspace; the split that finishes
    // last sums all partials in split order (so the result does not depend on which one that is),
    // then runs the epilogue.  No split ever waits for another.
    // The chip's eight XCDs have separate L2 caches.  Instead of writing back and invalidating whole
    // L2s around the hand-over, the partial tiles and the arrival counter are accessed with the
    // device-coherent cache policy (sc0 sc1: stores write through to memory, loads and the atomic
    // are served there), which keeps every other line of every L2 in place.
    // Bound by the trips to memory: so a partial is parked in the order the threads hold it, 1 KiB of whole lines per store (as
    // a row-major plane it left in 16-byte pieces, each a write to memory of its own), and the last split has the partials of
    // two splits in flight at once.  us, before / now: weight gradients 552 x 536 over 5768 rows
    // in three splits 34.8 / 23.3, 1200 x 520 over 2584 24.5 / 18.3, 520 x 856 over 2544 24.8 / 17.8.
    if (splits > 1) {
        constexpr int COHERENT = 1 | 16;         // buffer cache-policy bits sc0 | sc1
        constexpr int TILE_FLOATS = BM * BN;
        // (row blocks and splits at a time: the four-stage 128x128 tile, the one that a rule splits, has registers for all of two)
        constexpr int IB = NS > 2 ? TM : 1, SP_AHEAD = NS > 2 ? 2 : 1;
        auto part_rsrc = [&](int sp) __attribute__((always_inline)) {
            return __builtin_amdgcn_make_buffer_rsrc(P.ws + ((size_t)tile * splits + sp) * TILE_FLOATS, 0, TILE_FLOATS * 4, 0x00020000);
        };
        auto part_offset = [&](int i, int j, int g) __attribute__((always_inline)) { return (((i * TN + j) * 4 + g) * 64 * NW + tid) * 16; };
        __amdgpu_buffer_rsrc_t ws_rsrc = part_rsrc(split);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc_get(i, j, g)), ws_rsrc, part_offset(i, j, g), 0, COHERENT);
        __builtin_amdgcn_s_waitcnt(0);           // this wave's partial stores are acknowledged
        __syncthreads();                         // ... and every wave's
        unsigned *arrived = reinterpret_cast<unsigned *>(smem);   // the stages are no longer read by anyone
        if (tid == 0)
            *arrived = __hip_atomic_fetch_add(&P.counters[tile], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*arrived != (unsigned)(splits - 1))
            return;                              // not the last to finish: done
        if (tid == 0)                            // leave the counter ready for the next launch
            __hip_atomic_store(&P.counters[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i0 = 0; i0 < TM; i0 += IB) {
#pragma unroll
            for (int i = i0; i < i0 + IB; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        acc_set(i, j, g, f32x4_t{0.f, 0.f, 0.f, 0.f});
#pragma unroll SP_AHEAD
            for (int sp = 0; sp < splits; ++sp) {
                __amdgpu_buffer_rsrc_t rs = part_rsrc(sp);
#pragma unroll
                for (int i = i0; i < i0 + IB; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int g = 0; g < 4; ++g)
                            acc_set(i, j, g, acc_get(i, j, g) + __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, part_offset(i, j, g), 0, COHERENT)));
            }
        }
    }

    // Epilogue.  Accumulator register 4g+e of lane L holds row (L & 31), column 8g + 4(L >> 5) + e
    // of its 32x32 tile.  Bounds-checked buffer accesses: a lane outside the matrix reads zero
    // and its store is dropped.
    __syncthreads();                                 // the stores' scratch lies in a stage: all waves are done with them
    constexpr unsigned o_elem = OUT_BF16 ? 2 : 4;
    const unsigned o_bytes = (unsigned)(((int64_t)(M - 1) * P.ldo + N) * o_elem);
    __amdgpu_buffer_rsrc_t o_rsrc = __builtin_amdgcn_make_buffer_rsrc(cOut, 0, (int)o_bytes, 0x00020000);
    // The stores go through a wave-private LDS scratch so that they leave as whole 128-byte lines: the
    // accumulator layout would store 32-byte (bf16: 16-byte) pieces of thirty-two rows per instruction, which
    // the memory system handles markedly worse (measured: 70B down-projection rank step 438 -> 418 us).
    unsigned char *const scr = smem + land_stage * A_BYTES + wave * E_SCR_BYTES;
    if constexpr (!OUT_BF16) {
        // B_in comes in in the layout the tile leaves in: it is read once, stored on to the landing buffer from the
        // registers it came in (the delivery carried by the consumer) and added where the tile is read back from the
        // scratch.
        // Bound by memory: a reduce-scatter work item moves 768 KiB here at the rate a copy reaches.  Bringing B_in in under the
        // main loop instead (through LDS, 32x32x16 MFMAs) or landing it by a second read beside the GEMM measured, us per
        // carried rank step, against this: 8 x 1024 x 8192 x 3584 474 -> 436, x 1024 242 -> 223, 8 x 512 x 4096 x 1376 72.1 -> 71.5.
        if (RECV && !P.wait_at_start)
            wait_delivery(false);                    // B_in has travelled under the main loop
        __amdgpu_buffer_rsrc_t l_rsrc = __builtin_amdgcn_make_buffer_rsrc(
            PERSIST ? cLand : nullptr, 0, cRecv != nullptr && cLand != nullptr && !lands_first ? (int)r_bytes : 0, 0x00020000);
        // (256x256 tile: no branch, the allocator spills for it -- without a B_in, or nothing to land, the buffers' ranges are
        // empty: loads return zero, stores are dropped)
        const bool has_recv = RECV && (SPREAD || cRecv != nullptr);
        const bool lands = PERSIST && RECV && (SPREAD || (cRecv != nullptr && cLand != nullptr && !lands_first));
        if (has_recv && EARLY == 0)
            load_recv(0);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (has_recv && i + 1 < TM && i + 1 >= EARLY)
                load_recv(i + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                int lo[4];
                line_offsets(i, j, lo);
                u32x4_t b_in[4], sum[4];
                if constexpr (RECV) {
#pragma unroll
                    for (int s4 = 0; s4 < 4; ++s4)
                        sum[s4] = b_in[s4] = lv[i % LV][j][s4];
                    for (int b = 0; b < n_more; ++b) {   // further received partials, summed in index order
                        __amdgpu_buffer_rsrc_t m_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<float *>(P.recv_more[b]), 0, (int)r_bytes, 0x00020000);
#pragma unroll
                        for (int s4 = 0; s4 < 4; ++s4)
                            sum[s4] = __builtin_bit_cast(u32x4_t, __builtin_bit_cast(f32x4_t, sum[s4]) +
                                      __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(m_rsrc, lo[s4], 0, 0)));
                    }
                }
                if (lands)
#pragma unroll
                    for (int s4 = 0; s4 < 4; ++s4)
                        __builtin_amdgcn_raw_buffer_store_b128(b_in[s4], l_rsrc, lo[s4], 0, LINE_AUX);
                // chunk c (four columns) of row r of the sub-tile goes to plane c / 2, slot (r ^ c) + 32 (c & 1): the chunks of
                // a row lie 512 bytes apart and would all fall into one bank otherwise
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int r = MF16 ? 16 * (g >> 1) + (lane & 15) : lane & 31;
                    const int c = MF16 ? 4 * (g & 1) + (lane >> 4) : 2 * g + (lane >> 5);
                    *reinterpret_cast<f32x4_t *>(scr + (c >> 1) * 1024 + ((32 * (c & 1) + (r ^ c)) << 4)) = acc_get(i, j, g);
                }
                const int c = lane & 7, r8 = lane >> 3;
                const unsigned char *base = scr + (c >> 1) * 1024 + (32 * (c & 1)) * 16;
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4) {
                    const f32x4_t t = *reinterpret_cast<const f32x4_t *>(base + (((8 * s4 + r8) ^ c) << 4));
                    const f32x4_t o = has_recv ? __builtin_bit_cast(f32x4_t, sum[s4]) + t : t;     // "O <- B_in + O"
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o), o_rsrc, lo[s4], 0, LINE_AUX);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    // row r of the wave tile's row block i: 64-column rows of bf16 (128 bytes), their eight 16-byte
                    // chunks XOR-ed with the row so that the rows spread over the banks
                    const f32x4_t o = acc_get(i, j, g);
                    bf16x4_t h;
                    h[0] = static_cast<__bf16>(o[0]);
                    h[1] = static_cast<__bf16>(o[1]);
                    h[2] = static_cast<__bf16>(o[2]);
                    h[3] = static_cast<__bf16>(o[3]);
                    const int r = MF16 ? 16 * (g >> 1) + (lane & 15) : lane & 31;
                    const int ch = j * 4 + (MF16 ? 2 * (g & 1) + (lane >> 5) : g);
                    const int half = MF16 ? (lane >> 4) & 1 : lane >> 5;
                    *reinterpret_cast<bf16x4_t *>(scr + r * 128 + ((ch ^ (r & 7)) << 4) + half * 8) = h;
                }
            static_assert(!OUT_BF16 || TN == 2, "a wave tile row of 64 bf16 columns is one 128-byte line");
            const int c = lane & 7, r8 = lane >> 3;                  // eight 16-byte chunks (8 columns each) per row
            const int sn = n0 + wn * WTN + c * 8;
#pragma unroll
            for (int s4 = 0; s4 < 4; ++s4) {
                const int row = 8 * s4 + r8;
                const u32x4_t t = *reinterpret_cast<const u32x4_t *>(scr + row * 128 + ((c ^ (row & 7)) << 4));
                const int sm = m0 + wm * WTM + i * 32 + row;
                const int so = (sm < M && sn < N) ? (int)(((int64_t)sm * P.ldo + sn) * 2) : (int)OOB;
                __builtin_amdgcn_raw_buffer_store_b128(t, o_rsrc, so, 0, 0);
            }
        }
    }
    if constexpr (PERSIST)
        __syncthreads();                             // every wave is done with the LDS stages
    item += item_stride;
    } while (PERSIST && item < n_items);             // next work item
}

template <int BM, int BN, int WGM, int WGN, int NS, bool SPREAD>
hipError_t launch_cfg(const GemmParams &p, bool w_kn, bool out_bf16, hipStream_t s, int num_cu)
{
    bool any_recv = p.n_steps == 0 && p.recv != nullptr;     // (a persistent launch ignores recv)
    for (int j = 0; j < p.n_steps; ++j)
        any_recv = any_recv || p.recv_step[j] != nullptr;
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    int wgs = tiles_m * tiles_n * p.splits + p.cp_wgs;
    if (p.n_steps > 0) {                             // persistent: a grid that fills the chip once
        constexpr int per_cu = (NS * (BM + BN) * 64 * 2 <= 80 * 1024) ? 2 : 1;
        const int items = tiles_m * tiles_n * p.n_steps;
        wgs = items < num_cu * per_cu ? items : num_cu * per_cu;
        if (p.xcd_steps)                             // whole octets of workgroups: the same number per XCD
            wgs = (tiles_m * tiles_n * p.n_steps / 8 < num_cu * per_cu / 8 ? tiles_m * tiles_n * p.n_steps / 8
                                                                            : num_cu * per_cu / 8) * 8;
        if (const int cap = tuning().persist_wgs; cap >= 8 && cap < wgs)   // override: leave compute units free
            wgs = p.xcd_steps ? cap / 8 * 8 : cap;
    }
    const dim3 grid(wgs), block(64 * WGM * WGN);
    if (p.n_steps > 0) {                             // persistent rank step: fp32 or bf16 output, either weight order
        // (256x256 tile: the main loop on 16x16x32 MFMAs where the launcher asks for it, GemmParams::mfma16)
        auto go = [&](auto wkn, auto obf, auto recv, auto nt) {
            constexpr bool WKN = decltype(wkn)::value, OBF = decltype(obf)::value, RV = decltype(recv)::value, NTP = decltype(nt)::value;
            if constexpr (BM == 256 && BN == 256)
                if (p.mfma16) {
                    hipLaunchKernelGGL((gemm_bf16_dl_kernel<BM, BN, WGM, WGN, NS, SPREAD, WKN, OBF, RV, false, true, true, 0, NTP>),
                                       grid, block, 0, s, p, tiles_m, tiles_n);
                    return;
                }
            hipLaunchKernelGGL((gemm_bf16_dl_kernel<BM, BN, WGM, WGN, NS, SPREAD, WKN, OBF, RV, false, true, false, 0, NTP>),
                               grid, block, 0, s, p, tiles_m, tiles_n);
        };
        const auto yes = std::true_type{};
        const auto no = std::false_type{};
        if (p.a_t) {                                 // (whole 256x256 tiles: the 16x16x32 main loop, see the launcher)
            if constexpr (BM == 256 && BN == 256)
                if (w_kn && !out_bf16 && p.mfma16) {
                    auto go_t = [&](auto recv, auto hops, auto nt) {
                        hipLaunchKernelGGL((gemm_bf16_dl_kernel<BM, BN, WGM, WGN, NS, SPREAD, true, false, decltype(recv)::value, true, true, true,
                                                                decltype(hops)::value, decltype(nt)::value>), grid, block, 0, s, p, tiles_m, tiles_n);
                    };
                    auto go_nt = [&](auto hops) { p.non_temporal ? go_t(no, hops, yes) : go_t(no, hops, no); };
                    if (any_recv)
                        go_t(yes, std::integral_constant<int, 0>{}, no);
                    else if (p.hop_tiles == 0)
                        go_nt(std::integral_constant<int, 0>{});
                    else
                        p.hop_right ? go_nt(std::integral_constant<int, 2>{}) : go_nt(std::integral_constant<int, 1>{});
                    return hipGetLastError();
                }
            return hipErrorInvalidValue;
        }
        auto go_f32 = [&](auto wkn, auto recv) { p.non_temporal ? go(wkn, no, recv, yes) : go(wkn, no, recv, no); };
        auto go_w = [&](auto wkn) { out_bf16 ? go(wkn, yes, no, no) : any_recv ? go_f32(wkn, yes) : go_f32(wkn, no); };
        w_kn ? go_w(yes) : go_w(no);
        return hipGetLastError();
    }
    auto go = [&](auto wkn, auto obf, auto recv, auto a_t) {
        hipLaunchKernelGGL((gemm_bf16_dl_kernel<BM, BN, WGM, WGN, NS, SPREAD, decltype(wkn)::value, decltype(obf)::value, decltype(recv)::value,
                                                decltype(a_t)::value>), grid, block, 0, s, p, tiles_m, tiles_n);
    };
    const auto yes = std::true_type{};
    const auto no = std::false_type{};
    if (p.a_t) {
        if (!w_kn || out_bf16)
            return hipErrorInvalidValue;
        any_recv ? go(yes, no, yes, yes) : go(yes, no, no, yes);
    } else if (w_kn) {
        out_bf16 ? go(yes, yes, no, no) : any_recv ? go(yes, no, yes, no) : go(yes, no, no, no);
    } else {
        out_bf16 ? go(no, yes, no, no) : any_recv ? go(no, no, yes, no) : go(no, no, no, no);
    }
    return hipGetLastError();
}

}  // namespace

bool gemm_bf16_dl_supported(const GemmParams &p, bool w_kn)
{
    // byte extents of operands and outputs must stay below 2^31 (32-bit buffer offsets, OOB marker above them)
    const int64_t lim = (int64_t)1 << 31;
    const int64_t a_bytes = ((int64_t)(p.a_t ? p.K : p.M) * p.lda) * 2;
    const int64_t w_bytes = ((int64_t)(w_kn ? p.K : p.N) * p.ldw) * 2;
    const int64_t o_bytes = ((int64_t)p.M * p.ldo) * 4;
    return p.M > 0 && p.N > 0 && p.K > 0 && a_bytes < lim && w_bytes < lim && o_bytes < lim;
}

// Can a persistent all-gather launch carry its deliveries (GemmParams::land_step with steps that add nothing)?  Every
// tile shape can.  Slices with padding between their rows only over whole k-tiles: a copy in front moves the padding and the
// kernel does not, and which of the two a caller finds is part of the interface.  (All slices whose k is no multiple of 64
// used to be copied in front, us per rank step copied / carried: 4 x 130 x 2280 x 1696 25.4 / 16.6, 8 x 264 x 632 x 2848 40.0 /
// 26.4, 8 x 103 x 2176 x 816 17.9 / 12.5, 4 x 177 x 2256 x 5976 73.5 / 48.3, 8 x 705 x 4888 x 4184 246 / 242; of 70 drawn ones of 20
// GFLOP and more 0.88 on average, three slower by 1 to 3 %, and [n x k] 4 x 400 x 4808 x 4536, one round on 152 compute units, 120 /
// 128.  On two streams, copied in groups under the launches / carried: 8 x 173 x 1040 x 1720 46.0 / 38.2, 4 x 654 x 400 x 3232 59.6 /
// 48.1, 8 x 904 x 504 x 3512 84.7 / 78.5; of 30 drawn ones 0.88, none over 1 % slower.)
bool gemm_bf16_dl_carries_operand(const GemmParams &p)
{
    return p.n_steps > 0 && !p.a_t && (p.K % BK == 0 || p.lda == p.K);
}

// ... and a weight gradient (GemmParams::hop_tiles) on 256x256 tiles?  Whole tiles, blocks of whole k-tiles, two at the least (the
// prologue requests two), at rows without padding between them.
bool gemm_bf16_dl_carries_gathered(const GemmParams &p)
{
    return p.a_t && p.recv == nullptr && p.hop_tiles >= 2 && p.K % (p.hop_tiles * BK) == 0 && p.K / (p.hop_tiles * BK) < GemmParams::MAX_STEPS &&
           p.M % 256 == 0 && p.N % 256 == 0 && (p.hop_right ? p.ldw == p.N : p.lda == p.M);
}

hipError_t launch_gemm_bf16_dl(const GemmParams &p_in, bool w_kn, bool out_bf16, hipStream_t s, TileChoice t, int num_cu)
{
    if (p_in.n_steps > 0 && p_in.wait_flag != nullptr)
        return hipErrorInvalidValue;                  // the work-item loop waits for nothing
    GemmParams p = p_in;
    const Tuning tn = tuning();
    p.splits = t.splitk < 1 ? 1 : t.splitk;
    const int nk_all = (p.K + BK - 1) / BK;
    if (p.splits > nk_all)
        p.splits = nk_all;
    const int64_t tiles = (int64_t)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn);
    if (p.splits > 1 && (p.ws == nullptr || p.counters == nullptr || tiles > p.max_tiles ||
                         (size_t)tiles * p.splits * t.bm * t.bn * sizeof(float) > p.ws_bytes))
        p.splits = 1;                          // no (or too small a) workspace: plain kernel
    if (p.cp_src == nullptr || p.cp_dst == nullptr || p.cp_bytes == 0)
        p.cp_wgs = 0;
    // A single step is a rank step of one: the 16x16x32 main loop of whole 256x256 tiles, bands of tile columns per XCD (us per
    // step, launched for itself / as this: [n x k] weights, 2048 x 8192 x 3584 111 / 102, 4096 x 8192 x 1376 136 / 125; all-gather
    // 4096 x 4096 x 8192 213 / 205).
    // A weight gradient only where it is whole 256x256 tiles (8192 rows at once into 8192 x 3584 389 / 361, into 3584 x 8192
    // 388 / 346, in eight steps added in place 660 / 638 and 702 / 655); on the smaller tiles it loses by it: 512 rows into
    // 1376 x 4096 110 / 120, 300 into 4096 x 2048 141 / 144, 64 into 2048 x 2048 71 / 74.
    const bool whole_256 = t.bm == 256 && t.bn == 256 && p.M % 256 == 0 && p.N % 256 == 0 && tn.mfma16 != 0;
    if (p.hop_tiles > 0 && !(p.n_steps == 0 && p.a_t && whole_256 && p.splits == 1 && p.wait_flag == nullptr && p.cp_wgs == 0))
        return hipErrorInvalidValue;                  // callers ask gemm_bf16_carries_gathered first
    if (p.n_steps == 0 && (!p.a_t || whole_256) && p.splits == 1 && p.wait_flag == nullptr && p.cp_wgs == 0) {
        p.n_steps = 1;
        p.A_step[0] = p.A;
        p.recv_step[0] = p.recv;
        p.out_step[0] = p.out;
    }
    if (p.n_steps > 0) {
        for (int j = 0; j < p.n_steps; ++j)
            if (p.land_step[j] != nullptr && p.recv_step[j] == nullptr && !gemm_bf16_dl_carries_operand(p) &&
                !(p.n_steps == 1 && whole_256 && gemm_bf16_dl_carries_gathered(p)))
                return hipErrorInvalidValue;          // callers ask gemm_bf16_carries_delivery first
        p.splits = 1;
        p.cp_wgs = 0;
        p.cp_bytes = 0;
        // overrides: xcd_steps 0 = every XCD takes a band of every step; k_rotate 0 = every XCD walks k from 0
        // (whole steps per XCD not when one step carries the sum of several received partials: that step's
        // epilogue is heavy and would fall on one XCD)
        // (... or, with fewer steps than XCDs -- a group of steps launched on its own --, 8 / NB step groups x NB bands
        // of tile columns, which needs NB to divide the tile columns and 8 / NB the steps)
        const int tiles_n_ = (p.N + t.bn - 1) / t.bn;
        bool cut = false;
        for (int nb = 1; nb <= 8; nb *= 2)
            cut = cut || (tiles_n_ % nb == 0 && p.n_steps % (8 / nb) == 0);
        p.xcd_steps = cut && num_cu % 8 == 0 && p.n_recv_more == 0 && tn.xcd_steps != 0;
        // Step groups x column bands: per k-tile the 32 (or fewer) workgroups of an XCD that run side by side fetch
        // `a` left-operand bands of bm rows and `b` weight bands of bn columns, a = (step, tile row) pairs of the XCD
        // (at most its workgroups), b = the columns they spread over; the number of bands NB that makes a bm + b bn
        // smallest (ties: the fewest bands).  7B down-projection (2 tile rows x 16 tile columns per step): NB = 2,
        // 12 instead of 18 bands; the 70B shapes stay at NB = 1 (4 x 8 is already the best cut of 32).
        p.xcd_bands = 1;
        if (p.xcd_steps) {
            const int tiles_m = (p.M + t.bm - 1) / t.bm, tiles_n = (p.N + t.bn - 1) / t.bn;
            const int per_cu = (t.bm == 128 && t.bn == 128 && !t.deep) ? 2 : 1;
            const int items_x = tiles_m * tiles_n * p.n_steps / 8;
            const int wgs_x = items_x < num_cu * per_cu / 8 ? items_x : num_cu * per_cu / 8;
            long best = -1;
            for (int nb = 1; nb <= 8; nb *= 2) {
                if (tiles_n % nb != 0 || p.n_steps % (8 / nb) != 0)
                    continue;
                if (tn.xcd_bands > 0 && nb != tn.xcd_bands && p.n_steps % 8 == 0)
                    continue;                          // override: this many bands where the shape allows it
                const int rows = p.n_steps / (8 / nb) * tiles_m;
                const int a = rows < wgs_x ? rows : wgs_x;
                const int cols = tiles_n / nb;
                int b = (wgs_x + a - 1) / a;
                b = b < cols ? b : cols;
                const long cost = (long)a * t.bm + (long)b * t.bn;
                if (best < 0 || cost < best) {
                    best = cost;
                    p.xcd_bands = nb;
                }
            }
            if (best < 0 && p.n_steps % 8 != 0)
                p.xcd_steps = false;                   // (no cut fits: every XCD takes a band of every step)
        }
        // (measured with whole steps per XCD only; a ragged k tail stays the last k-tile of every work item,
        // which keeps all earlier iterations of the 256x256 main loop branch-free)
        // (nor where the pairwise schedule carries its deliveries: the sums are bit for bit those of its copied mode, whose last
        // step sums several partials and so keeps the k order)
        p.k_rotate = p.xcd_steps && tn.k_rotate != 0 && p.K % BK == 0 && !p.k_in_order && p.hop_tiles == 0;
        // fp32 lines past the caches: what a launch writes it never reads again, and B_in is read once.  Where rows begin
        // and end on 128-byte lines -- the caches put the halves of a shared line together.  us per carried rank step,
        // cached against not: 8 x 1024 x 8192 x 1024 232 / 216, 8 x 512 x 4096 x 1376 72.2 / 69.6, 8 x 128 x 4096 x 512 (46 MB)
        // 19.7 / 20.3, 8 x 100 x 2048 x 2048 (18 MB) 27.3 / 26.6, all-gather 8 x 1024 x 3584 x 8192 380 / 374; rows off the
        // lines: 2 x 1000 x 3000 x 520 25.1 / 32.3, 4 x 333 x 2088 x 1096 23.9 / 26.3.
        // Not, without a B_in, where rows lie a multiple of 16 KiB apart -- the lines of a tile then fall on few memory channels,
        // which the caches' write-backs spread over time --, unless the L2 caches hold the output anyway (32 MiB; what is left in
        // them is written back at the end of the launch) or the launch moves more than the last-level cache holds for
        // whoever reads the output next (256 MiB, and an eighth).  us cached / past the caches, buffers that come round / fresh
        // ones: all-gather steps 4096 x 8192 x 1024 71 / 88 and 76 / 89, with a reader behind 99 / 119 and 107 / 128; 2048 x 8192 x
        // 1024 38 / 41 and 38 / 42; all-gather 8 x 512 x 8192 x 512 49 / 57 and 57 / 57; 512 rows into 4096 x 4096 25.5 / 27.7.
        // Other rows: 4096 x 7936 x 1024 70 / 71 and 74 / 74, 4096 x 6144 x 1024 60 / 57 and 66 / 57.  1024 x 4096 x 1024 15.6 / 14.2
        // and 17.3 / 15.2.  All-gather 8 x 1024 x 8192 x 1024 (302 MB) 138 / 139 and 145 / 142, with a reader 212 / 220; 8 x 1024 x
        // 8192 x 3584 (386 MB) 367 / 361 and 367 / 362, with a reader 429 / 429.
        bool any_recv = false;
        uintptr_t low = (uintptr_t)(p.ldo * 4) | (uintptr_t)p.N * 4;
        for (int j = 0; j < p.n_steps; ++j) {
            low |= reinterpret_cast<uintptr_t>(p.out_step[j]) | reinterpret_cast<uintptr_t>(p.recv_step[j]) |
                   (p.recv_step[j] != nullptr ? reinterpret_cast<uintptr_t>(p.land_step[j]) : 0);
            any_recv = any_recv || p.recv_step[j] != nullptr;
        }
        const int64_t out_bytes = (int64_t)p.M * p.N * 4 * p.n_steps;
        const int64_t moved = out_bytes + ((int64_t)p.M * p.n_steps + p.N) * p.K * 2;
        p.non_temporal = !out_bf16 && low % 128 == 0 &&
                         (any_recv || p.ldo * 4 % (16 << 10) != 0 || out_bytes <= (int64_t)32 << 20 || moved > (int64_t)288 << 20);
        // Half the workgroups land their deliveries in front of the main loop where the work items fill the chip and their
        // multiplications do not far outlast the memory's part, which scales with what of the tiles lies inside the
        // matrix.  us per carried rank step, all in the epilogue / half in front: 8 x 1024 x 8192 at k = 512 180 / 170, 1024
        // 218 / 209, 2560 356 / 346, 3072 403 / 387, 3584 437 / 442; 8 x 512 x 4096 at 256 43.7 / 40.2, 1376 69.6 / 64.9, 2560 91.5 /
        // 86.9.  The smaller tiles, with two row blocks requested early: 8 x 256 x 4096 x 512 27.1 / 23.0, 2 x 512 x 4096 x 1376
        // 25.4 / 25.1, 8 x 300 x 4096 x 2048 77.7 / 79.8.  Fewer work items than compute units: 4 x 333 x 2088 x 1096 23.9 / 25.5,
        // 8 x 100 x 2048 x 2048 26.6 / 27.4.
        const int64_t items = tiles * p.n_steps;
        p.land_first = items >= num_cu && (int64_t)nk_all * tiles * t.bm * t.bn <= (int64_t)(t.bm == 256 && t.bn == 256 ? 48 : 24) * p.M * p.N;
        p.mfma16 = whole_256;                        // (override: COMMFUSE_MFMA16 = 0 | 1)
    }
    // LDS stages: as many as fit (160 KiB per CU); the 128x128 tile comes with two (two workgroups share a CU) or four (one
    // workgroup per CU, tiles requested three ahead).  Spreading the loads over the MFMAs beats a burst behind the barrier
    // (all-gather 8 x 512 x 1536 x 4096 on 256x128 61 / 54 us, reduce-scatter 2 x 128 x 5120 x 5248 on 128x128 53 / 37) but for
    // two workgroups per CU over long k ranges, which cover for each other (8 x 299 x 4808 x 4104 160 / 168, 8 x 896 x 4224 x
    // 4480 271 / 272; 8 x 480 x 2112 x 1408 41 / 36).
    if (t.bm == 256 && t.bn == 256) return launch_cfg<256, 256, 2, 4, 2, true>(p, w_kn, out_bf16, s, num_cu);
    if (t.bm == 256 && t.bn == 128) return launch_cfg<256, 128, 4, 2, 2, true>(p, w_kn, out_bf16, s, num_cu);
    if (t.deep) return launch_cfg<128, 128, 2, 2, 4, true>(p, w_kn, out_bf16, s, num_cu);
    if (nk_all <= 48) return launch_cfg<128, 128, 2, 2, 2, true>(p, w_kn, out_bf16, s, num_cu);
    return launch_cfg<128, 128, 2, 2, 2, false>(p, w_kn, out_bf16, s, num_cu);
}

}  // namespace cf
