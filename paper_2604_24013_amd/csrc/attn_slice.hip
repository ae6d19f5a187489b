// Attention of one query slice against the rank's full keys and values (Alg. 4: scores = Q_s[l] K^T,
// Softmax, times V), bf16 operands, fp32 accumulation and fp32 online softmax, for gfx950.
//
// Query blocks: one workgroup = 8 or 4 waves of 32 queries each of one (batch element, head), which share the key tiles; it
// walks over the keys in tiles of 64, a pipeline one tile deep (the scores of the next tile under the exponentials of this one).
// Keys over waves: one workgroup = 32 queries, its eight waves share out the keys in tiles of 32.  Per tile and wave:
//   S^T = K Q^T      v_mfma_f32_32x32x16_bf16 with the key tile as the MFMA "A" operand and the wave's
//                    queries (kept in registers for the whole walk) as "B": a lane then owns ONE query
//                    (lane & 31) and 16 of every 32 keys, so the softmax statistics of a query live in two
//                    lanes (lane, lane ^ 32) and need one cross-lane exchange per tile;
//   online softmax   m' = max(m, max S), P = exp2(S - m'), l = l * exp2(m - m') + sum P, O *= exp2(m - m')
//                    (query blocks keep m until a probability would exceed 2^8);
//   O^T += V^T P^T   the probabilities, rounded to bf16, are already in the register layout of an MFMA "B"
//                    operand if the 16 contraction slots of a slice are taken to mean the keys the lane
//                    holds (a fixed permutation of the slice's keys); the V tile stays [key x d] in LDS and
//                    its transposed fragments are fetched with the transposing LDS read at the row offsets
//                    of that same permutation.  No data moves between lanes, no P tile goes through LDS.
// K and V tiles go global -> LDS directly (buffer_load ... lds; query blocks: double-buffered); a key row of 256 bytes has
// its sixteen 16-byte chunks XOR-ed with (key & 15) so that the fragment reads of 16 consecutive keys hit 16
// different bank groups; the V tile uses the [k x n] weight-tile layout of the chunk GEMM.
// Keys beyond the sequence read as zero through the buffer bounds check and are masked to -inf; query rows
// beyond the slice are computed on zeros and not stored.
#include "cf_internal.h"

#include <cmath>
#include <cstdlib>
#include <type_traits>
#include <utility>

namespace cf {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));

constexpr unsigned OOB = 0x80000000u;
constexpr int DH = 128;                  // head dimension this kernel is written for
constexpr int BKV = 64;                  // keys per tile
constexpr int ROWB = DH * 2;             // bytes of one key / value row
constexpr int TILE_BYTES = BKV * ROWB;   // 16 KiB

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

// Wave-wide 16-byte-per-lane load from global memory straight into LDS (lane L lands at lds_addr + 16 L).
__device__ __forceinline__ void direct_load_16(i32x4_t rsrc, unsigned voffset, int soffset, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "buffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voffset), "s"(rsrc), "s"(soffset)
                 : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// f(FIRST), f(FIRST + STEP), ... as compile-time constants
template <int FIRST, int STEP, int... I, typename F>
__device__ __forceinline__ void each(F &f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, FIRST + STEP * I>{}), ...);
}

// Query blocks: NW waves of 32 queries each share the key tiles (NW = 8: two waves per SIMD of one workgroup; NW = 4: two
// workgroups per compute unit).
//
// What bounds it: the matrix pipe, with the vector ALU (maximum, exponential, conversion, row sum) and LDS (every wave reads
// every K and V tile) close behind: 2048 / 1700 / 2048 cycles per 64-key tile and compute unit.  So none may wait for another.
// The loop is a pipeline of one tile's depth inside each wave: the scores of tile t+1 are multiplied while tile t is
// exponentiated, and the maximum of tile t+1 is taken while tile t multiplies V, all in one basic block, MFMAs, exponentials and
// LDS reads dealt out evenly.  Before, a wave multiplied,
// exponentiated and multiplied again, and only its neighbour on the SIMD covered for it.  us, before / now: 8 heads x 8192
// queries x 8192 keys (NW = 8, the chip full) 256 / 237 = 1.16 PFLOP/s at 1.88 GHz (the chip's power limit; 58 % of the cycles
// are MFMAs, 44 before); 4 heads (one wave per SIMD, NW = 4) 192 / 140; 8 heads x 1024 queries, a quarter of the chip, 190 / 122.
// What is left, by parts taken out: without the exponentials 223, without any softmax 206, without the LDS reads 216.
// (A row sum of its own per tile instead of per pair of tiles: one addition and one move more per tile, sixteen tiles a
// workgroup -- 8 heads x 1024 queries x 8192 keys in eight splits -- 51.1 / 52.2; no sum between the keys and the row's, which
// loses what is under half a unit in the last place of the row so far, 51.3.)
template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void attn_slice_kernel(AttnParams P)
{
    constexpr int NT = 64 * NW;          // threads per workgroup
    constexpr int BQ = NW * 32;          // queries per workgroup
    constexpr int KT = BKV / 32;         // 32-key MFMA tiles per key tile
    constexpr int DS = DH / 16;          // 16-wide d slices (contraction of S^T)
    constexpr int DT = DH / 32;          // 32-wide d tiles (rows of O^T)
    constexpr int LOADS = TILE_BYTES / 1024 / NW;   // wave-loads per wave of a K or V tile
    constexpr int V_BASE = 2 * TILE_BYTES;          // LDS: two K tiles, two V tiles

    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * 2 * TILE_BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, lh = lane >> 5;

    const int qblocks = (P.c + BQ - 1) / BQ;
    const int KSP = P.ksplit;                                        // workgroups sharing a query block
    const int split = blockIdx.x % KSP;
    const int group = blockIdx.x / KSP;                              // (slice, batch element, head, query block)
    const int qb = group % qblocks;
    const int head = (group / qblocks) % P.heads;
    const int b = (group / (qblocks * P.heads)) % P.batch;
    const int slice = P.l + group / (qblocks * P.heads * P.batch);
    const int S = P.S;

    const size_t mat = (size_t)S * DH;                               // elements of one (b, head) matrix
    const __bf16 *Qm = static_cast<const __bf16 *>(P.Q) + ((size_t)b * P.heads + head) * mat;
    const __bf16 *Km = static_cast<const __bf16 *>(P.K) + ((size_t)b * P.heads + head) * mat;
    const __bf16 *Vm = static_cast<const __bf16 *>(P.V) + ((size_t)b * P.heads + head) * mat;
    const i32x4_t k_rsrc = make_rsrc(Km, (unsigned)(mat * 2));
    const i32x4_t v_rsrc = make_rsrc(Vm, (unsigned)(mat * 2));
    const unsigned lds_base = __builtin_amdgcn_readfirstlane(
        (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)smem);

    // The wave's queries as MFMA "B" fragments: lane (lq, lh) holds d = 16 ks + 8 lh + 0..7 of query lq.
    const int q_in_slice = qb * BQ + wave * 32;                      // first query of this wave in the slice
    const int qi = q_in_slice + lq;
    bf16x8_t qf[DS];
    {
        const __bf16 *qrow = Qm + (size_t)(slice * P.c + (qi < P.c ? qi : 0)) * DH;   // (a query beyond the slice is not stored)
#pragma unroll
        for (int ks = 0; ks < DS; ++ks)
            qf[ks] = *reinterpret_cast<const bf16x8_t *>(qrow + ks * 16 + lh * 8);
    }

    // Direct loads of key tile `kt` into K buffer / V buffer `buf`: wave-load j covers 4 rows of 256 bytes.
    // K: the lane at LDS chunk position cp of row r fetches global chunk cp ^ (r & 15).
    // V: [k x n] weight-tile layout: the 64-byte groups of a row are XOR-ed with (row & 3).
    // (The rows of a wave-load lie a multiple of sixteen from those of the wave's first: one per-lane offset serves all.)
    static_assert(NW * 4 % 16 == 0, "key rows of a wave-load");
    const int ld_row = wave * 4 + (lane >> 4), ld_cp = lane & 15;    // key row inside the tile, chunk of wave-load 0
    const unsigned k_off = (unsigned)(ld_row * ROWB + ((ld_cp ^ (ld_row & 15)) << 4));
    const unsigned v_off = (unsigned)(ld_row * ROWB + (((ld_cp >> 2) ^ (ld_row & 3)) << 6) + ((ld_cp & 3) << 4));
    auto issue = [&](int kt, const i32x4_t &rs, unsigned off, unsigned lds) __attribute__((always_inline)) {
        const int key0 = kt * BKV;
        const int left = S - key0;                                   // keys of the tile (none: it reads as zero and moves no data)
        const int soff = left > 0 ? key0 * ROWB : 0;
#pragma unroll
        for (int j = 0; j < LOADS; ++j)
            direct_load_16(rs, ld_row + j * NW * 4 < left ? off : OOB, soff + j * NW * 4 * ROWB, lds + wave * 1024 + j * NW * 1024);
    };

    // Fragment addresses inside a buffer.
    // K as "A" operand: lane (key = lq, lh) reads chunk (2 ks + lh) of its key row, swizzled.
    // V^T as "A" operand: transposing reads; lane (blk = lane >> 4, i16 = lane & 15); the two reads of a
    // slice start at key rows 4 lh + (i16 >> 2) and 8 more (the permutation the probabilities come in).
    int k_addr[DS];
#pragma unroll
    for (int ks = 0; ks < DS; ++ks)
        k_addr[ks] = lq * ROWB + (((2 * ks + lh) ^ (lq & 15)) << 4);
    const int blk = lane >> 4, i16 = lane & 15;
    const int v_kl = 4 * (blk >> 1) + (i16 >> 2);
    const int v_nl = (blk & 1) * 16 + (i16 & 3) * 4;
    int v_addr[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
        v_addr[t] = V_BASE + v_kl * ROWB + (((t) ^ (v_kl & 3)) << 6) + v_nl * 2;

    f32x16_t oacc[DT];
    float m_run = -3.402823466e38f;      // (finite: against -inf a tile whose scores are all -inf would give NaN)
    float l_run = 0.0f;                  // of the keys this lane holds; the query's other half lives in lane ^ 32
    float l_pair = 0.0f;                 // ... of a pair of tiles, which adds up by itself: what is small meets the row's sum once per pair
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            oacc[d][e] = 0.0f;
    const float sl2 = P.scale * 1.4426950408889634f;                 // scores are kept in units of log2(e)

    const int nkt_all = (S + BKV - 1) / BKV;
    const int kt0 = (int)(((long long)nkt_all * split) / KSP);       // this workgroup's key tiles: [kt0, nkt)
    const int nkt = (int)(((long long)nkt_all * (split + 1)) / KSP);

    // S^T = K Q^T of the tile in K buffer `buf`; register 4g+e of key tile j is key 32 j + 8 g + 4 lh + e
    auto scores = [&](int buf, f32x16_t (&sn)[KT]) __attribute__((always_inline)) {
        const unsigned char *st = smem + buf * TILE_BYTES;
#pragma unroll
        for (int j = 0; j < KT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                sn[j][e] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < DS; ++ks)
#pragma unroll
            for (int j = 0; j < KT; ++j) {
                const bf16x8_t kf = *reinterpret_cast<const bf16x8_t *>(st + k_addr[ks] + j * 32 * ROWB);
                sn[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sn[j], 0, 0, 0);
            }
    };
    auto maximum = [&](const f32x16_t (&sn)[KT]) __attribute__((always_inline)) {
        float mx = sn[0][0];
#pragma unroll
        for (int j = 0; j < KT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                mx = fmaxf(mx, sn[j][r]);
        return mx;
    };
    // Before a tile's scores are exponentiated: keys beyond the sequence are masked (the one tile that can hold them only), and
    // the running reference m is raised where the tile's maximum exceeds it by more than 2^RAISE (probabilities then stay below
    // 2^RAISE: no overflow), so the rescaling of the accumulators is rare and sits in a wave-uniform branch.  (The largest
    // probability is then rounded like any other; choose_attn says what that means for the choice between the kernels.)
    constexpr float RAISE = 8.0f;
    auto settle = [&](int kt, f32x16_t (&sn)[KT], float mx) __attribute__((always_inline)) {
        if ((kt + 1) * BKV > S) {                                    // uniform
            float ninf = -INFINITY;
            asm volatile("" : "+v"(ninf));                           // (keeps this a branch: not 32 selects in every tile)
#pragma unroll
            for (int j = 0; j < KT; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kt * BKV + j * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
                    if (key >= S)
                        sn[j][r] = ninf;
                }
            mx = maximum(sn);
        }
        const auto both = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, mx), __builtin_bit_cast(unsigned, mx), false, false);
        const unsigned half0 = both[0], half1 = both[1];
        const float mxs = fmaxf(__builtin_bit_cast(float, half0), __builtin_bit_cast(float, half1)) * sl2;   // scale > 0: the maximum of the scaled scores
        if (__builtin_amdgcn_ballot_w64(mxs > m_run + RAISE) != 0) { // (not where all scores so far are -inf)
            const float m_new = fmaxf(m_run, mxs);
            float alpha = exp2f(m_run - m_new);                      // 0 on the first tile with a finite score
            asm volatile("" : "+v"(alpha));                          // (keeps this a branch, as above)
            m_run = m_new;
            l_run *= alpha;
            l_pair *= alpha;
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    oacc[d][e] *= alpha;
        }
    };
    // One tile: probabilities P = exp2(S - m) rounded to bf16, their row sums (exactly the rounded values that multiply V, two to
    // a dot product with ones), O^T += V^T P^T; and under it, with `next`, the scores of tile kt+1 and their maximum.  Tile kt
    // and tile kt+1 lie in buffers B and 1 - B.  Thirty-two segments of one MFMA each -- sixteen of the scores, sixteen of V's
    // product --, the fragment of the third segment ahead requested in each, the 32 exponentials of the tile spread over
    // segments 0 .. 22 (before the slice of V that they multiply) and the maximum over the last eight.
    bf16x2_t ones;
    ones[0] = ones[1] = (__bf16)1.0f;
    auto tile = [&](int kt, f32x16_t (&sc)[KT], f32x16_t (&sn)[KT], auto b_tag, auto next_tag) __attribute__((always_inline)) {
        constexpr int B = decltype(b_tag)::value;
        constexpr bool NEXT = decltype(next_tag)::value;
        constexpr int FIRST = NEXT ? 0 : 16;                         // first segment
        constexpr int AHEAD = 3;
        bf16x8_t frag[AHEAD + 1], pf[KT * 2];                        // pf: "B" fragments of the 16-key slices
        auto fetch = [&](auto s_tag) __attribute__((always_inline)) {
            constexpr int s = decltype(s_tag)::value;
            if constexpr (s < 16) {
                frag[s % (AHEAD + 1)] = *reinterpret_cast<const bf16x8_t *>(smem + k_addr[s >> 1] + (1 - B) * TILE_BYTES + (s & 1) * 32 * ROWB);
            } else if constexpr (s < 32) {
                const unsigned char *pv = smem + v_addr[s & 3] + B * TILE_BYTES + ((s - 16) >> 2) * 16 * ROWB;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pv));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)(pv + 8 * ROWB));
                frag[s % (AHEAD + 1)] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        const float nm = -m_run;
        auto exponentials = [&](auto e_tag) __attribute__((always_inline)) {   // of elements e and e+1
            constexpr int e = decltype(e_tag)::value;
            bf16x2_t two;
#pragma unroll
            for (int i = 0; i < 2; ++i)                              // bare v_exp_f32: arguments below -126 give 0
                two[i] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[e >> 4][(e & 15) + i], sl2, nm));
            pf[e >> 3][(e & 7)] = two[0];
            pf[e >> 3][(e & 7) + 1] = two[1];
            l_pair = __builtin_amdgcn_fdot2_f32_bf16(two, ones, e == 0 && B == 0 ? 0.0f : l_pair, false);
            if constexpr (e == 30 && (B == 1 || !NEXT))
                l_run += l_pair;
        };
        float mx = -INFINITY;
        auto segment = [&](auto s_tag) __attribute__((always_inline)) {
            constexpr int s = decltype(s_tag)::value;
            fetch(std::integral_constant<int, s + AHEAD>{});
            if constexpr (s < 16) {
                if constexpr (s < 2)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        sn[s & 1][e] = 0.0f;
                sn[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[s % (AHEAD + 1)], qf[s >> 1], sn[s & 1], 0, 0, 0);
                if constexpr (s % 4 != 3)
                    exponentials(std::integral_constant<int, 2 * (s - s / 4)>{});
            } else {
                oacc[s & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[s % (AHEAD + 1)], pf[(s - 16) >> 2], oacc[s & 3], 0, 0, 0);
                if constexpr (NEXT && s < 24 && s % 2 == 0)
                    exponentials(std::integral_constant<int, 24 + (s - 16)>{});
                if constexpr (NEXT && s >= 24) {
                    constexpr int r = 4 * ((s - 24) & 3);
#pragma unroll
                    for (int e = r; e < r + 4; ++e)
                        mx = fmaxf(mx, sn[(s - 24) >> 2][e]);
                    asm volatile("" : "+v"(mx));                     // (here, not where it is used)
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (NEXT) {                                        // into what the last barrier released
            issue(kt + 1, v_rsrc, v_off, lds_base + V_BASE + (1 - B) * TILE_BYTES);
            issue(kt + 2, k_rsrc, k_off, lds_base + B * TILE_BYTES);
        }
        fetch(std::integral_constant<int, FIRST>{});
        fetch(std::integral_constant<int, FIRST + 1>{});
        fetch(std::integral_constant<int, FIRST + 2>{});
        if constexpr (!NEXT)
            each<0, 2>(exponentials, std::make_integer_sequence<int, 16>{});
        __builtin_amdgcn_sched_barrier(0);
        each<FIRST, 1>(segment, std::make_integer_sequence<int, 32 - FIRST>{});
        if constexpr (NEXT) {
            settle(kt + 1, sn, mx);
            wait_vmcnt<0>();                                         // V of tile kt+1 and K of tile kt+2 have landed
            __syncthreads();                                         // ... for every wave, and V of kt, K of kt+1 are read by all
        }
    };

    issue(kt0, k_rsrc, k_off, lds_base);
    issue(kt0, v_rsrc, v_off, lds_base + V_BASE);
    issue(kt0 + 1, k_rsrc, k_off, lds_base + TILE_BYTES);
    wait_vmcnt<0>();
    __syncthreads();
    f32x16_t sa[KT], sb[KT];
    scores(0, sa);
    settle(kt0, sa, maximum(sa));
    __syncthreads();                                                 // K of tile kt0 is read by all
    using buf0 = std::integral_constant<int, 0>;
    using buf1 = std::integral_constant<int, 1>;
    int kt = kt0;
    for (; kt + 2 < nkt; kt += 2) {
        tile(kt, sa, sb, buf0{}, std::true_type{});
        tile(kt + 1, sb, sa, buf1{}, std::true_type{});
    }
    if (kt + 2 == nkt) {
        tile(kt, sa, sb, buf0{}, std::true_type{});
        tile(kt + 1, sb, sa, buf1{}, std::false_type{});
    } else {
        tile(kt, sa, sb, buf0{}, std::false_type{});
    }
    {                                                                // the whole row sum, in both lanes of the query
        const auto both = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, l_run), __builtin_bit_cast(unsigned, l_run), false, false);
        const unsigned half0 = both[0], half1 = both[1];
        l_run = __builtin_bit_cast(float, half0) + __builtin_bit_cast(float, half1);
    }

    // Key split across workgroups: park (m, l, O) in the workspace, thread-major so that every access is a
    // coalesced 4 bytes per lane; the workgroup that arrives last merges all splits (its own included) in
    // split order.  Cross-XCD visibility as in the chunk GEMM's k-split: device-coherent cache policy on
    // exactly these accesses, relaxed agent-scope atomics on the counter.
    if (KSP > 1) {
        constexpr int COHERENT = 1 | 16;
        constexpr int NV = DT * 16 + 2;                              // floats per thread
        const size_t part = (size_t)NV * NT;
        auto part_rsrc = [&](int sp) {
            return __builtin_amdgcn_make_buffer_rsrc(P.ws + ((size_t)group * KSP + sp) * part, 0, (int)(part * 4), 0x00020000);
        };
        {
            __amdgpu_buffer_rsrc_t rs = part_rsrc(split);
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    // (through a plain VGPR: storing the accumulator elements straight from their AGPRs
                    // came out of this compiler as sixteen stores of element 0)
                    float v = oacc[d][e];
                    asm volatile("" : "+v"(v));
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, ((d * 16 + e) * NT + tid) * 4, 0, COHERENT);
                }
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, m_run), rs, ((DT * 16) * NT + tid) * 4, 0, COHERENT);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, l_run), rs, ((DT * 16 + 1) * NT + tid) * 4, 0, COHERENT);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        unsigned *arrived = reinterpret_cast<unsigned *>(smem);       // the key tiles are no longer read
        if (tid == 0)
            *arrived = __hip_atomic_fetch_add(&P.counters[group], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*arrived != (unsigned)(KSP - 1))
            return;
        if (tid == 0)
            __hip_atomic_store(&P.counters[group], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        float m_all = -INFINITY;
        // Eight maxima in flight (beyond the last: the last once more).  us of eight slices with their projections, one by one / so:
        // 8 heads x 8192 keys in eight splits 642 / 630, 2 x 4 x 6944 475 / 465.  (Partials 16 bytes a lane instead of 4: in eight
        // splits 1 to 7 % slower.)
        for (int sp0 = 0; sp0 < KSP; sp0 += 8) {
            float m[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                m[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(part_rsrc(sp0 + i < KSP ? sp0 + i : KSP - 1),
                                                                                      ((DT * 16) * NT + tid) * 4, 0, COHERENT));
#pragma unroll
            for (int i = 0; i < 8; ++i)
                m_all = fmaxf(m_all, m[i]);
        }
        float l_all = 0.0f;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                oacc[d][e] = 0.0f;
        // two splits per round: their loads (2 x 66 per lane) are in flight together, the sums stay in split order
        for (int sp = 0; sp < KSP; sp += 2) {
            const bool two = sp + 1 < KSP;
            __amdgpu_buffer_rsrc_t rs0 = part_rsrc(sp), rs1 = part_rsrc(two ? sp + 1 : sp);
            auto ld = [&](__amdgpu_buffer_rsrc_t rs, int idx) {
                return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (idx * NT + tid) * 4, 0, COHERENT));
            };
            const float m0 = ld(rs0, DT * 16), l0 = ld(rs0, DT * 16 + 1);
            const float m1 = ld(rs1, DT * 16), l1 = ld(rs1, DT * 16 + 1);
            float v0[DT][16], v1[DT][16];
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    v0[d][e] = ld(rs0, d * 16 + e);
                    v1[d][e] = ld(rs1, d * 16 + e);
                }
            const float f0 = exp2f(m0 - m_all);                      // every split holds at least one key tile
            const float f1 = two ? exp2f(m1 - m_all) : 0.0f;
            l_all += l0 * f0;
            l_all += l1 * f1;
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    oacc[d][e] += f0 * v0[d][e];
                    oacc[d][e] += f1 * v1[d][e];
                }
        }
        l_run = l_all;
    }

    // O = O^T / l, rounded to bf16, written as [token x (head, d)]: the left operand of the output projection.
    __bf16 *out = static_cast<__bf16 *>(P.out) + (size_t)(slice - P.l) * P.out_slice_stride;
    const float inv = 1.0f / l_run;
    if (qi < P.c) {
        __bf16 *orow = out + ((size_t)b * P.c + qi) * P.ldo + (size_t)head * DH;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4_t h;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    h[e] = (__bf16)(oacc[d][4 * g + e] * inv);
                *reinterpret_cast<u32x2_t *>(orow + d * 32 + 8 * g + 4 * lh) = __builtin_bit_cast(u32x2_t, h);
            }
    }
}

// Keys over waves: one workgroup = 32 queries of one (batch element, head); its eight waves split the KEYS -- wave w takes
// the 32-key tiles w, w + 8, ... -- each with K and V landing zones of its own in LDS, so that there is no barrier in the
// walk and the waves of a SIMD drift apart (one multiplies while the other exponentiates).  The zones are single: the next
// K tile is requested as soon as the scores have taken its predecessor out of LDS (it travels under the softmax and the
// product with V), the next V tile after that product.  The eight partial results (m, l, unnormalised O) are merged in
// LDS by all threads.  For slices with few queries; with a workspace the keys of a query block can be split over
// `ksplit` workgroups on top, which park their merged partials (16.5 KiB each).
constexpr int KW_WAVES = 8;
constexpr int KW_PART = 64 * 64 + 2 * 64;    // floats of a workgroup's parked partial: O [8 groups][64 lanes][8], m, l [64 lanes]
__global__ __launch_bounds__(64 * KW_WAVES) void attn_keys_over_waves_kernel(AttnParams P)
{
    constexpr int NW = KW_WAVES;
    constexpr int BK = 32;                   // keys per tile
    constexpr int TB = BK * ROWB;            // 8 KiB: one K (or V) tile
    constexpr int DS = DH / 16, DT = DH / 32;
    constexpr int WAVE_LDS = 2 * TB;         // [K | V]; afterwards the wave's O: 64 registers x 64 lanes

    __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * WAVE_LDS];
    __shared__ float stat[NW][2][64];        // m, l per wave and lane

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, lh = lane >> 5;

    const int qtiles = (P.c + 31) / 32;
    const int KSP = P.ksplit;
    // neighbouring workgroups (one per XCD in turn) take different heads: with 8 heads, each XCD's L2 serves one head's K, V
    const int head = blockIdx.x % P.heads;
    int rest = blockIdx.x / P.heads;
    const int split = rest % KSP;
    rest /= KSP;
    const int qt = rest % qtiles;
    rest /= qtiles;
    const int b = rest % P.batch, slice = P.l + rest / P.batch;
    const int group = (rest * qtiles + qt) * P.heads + head;
    const int S = P.S;

    const size_t mat = (size_t)S * DH;
    const __bf16 *Qm = static_cast<const __bf16 *>(P.Q) + ((size_t)b * P.heads + head) * mat;
    const i32x4_t k_rsrc = make_rsrc(static_cast<const __bf16 *>(P.K) + ((size_t)b * P.heads + head) * mat, (unsigned)(mat * 2));
    const i32x4_t v_rsrc = make_rsrc(static_cast<const __bf16 *>(P.V) + ((size_t)b * P.heads + head) * mat, (unsigned)(mat * 2));
    const unsigned lds_base = __builtin_amdgcn_readfirstlane(
        (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)smem) + wave * WAVE_LDS;
    unsigned char *my = smem + wave * WAVE_LDS;

    const int nkt = (S + BK - 1) / BK;
    const int t0 = (int)(((long long)nkt * split) / KSP), t1 = (int)(((long long)nkt * (split + 1)) / KSP);

    // wave-load j (1 KiB) covers rows 4j .. 4j+3 of the tile; layouts as in the kernel above
    unsigned k_off[8], v_off[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int row = j * 4 + (lane >> 4);
        const int cp = lane & 15;
        k_off[j] = (unsigned)(row * ROWB + ((cp ^ (row & 15)) << 4));
        const int inrow = cp << 4;
        v_off[j] = (unsigned)(row * ROWB + (((inrow >> 6) ^ (row & 3)) << 6) + (inrow & 63));
    }
    auto issue = [&](int kt, const i32x4_t &rs, const unsigned (&off)[8], unsigned lds) __attribute__((always_inline)) {
        const int key0 = kt * BK, soff = __builtin_amdgcn_readfirstlane(key0 * ROWB);
#pragma unroll
        for (int j = 0; j < 8; ++j)          // keys beyond the sequence read as zero
            direct_load_16(rs, key0 + j * 4 + (lane >> 4) < S ? off[j] : OOB, soff, lds + j * 1024);
    };
    if (t0 + wave < t1) {
        issue(t0 + wave, k_rsrc, k_off, lds_base);
        issue(t0 + wave, v_rsrc, v_off, lds_base + TB);
    }

    const int qi = qt * 32 + lq;
    const bool q_ok = qi < P.c;
    bf16x8_t qf[DS];
    {
        const __bf16 *qrow = Qm + (size_t)(slice * P.c + (q_ok ? qi : 0)) * DH;
#pragma unroll
        for (int ks = 0; ks < DS; ++ks)
            qf[ks] = *reinterpret_cast<const bf16x8_t *>(qrow + ks * 16 + lh * 8);   // (a query beyond the slice is not stored)
    }

    const int blk = lane >> 4, i16 = lane & 15;
    const int v_kl = 4 * (blk >> 1) + (i16 >> 2);
    const int v_nl = (blk & 1) * 16 + (i16 & 3) * 4;
    int v_addr[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
        v_addr[t] = TB + v_kl * ROWB + ((t ^ (v_kl & 3)) << 6) + v_nl * 2;

    f32x16_t oacc[DT], lacc;
#pragma unroll
    for (int e = 0; e < 16; ++e)
        lacc[e] = 0.0f;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            oacc[d][e] = 0.0f;
    bf16x8_t ones;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        ones[e] = (__bf16)1.0f;
    // (finite: against -inf a tile whose scores are all -inf would give NaN, and every wave starts on a tile of its own)
    float m_run = -3.402823466e38f;
    const float sl2 = P.scale * 1.4426950408889634f;
    asm volatile("" : "+v"(qf[0]), "+v"(qf[1]), "+v"(qf[2]), "+v"(qf[3]), "+v"(qf[4]), "+v"(qf[5]), "+v"(qf[6]), "+v"(qf[7]));
    // (the queries are in registers from here on: what the waits below count are the tiles' loads alone)

    for (int kt = t0 + wave; kt < t1; kt += NW) {
        const bool more = kt + NW < t1;
        wait_vmcnt<8>();                                             // K of tile kt has landed (its V may be in flight)
        __builtin_amdgcn_sched_barrier(0);
        bf16x8_t kf[DS];
#pragma unroll
        for (int ks = 0; ks < DS; ++ks)
            kf[ks] = *reinterpret_cast<const bf16x8_t *>(my + lq * ROWB + (((2 * ks + lh) ^ (lq & 15)) << 4));
        f32x16_t sacc;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            sacc[e] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < DS; ++ks)
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], sacc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (more)                                                    // (the last product has read its fragment: K is out of LDS)
            issue(kt + NW, k_rsrc, k_off, lds_base);

        // online softmax, as in the kernel above with the running maximum itself as the reference: a wave walks a few
        // tiles only, so that there is little rescaling to save by one that lags behind, and the largest probability
        // of a wave is not rounded
        if ((kt + 1) * BK > S) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (kt * BK + 8 * (r >> 2) + 4 * lh + (r & 3) >= S)
                    sacc[r] = -INFINITY;
        }
        float mx = sacc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r)
            mx = fmaxf(mx, sacc[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mxs = mx * sl2;
        if (__builtin_amdgcn_ballot_w64(mxs > m_run) != 0) {
            const float m_new = fmaxf(m_run, mxs);
            float alpha = exp2f(m_run - m_new);
            asm volatile("" : "+v"(alpha));
            m_run = m_new;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                lacc[e] *= alpha;
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    oacc[d][e] *= alpha;
        }
        const float nm = -m_run;
        bf16x8_t pf[2];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                pf[s2][e] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sacc[8 * s2 + e], sl2, nm));

        if (more)                                                    // V of tile kt has landed (K of the next may be in flight)
            wait_vmcnt<8>();
        else
            wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                const unsigned char *pv = my + v_addr[d] + s2 * 16 * ROWB;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4_t *)(pv));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4_t *)(pv + 8 * ROWB));
                const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[s2], oacc[d], 0, 0, 0);
            }
            lacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, pf[s2], lacc, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more)
            issue(kt + NW, v_rsrc, v_off, lds_base + TB);
    }

    // Merge: register r of lane L of every wave is the same (query, d) position.
    {
        float *mo = reinterpret_cast<float *>(my);
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float v = oacc[d][e];
                asm volatile("" : "+v"(v));
                mo[(d * 16 + e) * 64 + lane] = v;
            }
        stat[wave][0][lane] = m_run;
        stat[wave][1][lane] = lacc[0];                               // the whole row sum, in both lanes of the query
    }
    __syncthreads();
    float m_all = -INFINITY, l_all = 0.0f, o[8];
#pragma unroll
    for (int w = 0; w < NW; ++w)
        m_all = fmaxf(m_all, stat[w][0][lane]);                      // finite: every workgroup has a tile
#pragma unroll
    for (int e = 0; e < 8; ++e)
        o[e] = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float f = exp2f(stat[w][0][lane] - m_all);             // 0 for a wave that saw no key
        l_all += stat[w][1][lane] * f;
        const float *mo = reinterpret_cast<const float *>(smem + w * WAVE_LDS);
#pragma unroll
        for (int e = 0; e < 8; ++e)                                  // this thread: registers 8 wave .. + 7 of lane
            o[e] += mo[(wave * 8 + e) * 64 + lane] * f;
    }
    if (KSP > 1) {                                                   // hand-over between workgroups, as in the kernel above
        constexpr int COHERENT = 1 | 16;
        auto part_rsrc = [&](int sp) {
            return __builtin_amdgcn_make_buffer_rsrc(P.ws + ((size_t)group * KSP + sp) * KW_PART, 0, KW_PART * 4, 0x00020000);
        };
        __amdgpu_buffer_rsrc_t rs = part_rsrc(split);
        const f32x4_t o0 = {o[0], o[1], o[2], o[3]}, o1 = {o[4], o[5], o[6], o[7]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o0), rs, tid * 32, 0, COHERENT);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o1), rs, tid * 32 + 16, 0, COHERENT);
        if (wave == 0) {
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, m_all), rs, (4096 + lane) * 4, 0, COHERENT);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, l_all), rs, (4096 + 64 + lane) * 4, 0, COHERENT);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        unsigned *arrived = reinterpret_cast<unsigned *>(smem);
        if (tid == 0)
            *arrived = __hip_atomic_fetch_add(&P.counters[group], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*arrived != (unsigned)(KSP - 1))
            return;
        if (tid == 0)
            __hip_atomic_store(&P.counters[group], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // Bound by the trips to memory: four splits per trip, maxima and sums at once (one by one the maxima of three splits alone
        // were three trips), beyond the last the last once more, unused.  us of four to eight slices with their projections, before /
        // now, the same bits: 4 slices of 2 x 3 heads x 1120 keys 87.7 / 85.2, 8 of one head x 808 114 / 108, of two x 4712 211 / 202.
        constexpr int AT = 4;
        float m[AT], l[AT];
        f32x4_t a[AT], c[AT];
        auto request = [&](int sp0) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < AT; ++i) {
                __amdgpu_buffer_rsrc_t rp = part_rsrc(sp0 + i < KSP ? sp0 + i : KSP - 1);
                m[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rp, (4096 + lane) * 4, 0, COHERENT));
                l[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rp, (4096 + 64 + lane) * 4, 0, COHERENT));
                a[i] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rp, tid * 32, 0, COHERENT));
                c[i] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rp, tid * 32 + 16, 0, COHERENT));
            }
        };
        m_all = -INFINITY;
        if (KSP > AT) {
            for (int sp0 = AT; sp0 < KSP; sp0 += AT) {
                float mm[AT];
#pragma unroll
                for (int i = 0; i < AT; ++i)
                    mm[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(part_rsrc(sp0 + i < KSP ? sp0 + i : KSP - 1),
                                                                                           (4096 + lane) * 4, 0, COHERENT));
#pragma unroll
                for (int i = 0; i < AT; ++i)
                    m_all = fmaxf(m_all, mm[i]);
            }
        }
        request(0);
#pragma unroll
        for (int i = 0; i < AT; ++i)
            m_all = fmaxf(m_all, m[i]);
        l_all = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            o[e] = 0.0f;
        for (int sp0 = 0;;) {
#pragma unroll
            for (int i = 0; i < AT; ++i) {
                if (sp0 + i >= KSP)
                    break;
                const float f = exp2f(m[i] - m_all);
                l_all += l[i] * f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[e] += a[i][e] * f;
                    o[4 + e] += c[i][e] * f;
                }
            }
            if ((sp0 += AT) >= KSP)
                break;
            request(sp0);
        }
    }
    if (q_ok) {
        const float inv = 1.0f / l_all;
        // registers 8 wave .. + 7: d tile wave / 2, registers 8 (wave & 1) .. + 7 of it
        __bf16 *orow = static_cast<__bf16 *>(P.out) + (size_t)(slice - P.l) * P.out_slice_stride + ((size_t)b * P.c + qi) * P.ldo +
                       (size_t)head * DH + (wave >> 1) * 32 + (wave & 1) * 16 + 4 * lh;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            bf16x4_t h;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                h[e] = (__bf16)(o[4 * g + e] * inv);
            *reinterpret_cast<u32x2_t *>(orow + 8 * g) = __builtin_bit_cast(u32x2_t, h);
        }
    }
}

}  // namespace

bool attn_slice_supported(const AttnParams &p)
{
    return p.head_dim == DH && p.S > 0 && p.c > 0 && p.heads > 0 && p.batch > 0 &&
           (int64_t)p.S * DH * 2 < ((int64_t)1 << 31);
}

namespace {

// Which kernel, and over how many workgroups the keys of a query block are split.  The costs (us) are fitted to
// measurements over batch x heads x queries of the slice x keys:
//   * keys over waves (32 queries): 6.5 + 1.7 per eight 32-key tiles and round + 5 per further full round -- each workgroup reads all its keys
//     itself, 128 KiB per step of its eight waves, 0.9 us at the L1's rate.  2x3x280x1120: 13.5 (query blocks: 20.5 at best,
//     40 with one workgroup per compute unit, whose sixteen partials per block took most of it), 1x1x1024x8192: 21.5 with
//     six splits (37.6), 1x8x1024x8192: 60.1 (57.9);
//   * query blocks, eight waves (256 queries): 7 + 1.83 per 64-key tile and round, 1.33 in a round that leaves a third of the
//     chip idle.  4x8x4096x4096: 245, 2x8x2319x4638: 106 unsplit (keys over waves: 169);
//   * query blocks, four waves (128 queries): 7 + 1.04 per tile, 0.92 where a third of the chip idles, 1.95 with two workgroups
//     per compute unit, 1.65 with fewer than one and a half.  4x4x2048x2048: 41 (eight waves: 51), 1x8x1024x8192 with eight splits 53.6
//     (63.8), 2x8x2319x4638 with two 120 (144).
// A split costs its hand-over: 1.5 + 0.7 per workgroup of 16.5 KiB partials, 3 + 3 for the query blocks' 132 KiB, 1 + 2 for 66.
// The kernels round alike but not equally well, and a choice made for its time must not cost precision.  Query blocks keep a
// softmax reference that lags behind the maximum, so that even the largest probability of a row is rounded; every split of
// the keys starts a reference of its own.  Keys over waves keep the maximum itself, one per wave.  Error against 64 bits
// (2-norm, scores of sigma 4; the output's rounding alone is 1.66e-3): 2x8x2319x4638 keys over waves 1.68e-3, query blocks
// with two splits 1.87e-3, unsplit 1.89e-3; 4x2x1181x2362: 1.68e-3, seven splits 1.79e-3, three 1.84e-3.  So where query
// blocks of 256 leave a quarter of the chip idle, query blocks are a choice only with the keys split finely enough for a
// workgroup per compute unit (k0 splits); where no workspace takes the partials of that, a single slice has none.  And a faster
// loop of the query blocks does not move the line between the kernels: they are a choice where a loop without the pipeline would
// win (2.05 per tile, 1.65 in a round that leaves a third of the chip idle; four waves 1.38 and 2.1; a split 5 + 1.5), with at
// least as many splits as that loop would take -- 4x2x1181x2362 stays with keys over waves (40), four waves and three splits 25.6.
struct AttnChoice {
    int waves = 8;               // 0: keys over waves
    int ksplit = 1;
};

AttnChoice choose_attn(const AttnParams &p, int num_cu)
{
    const int64_t heads = (int64_t)p.heads * p.batch * p.n_slices;
    const int tiles32 = (p.S + 31) / 32, tiles64 = (p.S + 63) / 64;
    const bool can_split = p.ws != nullptr && p.counters != nullptr;
    const int64_t blocks = (p.c + 255) / 256 * heads;
    int k0 = 1;
    bool query_blocks = true;
    if (blocks * 4 < (int64_t)num_cu * 3) {
        int64_t k = (num_cu + blocks - 1) / blocks;
        k = k > 16 ? 16 : k;
        k = k > tiles64 ? tiles64 : k;
        if (can_split && k > 1 && blocks <= p.max_groups &&
            (size_t)(blocks * k) * (size_t)(64 + 2) * (64 * 8) * sizeof(float) <= p.ws_bytes)
            k0 = (int)k;
        else
            query_blocks = p.n_slices > 1;
    }
    // the cheapest of the candidates; query blocks with `least` splits or more (0: not at all), priced with or without the pipeline
    auto cheapest = [&](int least, bool piped) {
        AttnChoice best;
        double best_us = 0.0;
        for (int kind = 0; kind < 3; ++kind) {               // keys over waves, eight waves, four waves
            if (kind != 0 && least == 0)
                break;
            const int waves = kind == 0 ? 0 : kind == 1 ? 8 : 4;
            const int bq = kind == 0 ? 32 : 32 * waves;
            const int64_t groups = (p.c + bq - 1) / bq * heads;
            for (const int k : {1, 2, 3, 4, 6, 8, 12, k0}) {
                if (kind != 0 && k < least)
                    continue;
                const size_t part = kind == 0 ? (size_t)KW_PART : (size_t)(64 + 2) * (64 * waves);
                if (k > 1 && (!can_split || groups > p.max_groups || (groups * k > num_cu && (kind == 0 || k != least)) || k > (kind == 0 ? tiles32 : tiles64) ||
                              (size_t)groups * k * part * sizeof(float) > p.ws_bytes))
                    continue;
                const int64_t wgs = groups * k;
                const int64_t last = wgs % num_cu;
                const double whole = (double)(wgs / num_cu);
                const bool idle = last * 3 <= num_cu * 2;    // ... a third of the chip in the last round
                double us;
                if (kind == 0) {
                    const double rounds = (double)((wgs + num_cu - 1) / num_cu);
                    us = 6.5 + rounds * (((tiles32 + k - 1) / k + 7) / 8) * 1.7 + (wgs > num_cu ? 5.0 * (wgs - num_cu) / num_cu : 0.0) +
                         (k > 1 ? 1.5 + 0.7 * k : 0.0);
                } else {
                    const int64_t pairs = (wgs + 2 * num_cu - 1) / (2 * num_cu);
                    const double tile = kind == 1 ? (piped ? whole * 1.83 + (last == 0 ? 0.0 : idle ? 1.33 : 1.83)
                                                           : whole * 2.05 + (last == 0 ? 0.0 : idle ? 1.65 : 2.05))
                                        : wgs <= num_cu ? (piped ? (wgs * 3 <= num_cu * 2 ? 0.92 : 1.04) : 1.38)
                                                        : pairs * (piped ? (wgs * 2 <= num_cu * 3 ? 1.65 : 1.95) : 2.1);
                    const double split = kind == 1 ? 3.0 + 3.0 * k : 1.0 + 2.0 * k;
                    us = 7.0 + ((tiles64 + k - 1) / k) * tile + (k == 1 ? 0.0 : piped ? split : 5.0 + 1.5 * k);
                }
                if (best_us == 0.0 || us < best_us) {
                    best_us = us;
                    best.waves = waves;
                    best.ksplit = k;
                }
            }
        }
        return best;
    };
    const AttnChoice line = cheapest(query_blocks ? k0 : 0, false);
    return line.waves == 0 ? line : cheapest(line.ksplit, true);
}

}  // namespace

hipError_t launch_attn_slice(const AttnParams &p_in, hipStream_t s, int num_cu)
{
    AttnParams p = p_in;
    if (p.n_slices < 1)
        p.n_slices = 1;
    AttnChoice t = choose_attn(p, num_cu);
    const Tuning tn = tuning();                          // overrides
    if (tn.attn_qt >= 0 || tn.attn_waves || tn.attn_ksplit) {
        t.waves = tn.attn_qt == 0 ? 0 : tn.attn_qt == 2 ? 4 : tn.attn_waves ? tn.attn_waves : 8;   // 0: keys over waves; 1, 2: query blocks of 256, 128
        t.ksplit = tn.attn_ksplit ? tn.attn_ksplit : 1;      // workgroups per query block
    }
    const bool keys_over_waves = t.waves == 0;
    const int bq = keys_over_waves ? 32 : t.waves * 32;
    const int64_t groups = (int64_t)((p.c + bq - 1) / bq) * p.heads * p.batch * p.n_slices;
    const int tiles = keys_over_waves ? (p.S + 31) / 32 : (p.S + BKV - 1) / BKV;
    p.ksplit = t.ksplit < tiles ? t.ksplit : tiles;
    const size_t need = (size_t)groups * p.ksplit * (keys_over_waves ? (size_t)KW_PART : (size_t)(64 + 2) * (64 * t.waves)) * sizeof(float);
    if (p.ksplit > 1 && (p.ws == nullptr || p.counters == nullptr || need > p.ws_bytes || groups > p.max_groups))
        p.ksplit = 1;
    if (groups * p.ksplit >= ((int64_t)1 << 31))
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)(groups * p.ksplit)), block(64 * (keys_over_waves ? KW_WAVES : t.waves));
    if (keys_over_waves)
        hipLaunchKernelGGL(attn_keys_over_waves_kernel, grid, block, 0, s, p);
    else if (t.waves == 8)
        hipLaunchKernelGGL((attn_slice_kernel<8>), grid, block, 0, s, p);
    else
        hipLaunchKernelGGL((attn_slice_kernel<4>), grid, block, 0, s, p);
    return hipGetLastError();
}

}  // namespace cf
