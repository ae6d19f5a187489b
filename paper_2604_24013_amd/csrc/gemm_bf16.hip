// bf16 x bf16 -> fp32 chunk GEMM for gfx950 with the fused epilogue of the
// reduce-scatter step (Alg. 2: "O <- B_in + O", then "B_out <- O") or the plain
// in-place slice store of the all-gather step (Alg. 1: "O_s[l] <- ...").
//
// Design (CDNA4):
//  * v_mfma_f32_32x32x16_bf16, 64-wide wavefronts.  The MFMA "A" operand is fed
//    from the weight tile and the "B" operand from the activation tile, so a
//    lane's four consecutive accumulator registers are four consecutive output
//    columns of one output row: the epilogue moves 16-byte vectors.
//  * Workgroup tile BM x BN x 64, LDS double-buffered (two stages of
//    (BM+BN) x 64 bf16); the next k-tile is fetched from global memory into
//    registers while the current one is multiplied, then written to the other
//    stage: one barrier per k-tile.
//  * Both operand tiles sit in LDS with k contiguous (128-byte rows of eight
//    16-byte chunks) under an XOR swizzle that makes the 16-byte fragment reads,
//    the straight tile writes and the transposing writes of a [k x n] weight
//    tile all free of bank conflicts.
//  * A [k x n] weight tile (n contiguous in memory) is transposed in registers
//    (8x8 blocks of 16-bit values) on its way to LDS.
//  * Workgroup ids are remapped so that each XCD (own L2) works on a contiguous
//    band of tiles that share operand rows / columns.
#include "cf_internal.h"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

namespace cf {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int BK = 64;          // k extent of one LDS stage
constexpr int ROW_BYTES = 128;  // BK * sizeof(bf16)

// Byte offset of 16-byte chunk kc (0..7) of tile row `row` inside an operand tile.
__device__ __forceinline__ int lds_swz(int row, int kc)
{
    const int r0 = row & 1, r1 = (row >> 1) & 1, r2 = (row >> 2) & 1;
    const int r3 = (row >> 3) & 1, r4 = (row >> 4) & 1, r5 = (row >> 5) & 1;
    const int half = r0 ^ r3;
    const int kcp = kc ^ (((r1 ^ r4) << 2) | ((r2 ^ r5) << 1) | r3);
    return ((row >> 1) << 8) + (half << 7) + (kcp << 4);
}

// Tile of R rows x 64 k, source rows are k-contiguous in memory.
template <int R, int NT>
struct StraightLoader {
    static constexpr int CH = (R * 8) / NT;
    static_assert(CH >= 1 && (R * 8) % NT == 0, "tile rows vs threads");
    uint4 v[CH];

    __device__ __forceinline__ void load(const __bf16 *base, int64_t ld, int row0, int rows_total,
                                         int k0, int K, int tid)
    {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int c = tid + j * NT;
            const int row = c >> 3, kc = c & 7;
            const int grow = row0 + row, gk = k0 + kc * 8;
            uint4 x = make_uint4(0u, 0u, 0u, 0u);
            if (grow < rows_total && gk < K)
                x = *reinterpret_cast<const uint4 *>(base + (int64_t)grow * ld + gk);
            v[j] = x;
        }
    }
    __device__ __forceinline__ void store(unsigned char *lds, int tid) const
    {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int c = tid + j * NT;
            *reinterpret_cast<uint4 *>(lds + lds_swz(c >> 3, c & 7)) = v[j];
        }
    }
};

// Tile of 64 k x BN n from a [K x N] matrix (n contiguous): each of the first BN
// threads owns one 8(k) x 8(n) block, transposes it in registers and writes
// eight 16-byte k-runs.
template <int BN_, int NT>
struct TransposeLoader {
    static_assert(BN_ <= NT, "one 8x8 block per thread");
    uint4 v[8];

    __device__ __forceinline__ void load(const __bf16 *W, int64_t ldw, int n0, int N, int k0, int K, int tid)
    {
        if (tid < BN_) {
            const int kb = (tid >> 3) & 7;
            const int ncb = ((tid >> 6) << 3) + (tid & 7);
            const int gn = n0 + ncb * 8;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int gk = k0 + kb * 8 + j;
                uint4 x = make_uint4(0u, 0u, 0u, 0u);
                if (gk < K && gn < N)
                    x = *reinterpret_cast<const uint4 *>(W + (int64_t)gk * ldw + gn);
                v[j] = x;
            }
        }
    }
    __device__ __forceinline__ void store(unsigned char *lds, int tid) const
    {
        if (tid < BN_) {
            const int kb = (tid >> 3) & 7;
            const int ncb = ((tid >> 6) << 3) + (tid & 7);
            const unsigned in[8][4] = {
                {v[0].x, v[0].y, v[0].z, v[0].w}, {v[1].x, v[1].y, v[1].z, v[1].w},
                {v[2].x, v[2].y, v[2].z, v[2].w}, {v[3].x, v[3].y, v[3].z, v[3].w},
                {v[4].x, v[4].y, v[4].z, v[4].w}, {v[5].x, v[5].y, v[5].z, v[5].w},
                {v[6].x, v[6].y, v[6].z, v[6].w}, {v[7].x, v[7].y, v[7].z, v[7].w}};
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                unsigned o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned lo = in[2 * e][n >> 1], hi = in[2 * e + 1][n >> 1];
                    o[e] = (n & 1) ? ((lo >> 16) | (hi & 0xFFFF0000u)) : ((lo & 0xFFFFu) | (hi << 16));
                }
                *reinterpret_cast<uint4 *>(lds + lds_swz(ncb * 8 + n, kb)) = make_uint4(o[0], o[1], o[2], o[3]);
            }
        }
    }
};

// XCD-aware remap: hardware hands consecutive workgroup ids to the 8 XCDs in
// turn; give XCD x the contiguous tile range [start(x), start(x+1)).
__device__ __forceinline__ int xcd_remap(int pid, int total)
{
    constexpr int NXCD = 8;
    const int q = total / NXCD, rem = total % NXCD;
    const int xcd = pid % NXCD, idx = pid / NXCD;
    return xcd * q + (xcd < rem ? xcd : rem) + idx;
}

template <int BM, int BN, int WGM, int WGN, bool W_KN, bool OUT_BF16>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_kernel(GemmParams P, int tiles_m, int tiles_n)
{
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be a multiple of the MFMA tile");
    constexpr int A_BYTES = BM * ROW_BYTES, B_BYTES = BN * ROW_BYTES, STAGE = A_BYTES + B_BYTES;

    __shared__ __attribute__((aligned(256))) unsigned char smem[2 * STAGE];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WGM, wn = wave / WGM;

    const int tile = xcd_remap(blockIdx.x, tiles_m * tiles_n);
    const int m0 = (tile % tiles_m) * BM;      // M fastest: a band shares weight columns
    const int n0 = (tile / tiles_m) * BN;

    const __bf16 *A = static_cast<const __bf16 *>(P.A);
    const __bf16 *W = static_cast<const __bf16 *>(P.W);
    const int M = P.M, N = P.N, K = P.K;

    StraightLoader<BM, NT> la;
    StraightLoader<BN, NT> lw_nk;
    TransposeLoader<BN, NT> lw_kn;

    auto load_tiles = [&](int k0) {
        la.load(A, P.lda, m0, M, k0, K, tid);
        if constexpr (W_KN)
            lw_kn.load(W, P.ldw, n0, N, k0, K, tid);
        else
            lw_nk.load(W, P.ldw, n0, N, k0, K, tid);
    };
    auto store_tiles = [&](int stage) {
        unsigned char *sa = smem + stage * STAGE;
        la.store(sa, tid);
        if constexpr (W_KN)
            lw_kn.store(sa + A_BYTES, tid);
        else
            lw_nk.store(sa + A_BYTES, tid);
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                acc[i][j][e] = 0.0f;

    const int nk = (K + BK - 1) / BK;
    const int frow = lane & 31, fkc = lane >> 5;

    if (nk > 0) {
        load_tiles(0);
        store_tiles(0);
    }
    __syncthreads();

    for (int kt = 0; kt < nk; ++kt) {
        const bool more = (kt + 1) < nk;
        if (more)
            load_tiles((kt + 1) * BK);

        const unsigned char *sa = smem + (kt & 1) * STAGE;
        const unsigned char *sb = sa + A_BYTES;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            bf16x8_t af[TM], wf[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[i] = *reinterpret_cast<const bf16x8_t *>(sa + lds_swz(wm * WTM + i * 32 + frow, ks * 2 + fkc));
#pragma unroll
            for (int j = 0; j < TN; ++j)
                wf[j] = *reinterpret_cast<const bf16x8_t *>(sb + lds_swz(wn * WTN + j * 32 + frow, ks * 2 + fkc));
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[j], af[i], acc[i][j], 0, 0, 0);
        }

        if (more)
            store_tiles((kt + 1) & 1);
        __syncthreads();
    }

    // Epilogue.  Accumulator register 4g+e of lane L holds
    //   row m = tile row (L & 31), column n = 8g + 4(L >> 5) + e   of the 32x32 tile.
    const float *recv = P.recv;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * WTM + i * 32 + (lane & 31);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + wn * WTN + j * 32 + g * 8 + (lane >> 5) * 4;
                if (m < M && n < N) {
                    f32x4_t o;
                    o[0] = acc[i][j][4 * g + 0];
                    o[1] = acc[i][j][4 * g + 1];
                    o[2] = acc[i][j][4 * g + 2];
                    o[3] = acc[i][j][4 * g + 3];
                    const int64_t off = (int64_t)m * P.ldo + n;
                    if (recv != nullptr) {
                        const f32x4_t r = *reinterpret_cast<const f32x4_t *>(recv + off);
                        o = r + o;                       // "O <- B_in + O"
                    }
                    if constexpr (OUT_BF16) {
                        bf16x4_t h;
                        h[0] = static_cast<__bf16>(o[0]);
                        h[1] = static_cast<__bf16>(o[1]);
                        h[2] = static_cast<__bf16>(o[2]);
                        h[3] = static_cast<__bf16>(o[3]);
                        *reinterpret_cast<bf16x4_t *>(static_cast<__bf16 *>(P.out) + off) = h;
                    } else {
                        *reinterpret_cast<f32x4_t *>(static_cast<float *>(P.out) + off) = o;
                    }
                }
            }
        }
    }
}

template <int BM, int BN, int WGM, int WGN>
hipError_t launch_cfg(const GemmParams &p, bool w_kn, bool out_bf16, hipStream_t s)
{
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    const dim3 grid(tiles_m * tiles_n), block(64 * WGM * WGN);
    if (w_kn) {
        if (out_bf16)
            hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WGM, WGN, true, true>), grid, block, 0, s, p, tiles_m, tiles_n);
        else
            hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WGM, WGN, true, false>), grid, block, 0, s, p, tiles_m, tiles_n);
    } else {
        if (out_bf16)
            hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WGM, WGN, false, true>), grid, block, 0, s, p, tiles_m, tiles_n);
        else
            hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WGM, WGN, false, false>), grid, block, 0, s, p, tiles_m, tiles_n);
    }
    return hipGetLastError();
}

}  // namespace

// What the main loop and the hand-over of a k range split over ks workgroups per 128x128 tile take, in microseconds: a round,
// the k-tiles of a split and what all of them together ask of the caches, and the partial tiles (64 KiB each) there and back.
// Weight gradients have lines of their own: a whole range that is short is cheaper there (two 128x128 workgroups to a compute unit
// up to sixteen k-tiles) than the splits' line says at one, and splits cost more on the last fifth of the chip.
static double bf16_split_us(int tiles, int ktiles, int ks, int num_cu, bool a_t)
{
    const double per = (ktiles + ks - 1) / ks, share = (double)tiles * ks / num_cu;
    if (a_t && ks == 1)
        return 3.9 + 0.42 * per + (6.7 - 0.05 * per) * share;
    if (a_t)
        return 7.0 + 0.37 * per + (2.6 + 0.15 * per) * share + 0.54 * ks + (share > 0.8 ? 4.0 * (share - 0.8) : 0.0);
    return 4.5 + 0.34 * per + 0.23 * per * share + (ks > 1 ? 1.1 + 0.55 * ks + 0.011 * tiles * ks : 0.0);
}

TileChoice choose_tile_bf16(int M, int N, int K, int num_cu, int parts, bool a_t)
{
    // Measured on MI355X: the kernels are bound by the rate at which a CU can pull operand tiles
    // through its L1 (64 B/clk), so the largest tile that still fills the chip wins; a grid of at
    // most one 128x128 workgroup per CU runs best with four LDS stages, and when even that leaves
    // most CUs idle the k range is split (if the caller registered a workspace).
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int want = (num_cu * 7) / 8;
    TileChoice t{128, 128, 1};
    if (tiles(256, 256) >= want) return TileChoice{256, 256, 1};
    if (tiles(256, 128) >= want) return TileChoice{256, 128, 1};
    const int t128 = tiles(128, 128);
    if (t128 > num_cu) return t;                 // two workgroups per CU, two stages each
    // A grid of one workgroup per compute unit and less: the number of splits with the lowest estimate (us of a launch; fitted to 590
    // weight gradients of 512..8192 rows into 64..4096 x 64..4096, each whole and in 2 to 8 splits, rms 0.03 beside 1.4 us and more for a
    // B_in, which all of them pay; steps to a line of 229 earlier ones, rms 0.06).  us whole / as chosen: 552 x 536 over 5768 rows 43.7 /
    // 20.2 (in seven), 520 x 856 over 2544 in four 22.3 / 15.6, 776 x 1368 over 912 11.9 (whole; in two 13.4), 136 x 152 over 848 9.6 (whole;
    // in three 11.0), 1168 x 296 over 1232 in three 13.8 / 12.9, 248 x 120 over 1472 in four 13.4 / 11.7.  Of the 590 one is 5 % and more
    // behind the best, 0.3 % on average; by the steps' line 20 and 0.7 %.
    // Of the splits whose partial tiles the workspace takes: with room for 8 k n floats 144 x 640 over 7000 rows runs in four (in eight
    // with more room, 18.0 us) 20.8, 296 x 584 over 7752 in five (in eight 20.2) 21.7; left whole they take 47 and 56.
    t.deep = true;
    const int ktiles = (K + 63) / 64;
    double best = 0.0;
    for (int ks = 1; ks <= 8 && (ks == 1 || t128 * ks <= parts) && ktiles >= 2 * ks; ++ks) {
        const double us = bf16_split_us(t128, ktiles, ks, num_cu, a_t);
        if (ks == 1 || us < best) {
            best = us;
            t.splitk = ks;
        }
    }
    return t;
}

static bool staged_kernel_forced()                   // "staged": the register-staged kernel of this file
{
    return tuning().staged != 0;
}

bool gemm_bf16_takes_recv_list(const GemmParams &p, bool w_kn)
{
    return p.M > 0 && p.N > 0 && !staged_kernel_forced() && gemm_bf16_dl_supported(p, w_kn);
}

// Tile of a launch by area: the per-step choice, or the persistent rank step's cost model.
static TileChoice tile_by_area(const GemmParams &p, int num_cu)
{
    const size_t parts = p.ws == nullptr || p.counters == nullptr ? 0 : p.ws_bytes / (128 * 128 * sizeof(float));
    TileChoice t = choose_tile_bf16(p.M, p.N, p.K, num_cu, parts < (size_t)num_cu ? (int)parts : num_cu, p.a_t);
    if (p.n_steps > 0) {
        // Persistent rank step: n_steps * tiles work items share one grid, so a step need not fill the chip
        // alone.  Cost of a tile shape = rounds over the chip x tile area x its measured cost per flop
        // (per-k-tile time of a full grid: 256x256 1.00, 256x128 1.15, 128x128 1.30, relative).
        const struct { int bm, bn; double cost; } cand[3] = {{256, 256, 1.00}, {256, 128, 1.15}, {128, 128, 1.30}};
        double best = 0.0;
        for (int c = 0; c < 3; ++c) {
            const int64_t items = (int64_t)((p.M + cand[c].bm - 1) / cand[c].bm) * ((p.N + cand[c].bn - 1) / cand[c].bn) * p.n_steps;
            const int64_t rounds = (items + num_cu - 1) / num_cu;
            const double cost = (double)rounds * cand[c].bm * cand[c].bn * cand[c].cost;
            if (c == 0 || cost < best) {
                best = cost;
                t.bm = cand[c].bm;
                t.bn = cand[c].bn;
            }
        }
        t.splitk = 1;
        t.deep = true;                               // 128x128: one workgroup per CU, four stages
    }
    return t;
}

double gemm_share_with_recv(const GemmParams &p)
{
    if (p.n_steps <= 0)
        return p.recv != nullptr ? 1.0 : 0.0;
    int n = 0;
    for (int j = 0; j < p.n_steps; ++j)
        n += p.recv_step[j] != nullptr;
    return (double)n / p.n_steps;
}

// What a launch takes with tile t, in microseconds: per work item and k-tile, R rounds over the chip, and less where the last
// round leaves compute units idle (the others' operands come faster), plus the megabytes of fp32 output, of the left operand
// and what goes with a B_in, which the share r of the steps has.  Fitted (relative error, rms 0.07 to 0.13) to 3200 steps and carried rank steps of 16..8192 rows x
// 128..8192 x 128..8192 on each tile, on buffers that come round and on ones cold in the caches; for weight gradients, whose left
// operand is read by k-rows, to 90 of 32..8192 rows into 256..8192 x 256..8192 (rms 0.04 to 0.12).
static double tile_estimate_us(const GemmParams &p, TileChoice t, int num_cu, double r)
{
    const int steps = p.n_steps > 0 ? p.n_steps : 1;
    const int64_t items = (int64_t)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn) * steps;
    const double kt = (p.K + 63) / 64, mb = (double)p.M * p.N * steps * 4e-6;
    const bool two = t.bm == 128 && !t.deep;
    const int64_t wgs = (int64_t)num_cu * (two ? 2 : 1);
    const double share = (double)items / wgs, rounds = (double)((items + wgs - 1) / wgs);
    if (p.a_t) {
        if (t.bm == 256 && t.bn == 256)
            return 1.8 + rounds * (6.2 + 0.88 * kt) + 0.59 * kt * share + 0.083 * mb;
        if (t.bm == 256)
            return 2.5 + rounds * (3.9 + 0.46 * kt) + 0.455 * kt * share + 0.071 * mb;
        if (two)
            return 3.4 + rounds * (1.7 + 0.35 * kt) + 0.725 * kt * share + 0.095 * mb;
        return 2.3 + rounds * (4.3 + 0.31 * kt) + 0.27 * kt * share;
    }
    const double ma = (double)p.M * p.K * steps * 2e-6;
    if (t.bm == 256 && t.bn == 256)
        return 0.6 + rounds * (6.4 + 0.98 * kt + 3.8 * r) + 0.24 * kt * share + (0.11 + 0.3 * r) * mb + 0.14 * ma;
    if (t.bm == 256)
        return 1.5 + rounds * (3.8 + 0.56 * kt + 1.8 * r) + 0.17 * kt * share + (0.098 + 0.17 * r) * mb + 0.22 * ma;
    if (two)
        return 2.1 + (double)((items + num_cu - 1) / num_cu) * (2.1 + 0.12 * kt) + rounds * (0.4 * kt + 0.87 * r) + 0.34 * kt * share +
               (0.022 + 0.23 * r) * mb + 0.07 * ma;
    return 2.0 + rounds * (3.6 + 0.36 * kt + 1.2 * r) + 0.14 * kt * share + (0.038 + 0.13 * r) * mb + 0.1 * ma;
}

// The overrides: tile shape, stages, k-splits per output tile.
static TileChoice with_overrides(TileChoice t)
{
    const Tuning tn = tuning();
    if (tn.tile_bm > 0) {
        t.bm = tn.tile_bm;
        t.bn = tn.tile_bn;
    }
    if (tn.deep >= 0)
        t.deep = tn.deep != 0;
    if (tn.splitk >= 1)
        t.splitk = tn.splitk;
    return t;
}

// Tile of a launch before the overrides: the one whose estimate is lowest, unless the one by area splits the k range.  256x256 by
// area changes for an estimate 5 % lower only, for one 10 % lower where the tiles are whole (the 16x16x32 main loop): there it is
// loosest.  us on 256x256 / 256x128, all-gather step 8192 x 3072 x 1024 59 / 75, reduce-scatter steps 2048 x 8192 x 1024 53 / 59,
// 8192 x 8192 x 1024 234 / 273, 4096 x 6144 x 1024 83 / 73, 2560 x 8192 x 4096 197 / 178.  Of 3200 launches drawn from the sizes
// above the tile so chosen is 0.6 % behind the fastest on average and 10 % and more behind in 20; by area alone 4.4 % and 540, by
// an estimate that knew neither B_in nor left operand, fitted to 1024 rows at most, 1.5 % and 85.  Weight gradients change for an
// estimate 7 % lower: 1928 rows into 1608 x 4712, 256x128 53.6, two 128x128 per compute unit 38.2.
static TileChoice tile_by_estimate(const GemmParams &p, int num_cu, double *t_us = nullptr)
{
    TileChoice t = tile_by_area(p, num_cu);
    if (t.splitk == 1) {
        static const TileChoice cand[4] = {{256, 256, 1}, {256, 128, 1}, {128, 128, 1, true}, {128, 128, 1}};
        const bool large = t.bm == 256 && t.bn == 256, whole = p.M % 256 == 0 && p.N % 256 == 0;
        const double r = gemm_share_with_recv(p), area_us = tile_estimate_us(p, t, num_cu, r);
        double best = (p.a_t ? 0.93 : large ? (whole ? 0.9 : 0.95) : 1.0) * area_us, its_us = area_us;
        for (const TileChoice &c : cand) {
            const double us = tile_estimate_us(p, c, num_cu, r);
            if (us < best) {
                best = its_us = us;
                t = c;
            }
        }
        if (t_us != nullptr)
            *t_us = its_us;
    }
    return t;
}

static TileChoice tile_of_launch(const GemmParams &p, int num_cu)
{
    const Tuning tn = tuning();
    return with_overrides(tn.tile_bm == 0 && tn.deep < 0 ? tile_by_estimate(p, num_cu) : tile_by_area(p, num_cu));
}

double gemm_bf16_rank_step_us(const GemmParams &p, int num_cu)
{
    double us = 0.0;
    tile_by_estimate(p, num_cu, &us);                // (a rank step's k range is not split)
    // an all-gather that cannot carry its deliveries has them copied in front: 6 us, and 0.8 us per megabyte of them
    return gemm_share_with_recv(p) == 0.0 && !gemm_bf16_dl_carries_operand(p) ? us + 6.0 : us;
}

double gemm_bf16_tile_us(const GemmParams &p, int num_cu)
{
    const TileChoice t = tile_by_area(p, num_cu);
    const int64_t tiles = (int64_t)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn);
    if (p.n_steps > 0) {                             // rank steps over k ranges that tile_estimate_us has not seen
        const int64_t items = tiles * p.n_steps, wgs = (int64_t)num_cu * (t.bm == 128 && !t.deep ? 2 : 1);
        const double kt = (p.K + 63) / 64;
        const double round = t.bm == 128 ? 8 + 0.55 * kt : t.bn == 128 ? 14 + 0.97 * kt : 14 + 1.5 * kt;
        return (double)((items + wgs - 1) / wgs) * round;
    }
    double us = 0.0;
    if (t.splitk > 1) {
        // a step whose k range the launcher splits through the workspace: fitted to 759 steps of 64..1024 x 128..8192 x 512..8192
        // with a B_in, split in 1 to 8 (rms 0.08): 213 x 3496 x 6448 in four 28 us (the few-rows kernel 33), 372 x 4736 x 2184 in two 22
        const double per = ((p.K + 63) / 64 + t.splitk - 1) / t.splitk, all = (double)(tiles * t.splitk);
        us = 7.6 + 0.44 * per + 0.145 * per * all / num_cu + 0.61 * t.splitk + 0.012 * all;
    } else {
        tile_by_estimate(p, num_cu, &us);
        if (choose_tile_bf16(p.M, p.N, p.K, num_cu, num_cu, p.a_t).splitk > 1)   // (no workspace for the splits: 384 x 4096 x 8192 72 us, the few-rows kernel 61)
            us = 1.05 * tile_estimate_us(p, TileChoice{128, 128, 1, true}, num_cu, gemm_share_with_recv(p));
    }
    return us;
}

size_t gemm_bf16_split_ws_bytes(const GemmParams &p_in, bool w_kn, int num_cu)
{
    GemmParams p = p_in;                             // (as it is launched with a workspace)
    p.ws = reinterpret_cast<float *>(16);
    p.counters = reinterpret_cast<unsigned *>(16);
    p.ws_bytes = ~(size_t)0;
    p.max_tiles = 1 << 30;
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || gemm_rows_takes(p, true, w_kn, num_cu))
        return 0;
    const TileChoice t = tile_of_launch(p, num_cu);
    const size_t tiles = (size_t)((p.M + t.bm - 1) / t.bm) * (size_t)((p.N + t.bn - 1) / t.bn);
    return t.splitk > 1 ? tiles * t.splitk * t.bm * t.bn * sizeof(float) : 0;
}

bool gemm_bf16_carries_delivery(const GemmParams &p, bool w_kn, bool out_bf16, int num_cu, bool reduce_scatter)
{
    if (p.M <= 0 || p.N <= 0 || p.n_steps <= 0 || staged_kernel_forced() || !gemm_bf16_dl_supported(p, w_kn))
        return false;
    if (!reduce_scatter && !gemm_bf16_dl_carries_operand(p))
        return false;
    // Partial sums with padding between their rows: every tile could carry them, but a copy in front lands the padding and the
    // epilogue does not, and which of the two a caller finds is part of the interface.  The line is the interface's: 256x256
    // tiles by area (or by override) over 18 k-tiles, 20 with a ragged last one, land without it.
    if (reduce_scatter && p.ldo != p.N) {
        const TileChoice t = with_overrides(tile_by_area(p, num_cu));
        if (t.bm != 256 || t.bn != 256 || (p.K + 63) / 64 < 18 + (p.K % 64 != 0 ? 2 : 0))
            return false;
    }
    // Wherever the launch can, it does (measured against deliveries copied in front of the launch: 7B down-projection rank
    // step 76.6 -> 57 us on warm buffers, attention layer's rank step 520 -> 492 us).
    // COMMFUSE_CARRY=0 keeps the copies in front.
    const Tuning tn = tuning();
    return tn.carry >= 0 ? tn.carry != 0 : true;
}

// A weight gradient carries its deliveries on whole 256x256 tiles with whole k-tiles per block of rows: the loop there has the
// registers, and a k-tile that lies in two neighbours' buffers would need two descriptors per load.  The copy in front moves the
// operand twice and leaves the kernel to read it again; here the launch writes it once.  us of both data and both weight
// gradients, copied / carried, results the same bits: 8 x 1024 x 8192 x 3584 1616 / 1566, 8 x 512 x 8192 x 3584 856 / 838, 8 x 128
// x 8192 x 3584 317 / 306, 8 x 1024 x 5120 x 2560 869 / 823, 8 x 256 x 4096 x 4096 277 / 264; level at 2 x 1024 x 8192 x 3584 (465).
bool gemm_bf16_carries_gathered(const GemmParams &p, int num_cu)
{
    const Tuning tn = tuning();
    if (p.M <= 0 || p.N <= 0 || p.K <= 0 || staged_kernel_forced() || !gemm_bf16_dl_supported(p, true) || tn.carry == 0 || tn.mfma16 == 0)
        return false;
    const TileChoice t = tile_of_launch(p, num_cu);
    return t.bm == 256 && t.bn == 256 && t.splitk <= 1 && gemm_bf16_dl_carries_gathered(p);
}

int gemm_bf16_steps_per_launch(const GemmParams &p, bool w_kn, int num_cu)
{
    if (p.M <= 0 || p.N <= 0 || p.n_steps <= 1 || staged_kernel_forced() || !gemm_bf16_dl_supported(p, w_kn))
        return p.n_steps > 0 ? p.n_steps : 1;
    const TileChoice t = tile_of_launch(p, num_cu);
    const int64_t tiles = (int64_t)((p.M + t.bm - 1) / t.bm) * ((p.N + t.bn - 1) / t.bn);
    const int64_t wgs = (int64_t)num_cu * ((t.bm == 128 && t.bn == 128 && !t.deep) ? 2 : 1);
    int64_t per_round = (wgs + tiles - 1) / tiles;       // steps that fill the chip once (rounded up)
    if (per_round < 1)
        per_round = 1;
    const int64_t launches = (p.n_steps + per_round - 1) / per_round;
    return (int)((p.n_steps + launches - 1) / launches);   // equal groups
}

hipError_t launch_gemm_bf16(const GemmParams &p, bool w_kn, bool out_bf16, hipStream_t s, int num_cu)
{
    if (p.M <= 0 || p.N <= 0)
        return hipSuccess;
    if (gemm_rows_takes(p, true, w_kn, num_cu))
        return launch_gemm_rows(p, true, w_kn, out_bf16, s, num_cu);
    const TileChoice t = tile_of_launch(p, num_cu);
    const bool staged = staged_kernel_forced();
    if (!staged && gemm_bf16_dl_supported(p, w_kn))
        return launch_gemm_bf16_dl(p, w_kn, out_bf16, s, t, num_cu);
    if (p.n_recv_more != 0 || p.a_t || p.n_steps > 0)
        return hipErrorInvalidValue;                 // callers ask gemm_bf16_takes_recv_list first
    if (t.bm == 256 && t.bn == 256) return launch_cfg<256, 256, 2, 4>(p, w_kn, out_bf16, s);
    if (t.bm == 256 && t.bn == 128) return launch_cfg<256, 128, 4, 2>(p, w_kn, out_bf16, s);
    return launch_cfg<128, 128, 2, 2>(p, w_kn, out_bf16, s);
}

}  // namespace cf
