// Internal declarations shared by the translation units of libcommfuse.so.
// Nothing here is part of the C ABI (that is include/commfuse.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace cf {

// One chunk GEMM: out[M x N] = A[M x K] * W (+ recv), fp32 accumulation.
// A points at the first row of the slice; W is [K x N] (w_kn) or [N x K].
// With a_t the left operand is given transposed, as [K x M] with row stride lda (the weight-gradient
// contraction over tokens: both operands then have the contraction index as their row index).
struct GemmParams {
    bool a_t = false;    // direct-to-LDS bf16 kernel, w_kn, fp32 output only
    const void *A = nullptr;
    const void *W = nullptr;
    const float *recv = nullptr;   // nullable: B_in of Alg. 2
    // further received partials, added after `recv` in index order before the product is added
    // (pairwise schedule with the aggregation deferred to the last step; direct-to-LDS bf16 and few-rows kernels)
    static constexpr int MAX_RECV_MORE = 15;
    const float *recv_more[MAX_RECV_MORE] = {};
    int n_recv_more = 0;
    bool k_in_order = false;         // persistent mode: every k loop starts at 0
    void *out = nullptr;
    int64_t lda = 0, ldw = 0, ldo = 0;
    int M = 0, N = 0, K = 0;
    // split-K workspace (direct-to-LDS bf16 kernel only): partial tiles and per-tile arrival counters
    float *ws = nullptr;
    unsigned *counters = nullptr;
    size_t ws_bytes = 0;
    int max_tiles = 0;
    int splits = 1;
    // optional delivery carried by extra workgroups of the same launch (direct-to-LDS bf16 kernel only):
    // cp_bytes (a multiple of 16) from cp_src to cp_dst, both 16-byte aligned, by cp_wgs workgroups
    // optional device-side wait (direct-to-LDS bf16 kernel only): the kernel waits, with a bounded spin,
    // until *wait_flag != 0 before it first touches the delivered buffer (the slice for an all-gather
    // step, B_in for a reduce-scatter step); on time-out it sets bit 0 of *status and carries on
    const unsigned *wait_flag = nullptr;
    unsigned *status = nullptr;
    unsigned spin_limit = 0;
    bool wait_at_start = false;   // true: before the first operand load; false: before the B_in loads
    // persistent mode (direct-to-LDS bf16 kernel only): n_steps > 0 makes one launch run that many chunk GEMMs
    // of the same shape, step s with its own left operand, B_in (nullable as above) and output; A, recv and out are then
    // ignored, and a wait_flag is refused
    static constexpr int MAX_STEPS = 16;
    int n_steps = 0;
    bool k_rotate = false;   // persistent mode: XCD x starts its k loops x/8 of the way into the k range (set by the launcher)
    bool xcd_steps = false;  // persistent mode: XCD x runs steps x, x+8, ... whole (set by the launcher)
    int xcd_bands = 1;       // ... or, > 1: 8 / xcd_bands step groups x xcd_bands bands of tile columns (set by the launcher)
    bool non_temporal = false;   // persistent mode, fp32 output: B_in, its landed copy and the output pass the caches by (set by the launcher)
    bool land_first = false; // persistent mode: every other workgroup lands its deliveries in front of the main loop (set by the launcher)
    bool mfma16 = false;     // persistent mode, 256x256 tile: main loop on v_mfma_f32_16x16x32_bf16 (set by the launcher)
    const void *A_step[MAX_STEPS] = {};
    const float *recv_step[MAX_STEPS] = {};
    void *out_step[MAX_STEPS] = {};
    // the delivery carried by the consumer (persistent launch).  Reduce-scatter: recv_step[s] points at what the
    // neighbour sends (its buffer, not this rank's landing buffer), and the epilogue that adds B_in also stores it to
    // land_step[s], the landing buffer.  All-gather: A_step[s] points at the
    // neighbour's buffer, and every k-tile of the slice that comes in through LDS is stored on to land_step[s]
    // (same layout as A_step[s]) by one of the workgroups that load it.  Either way the emulated transfer happens
    // inside the kernel.  Null = the operand is already where recv_step[s] / A_step[s] points.
    void *land_step[MAX_STEPS] = {};
    const void *cp_src = nullptr;
    void *cp_dst = nullptr;
    size_t cp_bytes = 0;
    int cp_wgs = 0;
    // A weight gradient that carries its deliveries (one step, a_t, whole 256x256 tiles): the rows of one operand come in
    // blocks of hop_tiles k-tiles, block b at A_step[1 + b] -- the address that row 0 of a gathered buffer would have --, and
    // every k-tile but those of block hop_own is stored on to land_step[0], the gathered buffer, by one of the workgroups that
    // load it.  hop_right: it is the right operand that travels.  A (W) points at block 0.
    int hop_tiles = 0, hop_own = 0;
    bool hop_right = false;
    // Few-rows kernel only: where recv_more[i] is stored on to (nullable).  Last on purpose: between recv_more and out it made
    // every single step of the tile kernels with [n x k] weights 0.65 us longer (384 x 4096 x 512: 14.2 -> 14.85 us), with code
    // that differs in nothing but register numbers and the fields' offsets in the kernel argument.
    float *land_more[MAX_RECV_MORE] = {};
};
static_assert(offsetof(GemmParams, out) <= 0xb0 && offsetof(GemmParams, land_more) + sizeof(GemmParams::land_more) == sizeof(GemmParams),
              "what the tile kernels do not read stands behind what they do");

// Attention of one query slice (Alg. 4): out[(b, s) x (head, d)] = softmax(scale * Q_l K^T) V per (b, head).
// Q, K, V are [batch, heads, S, head_dim] bf16, contiguous; out is bf16 with row stride ldo elements.
struct AttnParams {
    const void *Q, *K, *V;
    void *out;
    int batch, heads, S, head_dim;
    int c;               // queries of the slice per batch element (S / N)
    int l;               // slice index: queries [l*c, (l+1)*c)
    int64_t ldo;
    float scale;
    // several slices in one launch: slices l, l+1, ..., l+n_slices-1, the output
    // of slice l+i starting out_slice_stride elements after that of slice l+i-1
    int n_slices = 1;
    int64_t out_slice_stride = 0;
    // key split across workgroups: the key tiles are divided over `ksplit` workgroups per
    // query block, which park (m, l, unnormalised O) in the workspace; the last one to finish merges them
    int ksplit = 1;
    float *ws = nullptr;
    unsigned *counters = nullptr;
    size_t ws_bytes = 0;
    int max_groups = 0;
};

// Tuning overrides (environment variables COMMFUSE_*; tests use them to force every code path).  They are read
// ONCE, at the first call into the library -- unless COMMFUSE_TUNING_LIVE is set to a non-zero value at that
// moment, in which case every call of tuning() reads the environment again (test mode).  A field keeps its
// "unset" value when its variable is absent.  The struct is plain data: it is part of the key under which a
// captured graph is cached, because the choices are baked into the captured launches.
struct Tuning {
    int tile_bm = 0, tile_bn = 0;   // COMMFUSE_TILE = "256x256" | "256x128" | "128x128"   (0 = unset)
    int deep = -1;                  // COMMFUSE_DEEP = 0 | 1                               (-1 = unset)
    int splitk = 0;                 // COMMFUSE_SPLITK = 1..8                              (0 = unset)
    int staged = 0;                 // COMMFUSE_KERNEL = "staged"
    int prefetch = -1;              // COMMFUSE_PREFETCH: any value keeps a launch on the tile kernels (-1 = unset)
    int xcd_steps = -1;             // COMMFUSE_XCD_STEPS = 0 | 1                          (-1 = unset)
    int k_rotate = -1;              // COMMFUSE_K_ROTATE = 0 | 1                           (-1 = unset)
    int xcd_bands = 0;              // COMMFUSE_XCD_BANDS = 1 | 2 | 4: column bands per step group (0 = unset: by shape)
    int stream_recv = -1;           // COMMFUSE_STREAM_RECV: any value keeps a launch on the tile kernels (-1 = unset)
    int mfma16 = -1;                // COMMFUSE_MFMA16 = 0 | 1: 16x16x32 MFMAs in the 256x256 persistent kernel (-1 = unset)
    int persist_wgs = 0;            // COMMFUSE_PERSIST_WGS = cap on the persistent kernel's grid (0 = unset)
    int carry = -1;                 // COMMFUSE_CARRY = 0: a one-launch RS / AG / pairwise RS / weight gradient never carries its
                                    // deliveries under CF_FUSED_COPY (-1 = unset, 1: wherever the launch can)
    int tile_f32_bm = 0;            // COMMFUSE_TILE_F32 = "128x128" | "64x64"             (0 = unset)
    int rows = -1;                  // COMMFUSE_ROWS = 0: never the few-rows kernel            (-1 = unset)
    int rows_mf = 0, rows_nc = 0, rows_ks = 0;   // COMMFUSE_ROWS = "MFxNCxKS": that shape of it (0 = unset)
    unsigned spin_limit = 0;        // COMMFUSE_SPIN_LIMIT                                 (0 = unset)
    int attn_qt = -1;               // COMMFUSE_ATTN_QT = 0 | 1 | 2                        (-1 = unset)
    int attn_waves = 0;             // COMMFUSE_ATTN_WAVES = 4 | 8                         (0 = unset)
    int attn_ksplit = 0;            // COMMFUSE_ATTN_KSPLIT                                (0 = unset)
};
Tuning tuning();

struct TileChoice {
    int bm, bn;          // workgroup tile
    int splitk;          // k-splits per output tile (1 = none)
    bool deep = false;   // 128x128 only: four LDS stages, one workgroup per CU
};

// Chooses the workgroup tile for a chunk GEMM from its shape and the number of
// compute units (the per-step grids are small against 256 CUs); `parts`: how many
// partial 128x128 tiles of a split k range the workspace takes, num_cu at the most;
// `a_t`: a weight gradient.
TileChoice choose_tile_bf16(int M, int N, int K, int num_cu, int parts, bool a_t);

hipError_t launch_gemm_bf16(const GemmParams &p, bool w_kn, bool out_bf16, hipStream_t s, int num_cu);
// True if launch_gemm_bf16 would run the kernel that honours GemmParams::recv_more for these operands.
bool gemm_bf16_takes_recv_list(const GemmParams &p, bool w_kn);
// True if launch_gemm_bf16 would run this persistent launch (reduce_scatter: its steps add a received partial;
// else an all-gather's) on a kernel that honours GemmParams::land_step (the delivery carried by the consumer)
// for every step that receives.
bool gemm_bf16_carries_delivery(const GemmParams &p, bool w_kn, bool out_bf16, int num_cu, bool reduce_scatter);
// The same of a weight gradient (GemmParams::hop_tiles), with the shape and the workspace that it will be launched with.
bool gemm_bf16_carries_gathered(const GemmParams &p, int num_cu);
// Steps per launch when a persistent rank step of p.n_steps steps is cut into launches that fill the chip about once
// each (equal groups; p.n_steps when the whole rank step is one round or less).
int gemm_bf16_steps_per_launch(const GemmParams &p, bool w_kn, int num_cu);
// Direct-to-LDS variant of the bf16 kernel (operand extents below 2^31 bytes).
bool gemm_bf16_dl_supported(const GemmParams &p, bool w_kn);
hipError_t launch_gemm_bf16_dl(const GemmParams &p, bool w_kn, bool out_bf16, hipStream_t s, TileChoice t, int num_cu);
bool gemm_bf16_dl_carries_operand(const GemmParams &p);
bool gemm_bf16_dl_carries_gathered(const GemmParams &p);
// The kernel for few rows (gemm_rows.hip; bf16 and fp32 operands): does it run this launch -- one chunk GEMM, or with
// n_steps > 0 all steps of a rank step, whose deliveries it then carries where land_step / land_more are set?
bool gemm_rows_takes(const GemmParams &p, bool bf16, bool w_kn, int num_cu);
// Share of a launch's (sub-)steps that add a B_in: none of an all-gather's, the last of a pairwise reduce-scatter's.
double gemm_share_with_recv(const GemmParams &p);
// What the tile kernels take for this launch, roughly, in microseconds (for the rule between them and the one above):
// the steps of a rank step in one launch, and single steps.
double gemm_bf16_rank_step_us(const GemmParams &p, int num_cu);
double gemm_bf16_tile_us(const GemmParams &p, int num_cu);
double gemm_f32_tile_us(const GemmParams &p, int num_cu);
// Bytes of partial tiles that kernel parks when it splits the k range of this single step (0: it does not).
size_t gemm_rows_ws_bytes(const GemmParams &p, bool bf16, bool w_kn, int num_cu);
// ... and the tile kernels, of this single step or weight gradient.
size_t gemm_bf16_split_ws_bytes(const GemmParams &p, bool w_kn, int num_cu);
hipError_t launch_gemm_rows(const GemmParams &p, bool bf16, bool w_kn, bool out_bf16, hipStream_t s, int num_cu);
hipError_t launch_gemm_f32(const GemmParams &p, bool w_kn, hipStream_t s, int num_cu);

bool attn_slice_supported(const AttnParams &p);
hipError_t launch_attn_slice(const AttnParams &p, hipStream_t s, int num_cu);

// dst[s][e] += src[s][e], e in [0, n), for n_seg disjoint segments, any 4-byte alignment
// (land: nullable -- what is read from src[s] is also stored to land[s], the delivery carried by the consumer)
hipError_t launch_dp_reduce_segments(float *const *dst, const float *const *src, float *const *land, int n_seg, int64_t n,
                                     hipStream_t s);
// dst <- (((dst + src[0]) + src[1]) + ...) over n elements, one pass when n_src <= 15 (else one pass per source: same
// additions, same order, same bits)
hipError_t launch_dp_reduce_multi(float *dst, const float *const *src, int n_src, int64_t n, hipStream_t s,
                                  float *const *land = nullptr, bool init = false);   // init: dst <- (src[0] + src[1]) + ...
// n (<= 16) copies of `bytes` bytes each in one launch; copy_batch_takes says whether the arguments qualify
// (16-byte aligned pointers, bytes a multiple of 16), else the caller copies one by one
bool copy_batch_takes(const void *const *src, void *const *dst, int n, size_t bytes);
hipError_t launch_copy_batch(const void *const *src, void *const *dst, int n, size_t bytes, hipStream_t s);

// Writes `value` to each of dst[0..count) with device-coherent stores (flags polled by other kernels).
hipError_t launch_set_words(unsigned *dst, int count, unsigned value, hipStream_t s);

// Fills a buffer with 0xFF bytes (a NaN pattern for fp32 and bf16) -- debug poison.
hipError_t launch_fill_ff(void *dst, size_t bytes, hipStream_t s);

}  // namespace cf
