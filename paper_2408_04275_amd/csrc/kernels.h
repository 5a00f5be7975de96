// Internal launch interface between the C-ABI layer (api.hip) and the kernel files.
// Every launcher enqueues on `st` and returns the launch status; none synchronises.
#pragma once
#include "common.h"

namespace mmt {

enum { DT_F32 = 0, DT_BF16 = 1 };
enum { GEMM_NT = 0, GEMM_NN = 1, GEMM_TN = 2 };
enum { MASK_CAUSAL = 0, MASK_BIDIR = 1 };

struct GemmArgs {
    int layout;                 // GEMM_NT / GEMM_NN / GEMM_TN
    int M, N, K;
    const void *A; int lda;
    const void *B; int ldb;
    void *C; int ldc;
    const void *bias;           // [N] or null
    const void *residual;       // [M, ldc] or null
    bool accumulate;            // C += result
    bool c_f32 = false;         // C is fp32 whatever the operands' dtype (bias / residual are not combined with it)
    // optional scratch for the fp32 partial products of a last round cut along K (NN and TN, bf16) or of a whole product with
    // few tiles (NN, bf16), 256-byte aligned
    void *split_ws = nullptr;
    size_t split_ws_bytes = 0;
    // when not null and the product is cut as a whole (bf16 NN): its partial products [*chunks][M][N] are left in split_ws for the caller to
    // add up, and C is not written.  Otherwise left alone.
    int *chunks = nullptr;
    // measurement aid (matrix-core kernel only): when not null, device uint64[4]; the first workgroup stores the
    // shader-clock counter and the constant 100 MHz counter at its start ([0], [1]) and at its end ([2], [3])
    unsigned long long *clock_probe = nullptr;
};

// gemm_simple.hip: any dtype, any shape, LDS-tiled FMA kernel (what the matrix-core kernels do not take).
hipError_t gemm_simple(int dtype, const GemmArgs &g, hipStream_t st);
// gemm_f32.hip: fp32 storage on the fp32 matrix instruction.  `supported` checks alignment requirements.
bool gemm_f32_supported(const GemmArgs &g);
hipError_t gemm_f32(const GemmArgs &g, hipStream_t st);
// ... weight gradients with few tiles of 64 x 64 (below 384), up to 4 in one launch
bool gemm_f32_few_tiles(const GemmArgs &g);
struct ReduceJobSet;
// reduce: when not null, sums (reduce.h) that the same launch adds up, to fp32 outputs
hipError_t gemm_f32_group(const GemmArgs *gs, int n, const ReduceJobSet *reduce, hipStream_t st);
// ... products whose epilogue does the elementwise work behind them.  C = [gate | up], m [M, N / 2] = silu(gate) up
bool gemm_f32_swiglu_supported(const GemmArgs &g);
hipError_t gemm_f32_swiglu(const GemmArgs &g, void *m, hipStream_t st);
// C's first `rotated` heads of d columns get the rotary embedding (cs: [M, d / 2])
bool gemm_f32_rope_supported(const GemmArgs &g, int d);
hipError_t gemm_f32_rope(const GemmArgs &g, int d, int rotated, const float2 *cs, hipStream_t st);
// the product is the gradient of silu(gate) up with gu = [gate | up]: C = [d_gate | d_up], leading dimension 2 N
bool gemm_f32_swiglu_bwd_supported(const GemmArgs &g);
hipError_t gemm_f32_swiglu_bwd(const GemmArgs &g, const void *gu, hipStream_t st);
// gemm_mfma.hip: bf16 MFMA kernel.  `supported` checks alignment requirements.
bool gemm_mfma_supported(const GemmArgs &g);
hipError_t gemm_mfma(const GemmArgs &g, hipStream_t st);
// How a product runs on n_cu compute units: tiles of tile_m x tile_n; all of it in `chunks` chunks of K (1: whole), or the last
// tail_tiles tiles of the order in `chunks` chunks each.  Chunks are k_chunk long, the last one shorter.
struct GemmPlan { int shape, tile_m, tile_n, tail_tiles, chunks, k_chunk; };
GemmPlan gemm_mfma_plan(const GemmArgs &g, int n_cu);
// units of 512 clocks by which every second workgroup of a weight gradient with fp32 output starts later on n_cu compute units
int gemm_mfma_late_start(const GemmArgs &g, int n_cu);
// Scratch (GemmArgs::split_ws) with which no cut along K is restricted: input gradients of up to M rows (NN), weight gradients over
// up to K tokens (TN).  Neither falls as that argument grows.
size_t gemm_mfma_nn_scratch(long M, long N, long K);
size_t gemm_mfma_tn_scratch(long M, long N, long K);
// Weight gradients with few output tiles (gemm_mfma_few_tiles: transposed-A layout, no bias / residual, at most 128 tiles of
// 256 x 256) computed together in one launch; up to 4, all with the same K and accumulate / c_f32.
bool gemm_mfma_few_tiles(const GemmArgs &g);
// reduce: when not null, sums (reduce.h) that the same launch adds up, to outputs of the gradients' type; worth it where the launch has room.
bool gemm_mfma_group_has_room(const GemmArgs *gs, int n, const ReduceJobSet &sums);
bool gemm_mfma_group_has_room(const GemmArgs *gs, int n, const ReduceJobSet &sums, int n_cu);
hipError_t gemm_mfma_group(const GemmArgs *gs, int n, const ReduceJobSet *reduce, hipStream_t st);

// Segment bookkeeping produced by prep_tokens():
//   tok_seg[t]  = index of the segment that holds token t
//   tok_info[t] = {start of that segment, end of that segment with bit 30 set if it is bidirectional}
constexpr int COLSUM_HEAD = 96;
constexpr int ATTN_LANE_SEGMENTS = 64;      // one per lane of a wavefront
struct AttnArgs {
    int T, S, nh, nkv, d;
    float scale;
    const int *cu;              // device [S+1]
    const uint8_t *modes;       // device [S] or null
    int default_mode;
    const int *tok_seg;         // device [T]
    const void *qkv; int ld_qkv;
    void *o;                    // [T, nh*d]
    float *lse;                 // [nh, T]
    const void *d_o;            // bwd: [T, nh*d]
    void *d_qkv;                // bwd: [T, ld_qkv]
    float *Dsum;                // bwd scratch: [nh, T]; D = rowsum(dO * O) per query and head (the bf16 kernels keep -D there; the fp32 matrix kernels write and
                                // read it where dQ and dK/dV are two launches)
    // MFMA path: tok_info[t] = {segment start, segment end | (bidirectional ? 1 << 30 : 0)}; may be null for a pack of at most
    // ATTN_LANE_SEGMENTS segments (cu and modes are read instead)
    const int2 *tok_info;
    // MFMA path, backward: when not null, the [T, d/2] (cos, sin) table of the rotary embedding; dQ and dK are
    // then rotated back in the kernels' epilogues (otherwise the caller does it afterwards)
    const float2 *rope_cs;
    // MFMA path, backward, grouped heads: scratch for fp32 partial sums of dK and dV (may be null), [parts][T][2 nkv d]
    float *dkv_part; size_t dkv_part_bytes;
    // MFMA path, backward, heads of up to COLSUM_HEAD features, one query head per key/value head: when not null, receives the column sums
    // of d_qkv over every 32 tokens, [ceil(T / 32)][ld_qkv] fp32 (the gradient of the bias that qkv has)
    float *colsum;
    int dkv_parts;              // workgroups that share a group's query heads; set by attn_mfma_bwd
    // MFMA path: dispatch order of the query tiles (256 queries: forward, dQ) and of the key tiles (128
    // keys: dK/dV), heaviest first; use_order = 0 means index order (more tiles than the tables hold)
    int use_order;
    int q_steps;                // 64-key steps of all query tiles together (0: not counted, use_order = 0)
    uint8_t order_q[64];
    uint8_t order_k[128];
    // MFMA path, measurement aid: when not null, device [3][1024] counters; every workgroup adds its run time
    // (100 MHz ticks) to the entry of the compute unit it ran on (forward: row 0, dQ: row 1, dK/dV: row 2)
    unsigned long long *cu_busy;
};
// reorder.hip (host): Algorithm 1 and the tile orders above
int intra_reorder(const double *sizes, int n, int m, int32_t *order, int32_t *group_begin, double *group_load);
void attn_tile_order(const int32_t *cu_host, const uint8_t *modes_host, int default_mode, int S, int T, AttnArgs &a);
// pipeline.hip (host): timeline of the one-forward-one-backward pipeline schedule and Algorithm 2.
// fwd / bwd: [p][l] durations by original microbatch index; order: [l] (null: identity); return 0 on success
int pipeline_1f1b(const double *fwd, const double *bwd, int p, int l, const int32_t *order, double *makespan,
                  double *intervals /* [l] or null */);
int inter_reorder(const double *fwd, const double *bwd, int p, int l, const double *sizes /* [l] or null */, int32_t *order,
                  double *intervals_seen /* [l] or null */, int32_t *n_seen /* or null */);
// attn_simple.hip: fp32 storage on the vector ALUs, any size
hipError_t attn_simple_fwd(const AttnArgs &a, hipStream_t st);
hipError_t attn_simple_bwd(const AttnArgs &a, hipStream_t st);
// attn_f32.hip: fp32 storage on the fp32 matrix instruction (backward: dQ and dK are rotated back if rope_cs is given)
bool attn_f32_supported(const AttnArgs &a);
hipError_t attn_f32_fwd(const AttnArgs &a, hipStream_t st);
hipError_t attn_f32_bwd(const AttnArgs &a, hipStream_t st);
int attn_f32_bwd_launches(int T, int nh, int nkv, int d);
// attn_mfma.hip: bf16 storage, matrix cores
hipError_t attn_mfma_fwd(const AttnArgs &a, hipStream_t st);
hipError_t attn_mfma_bwd(const AttnArgs &a, hipStream_t st);

// Backward, grouped heads: workgroups that share the query heads of a group (1: none), each with an fp32 partial result of
// attn_dkv_part_bytes; parts * that never exceeds DKV_PART_BYTES_MAX.  attn_dkv_room: the most that any pack of up to T tokens takes
// (a longer pack has fewer shares).
constexpr size_t DKV_PART_BYTES_MAX = size_t(96) << 20;
inline size_t attn_dkv_part_bytes(int T, int nkv, int d) { return (size_t)T * 2 * nkv * d * 4; }
int attn_dkv_parts(int T, int nh, int nkv, int d);
size_t attn_dkv_room(int T, int nh, int nkv, int d);

// elementwise.hip
hipError_t fill_zero(void *p, size_t elems, int dtype, hipStream_t st);
// Token bookkeeping of a pack: tok_seg, tok_info (see AttnArgs) and, if rope_cs is not null, the [T, d/2] rotary table.
struct TokenPrep {
    const int *cu;              // device [S+1]
    const uint8_t *modes;       // device [S] or null
    int default_mode, S, T;
    int *tok_seg;
    int2 *tok_info;
    int d;
    float rope_base;
    float2 *rope_cs;
};
hipError_t prep_tokens(const TokenPrep &p, hipStream_t st);
// prep: when not null, the same launch does that bookkeeping
hipError_t norm_fwd(int dtype, bool layernorm, const void *x, const void *g, const void *b, void *out,
                    float *mean, float *rstd, int T, int H, float eps, const TokenPrep *prep, hipStream_t st);
// d_in = norm_bwd(d_out) + d_res;  gain/bias gradient partial sums go to part_g/part_b, the column sums of d_in
// and of d_res to part_din / part_dres ([norm_bwd_blocks(T, H), H] fp32 each; null = skip).
int norm_bwd_blocks(int T, int H);
// A d_out that is still in fp32 parts [n_parts][T][H] (see GemmArgs::chunks), which the kernel adds up itself, comes as `parts` (n_parts: 0 if it is not).
bool norm_bwd_adds_parts(int dtype, bool layernorm, int H);
struct NormParts { const float *p = nullptr; int n = 0; };
hipError_t norm_bwd(int dtype, bool layernorm, const void *d_out, const void *x, const void *g,
                    const float *mean, const float *rstd, const void *d_res, void *d_in,
                    float *part_g, float *part_b, float *part_din, float *part_dres, int T, int H, NormParts parts, hipStream_t st);
// out[c] (+)= sum_r part[r, c]
hipError_t reduce_partials(int dtype, const float *part, int rows, int N, void *out, bool accumulate,
                           hipStream_t st);
int colsum_slabs(int T);
int colsum_slabs_max(int T);    // the most slabs that a pack of up to T tokens has (longer packs have longer slabs)
// out[N] (+)= the sum of the rows of part[rows, N], for up to eight arrays of different shapes in one launch (null part or out: skipped)
struct ReduceJob { const float *part; void *out; int rows, N; };
hipError_t reduce_jobs(int dtype, const ReduceJob *jobs, int n, bool accumulate, hipStream_t st);
hipError_t colsum_partials(int dtype, const void *in, int T, int N, int ld, float *part, hipStream_t st);
hipError_t rope_inplace(int dtype, void *qkv, int ld, int T, int n_rot_heads, int d, const float2 *rope_cs,
                        bool inverse, hipStream_t st);
hipError_t swiglu_fwd(int dtype, const void *gu, void *m, int T, int F, hipStream_t st);
hipError_t swiglu_bwd(int dtype, const void *d_m, const void *gu, void *d_gu, int T, int F, hipStream_t st);
hipError_t gelu_fwd(int dtype, const void *z, void *a, long n, hipStream_t st);
hipError_t gelu_bwd(int dtype, const void *d_a, const void *z, void *d_z, long n, hipStream_t st);
// the same over [T, N] rows, with the column sums of d_z as partial sums part[colsum_slabs(T), N]
hipError_t gelu_bwd_colsum(int dtype, const void *d_a, const void *z, void *d_z, int T, int N, float *part, hipStream_t st);


// optimizer.hip: one AdamW step on fp32 master weights; omb = 1 - beta, inv_bias1 = 1 / (1 - beta1^t),
// inv_bias2 = 1 / (1 - beta2^t), all four evaluated in double by the caller
struct AdamArgs {
    float lr, beta1, beta2, omb1, omb2, eps, weight_decay, grad_scale, inv_bias1, inv_bias2;
    int zero_grad;
};
// whether a shard of n elements is streamed (param_bytes: per element of the working copy, 0 without one)
bool adam_streams(size_t n, size_t param_bytes);
hipError_t adam_step(int param_dtype, size_t n, float *w, float *g, float *m, float *v, void *p, const AdamArgs &a,
                     hipStream_t st);

}  // namespace mmt
