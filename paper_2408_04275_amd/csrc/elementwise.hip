// HBM-bound kernels of the layer: token bookkeeping, RMSNorm / LayerNorm forward and
// backward, rotary embedding, SwiGLU / GELU, column sums.  All arithmetic is fp32;
// storage is fp32 or bf16.  Every kernel moves 16 bytes per lane per access and
// touches each tensor once (rows are re-read from cache, not from HBM).
#include "kernels.h"
#include "reduce.h"
#include <algorithm>
#include <type_traits>
#include <atomic>

namespace mmt {

// ---- 8-element vector access --------------------------------------------------------
__device__ __forceinline__ void load8(const float *p, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t *p, float (&v)[8]) {
    const uint4 a = *reinterpret_cast<const uint4 *>(p);
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void store8(float *p, const float (&v)[8]) {
    *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4 *>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16_t *p, const float (&v)[8]) {
    uint4 a;
    a.x = pack_bf16x2(v[0], v[1]); a.y = pack_bf16x2(v[2], v[3]);
    a.z = pack_bf16x2(v[4], v[5]); a.w = pack_bf16x2(v[6], v[7]);
    *reinterpret_cast<uint4 *>(p) = a;
}

// Streaming forms for tensors that a kernel passes over once and that are far larger than the caches.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
__device__ __forceinline__ void load8_stream(const bf16_t *p, float (&v)[8]) {
    const u32x4_t a = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(a[i] << 16);
        v[2 * i + 1] = __uint_as_float(a[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void load8_stream(const float *p, float (&v)[8]) { load8(p, v); }
__device__ __forceinline__ void store8_stream(bf16_t *p, const float (&v)[8]) {
    u32x4_t a;
    a[0] = pack_bf16x2(v[0], v[1]); a[1] = pack_bf16x2(v[2], v[3]);
    a[2] = pack_bf16x2(v[4], v[5]); a[3] = pack_bf16x2(v[6], v[7]);
    __builtin_nontemporal_store(a, reinterpret_cast<u32x4_t *>(p));
}
__device__ __forceinline__ void store8_stream(float *p, const float (&v)[8]) { store8(p, v); }

// Eight elements as loaded, not yet widened to fp32: what a kernel holds for a row it has requested ahead of time
// (four registers per chunk in bf16 instead of eight).
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> { uint4 a; };
template <> struct Raw8<float> { float4 a, b; };
__device__ __forceinline__ void load_raw8(const bf16_t *p, Raw8<bf16_t> &r) {
    // streaming form: each of these tensors is passed over once (norm backward at the 7B shape: 49.8 -> 46.4 us)
    const u32x4_t a = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
    r.a = make_uint4(a[0], a[1], a[2], a[3]);
}
__device__ __forceinline__ void load_raw8(const float *p, Raw8<float> &r) {
    r.a = *reinterpret_cast<const float4 *>(p); r.b = *reinterpret_cast<const float4 *>(p + 4);
}
__device__ __forceinline__ Raw8<bf16_t> load_plain8(const bf16_t *p) { return {*reinterpret_cast<const uint4 *>(p)}; }
__device__ __forceinline__ Raw8<float> load_plain8(const float *p) { return {*reinterpret_cast<const float4 *>(p), *reinterpret_cast<const float4 *>(p + 4)}; }
__device__ __forceinline__ void unpack8(const Raw8<bf16_t> &r, float (&v)[8]) {
    const uint32_t w[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void unpack8(const Raw8<float> &r, float (&v)[8]) {
    v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w; v[4] = r.b.x; v[5] = r.b.y; v[6] = r.b.z; v[7] = r.b.w;
}

// ---- token bookkeeping ---------------------------------------------------------------
// tok_seg[t] = s with cu[s] <= t < cu[s+1].
__device__ __forceinline__ int find_segment(const int *__restrict__ cu, int S, int t) {
    int lo = 0, hi = S;               // last s in [0, S) with cu[s] <= t
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ void token_entry(const TokenPrep &p, int t) {
    if (t >= p.T) return;
    const int s = find_segment(p.cu, p.S, t);
    p.tok_seg[t] = s;
    const int mode = p.modes ? p.modes[s] : p.default_mode;
    p.tok_info[t] = make_int2(p.cu[s], p.cu[s + 1] | (mode == MASK_BIDIR ? (1 << 30) : 0));
}

// rope_cs[t, i] = (cos, sin)(pos(t) * base^(-2i/d)), pos(t) = t - cu[seg(t)]; evaluated in double
// so that the fp32 table is correctly rounded for any position.
__device__ __forceinline__ void rope_entry(const TokenPrep &p, long idx) {
    const int half = p.d >> 1;
    if (idx >= (long)p.T * half) return;
    const int t = (int)(idx / half), i = (int)(idx % half);
    const double pos = (double)(t - p.cu[find_segment(p.cu, p.S, t)]);
    const double phi = pos * exp(-2.0 * i / p.d * log((double)p.rope_base));
    p.rope_cs[idx] = make_float2((float)cos(phi), (float)sin(phi));
}

// Workgroup b of the bookkeeping: 256 tokens each, then 256 entries of the rotary table each.
static int token_prep_blocks(const TokenPrep &p) {
    return ceil_div(p.T, 256) + (p.rope_cs ? ceil_div((long)p.T * (p.d / 2), 256) : 0);
}
__device__ __forceinline__ void token_prep(const TokenPrep &p, int b) {
    const int tok_blocks = (p.T + 255) / 256;
    if (b < tok_blocks) token_entry(p, b * 256 + threadIdx.x);
    else rope_entry(p, (long)(b - tok_blocks) * 256 + threadIdx.x);
}

__global__ __launch_bounds__(256) void token_prep_kernel(TokenPrep p) { token_prep(p, blockIdx.x); }

hipError_t prep_tokens(const TokenPrep &p, hipStream_t st) {
    if (p.T == 0) return hipSuccess;
    token_prep_kernel<<<token_prep_blocks(p), 256, 0, st>>>(p);
    return hipGetLastError();
}

// ---- normalisation forward -----------------------------------------------------------
// RMSNorm: out = x * rsqrt(mean(x^2) + eps) * g.
// LayerNorm: out = (x - mean) * rsqrt(var_biased + eps) * g + b (variance about the mean, two passes).
// The first prep_blocks workgroups do a layer's token bookkeeping instead, which the kernels after this one need: in launches
// of their own the two tables cost a small pack 2 x 4.7 us.
//
// Rows of at most 256 * 8 * MAXC elements, a workgroup walking every `blocks`-th row: the row stays in registers between the
// statistics and the scaling (one read of x), the gain and bias are fetched once per workgroup, and the next row is requested
// before the current one is reduced, so that a workgroup always has a row in flight (with one short-lived workgroup per row the
// kernel reached 5.5 TB/s).
template <typename T, bool LN, int MAXC>
__global__ __launch_bounds__(256) void norm_fwd_rows_kernel(const T *__restrict__ x, const T *__restrict__ g,
                                                            const T *__restrict__ b, T *__restrict__ out,
                                                            float *__restrict__ mean, float *__restrict__ rstd,
                                                            int nrows, int H, float eps, TokenPrep prep, int prep_blocks) {
    if ((int)blockIdx.x < prep_blocks) return token_prep(prep, blockIdx.x);
    const unsigned block = blockIdx.x - prep_blocks, blocks = gridDim.x - prep_blocks;
    __shared__ float red[4];
    float gv[MAXC][8], bv[LN ? MAXC : 1][8], cur[MAXC][8], nxt[MAXC][8];
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        const int c = (threadIdx.x + i * 256) * 8;
        if (c < H) {
            load8(g + c, gv[i]);
            if (LN) load8(b + c, bv[i]);
            if (block < nrows) load8(x + (size_t)block * H + c, cur[i]);
        }
    }
    for (size_t row = block; row < (size_t)nrows; row += blocks) {
        const size_t next = row + blocks;
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = (threadIdx.x + i * 256) * 8;
            if (c < H && next < (size_t)nrows) load8(x + next * H + c, nxt[i]);
        }
        float mu = 0.f;
        if (LN) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < MAXC; ++i)
                if ((threadIdx.x + i * 256) * 8 < H) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) s += cur[i][j];
                }
            mu = block_sum<4>(s, red) / H;
        }
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if ((threadIdx.x + i * 256) * 8 < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) ss += (cur[i][j] - mu) * (cur[i][j] - mu);
            }
        const float r = 1.0f / sqrtf(block_sum<4>(ss, red) / H + eps);
        if (threadIdx.x == 0) {
            rstd[row] = r;
            if (LN) mean[row] = mu;
        }
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = (threadIdx.x + i * 256) * 8;
            if (c < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) cur[i][j] = (cur[i][j] - mu) * r * gv[i][j] + (LN ? bv[i][j] : 0.f);
                store8(out + row * H + c, cur[i]);
#pragma unroll
                for (int j = 0; j < 8; ++j) cur[i][j] = nxt[i][j];
            }
        }
    }
}

// The same for rows of at most 512 * MAXC elements (MAXC <= 4), one wavefront per row: a 1024-wide row gives only half of a
// workgroup's threads a chunk of 8, and its sums are a few cross-lane steps without a barrier.  9536 rows of 1024: 15.4 -> 10.4 us.
template <typename T, bool LN, int MAXC>
__global__ __launch_bounds__(256) void norm_fwd_wave_kernel(const T *__restrict__ x, const T *__restrict__ g,
                                                            const T *__restrict__ b, T *__restrict__ out,
                                                            float *__restrict__ mean, float *__restrict__ rstd,
                                                            int nrows, int H, float eps, TokenPrep prep, int prep_blocks) {
    if ((int)blockIdx.x < prep_blocks) return token_prep(prep, blockIdx.x);
    const int lane = threadIdx.x & 63, step = (gridDim.x - prep_blocks) * 4;
    int row = (blockIdx.x - prep_blocks) * 4 + (threadIdx.x >> 6);
    float gv[MAXC][8], bv[LN ? MAXC : 1][8];
    Raw8<T> nxt[MAXC];
    auto request = [&](int r) {
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = (lane + i * 64) * 8;
            if (c < H && r < nrows) nxt[i] = load_plain8(x + (size_t)r * H + c);
        }
    };
    request(row);
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        const int c = (lane + i * 64) * 8;
        if (c < H) {
            load8(g + c, gv[i]);
            if (LN) load8(b + c, bv[i]);
        }
    }
    for (; row < nrows; row += step) {
        float cur[MAXC][8];
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            if ((lane + i * 64) * 8 < H) unpack8(nxt[i], cur[i]);
            else {
#pragma unroll
                for (int j = 0; j < 8; ++j) cur[i][j] = 0.f;
            }
        }
        request(row + step);
        float mu = 0.f;
        if (LN) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < MAXC; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) s += cur[i][j];
            mu = wave_sum(s) / H;
        }
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if ((lane + i * 64) * 8 < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) ss += (cur[i][j] - mu) * (cur[i][j] - mu);
            }
        const float r = 1.0f / sqrtf(wave_sum(ss) / H + eps);
        if (lane == 0) {
            rstd[row] = r;
            if (LN) mean[row] = mu;
        }
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = (lane + i * 64) * 8;
            if (c < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) cur[i][j] = (cur[i][j] - mu) * r * gv[i][j] + (LN ? bv[i][j] : 0.f);
                store8(out + (size_t)row * H + c, cur[i]);
            }
        }
    }
}

// One launch of norm_fwd_rows_kernel or norm_fwd_wave_kernel: exactly as many workgroups as the device keeps resident at once (a grid one
// workgroup per compute unit larger runs a second, nearly empty round: 22.9 -> 26.9 us at the 7B shape).
template <typename K>
hipError_t resident_workgroups(std::atomic<int> &cached, K kern, int &grid) {
    grid = cached.load(std::memory_order_relaxed);
    if (grid) return hipSuccess;
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 256, 0);
    if (e != hipSuccess) return e;
    grid = (cus > 0 ? cus : 256) * (per_cu > 0 ? per_cu : 4);
    cached.store(grid, std::memory_order_relaxed);
    return hipSuccess;
}
// WAVE_ROWS: a wavefront per row (four per workgroup), otherwise a workgroup per row
template <typename T, bool LN, int MAXC, bool WAVE_ROWS>
hipError_t launch_norm_fwd_rows(const void *x, const void *g, const void *b, void *out, float *mean, float *rstd, int nrows,
                                int H, float eps, const TokenPrep *prep, hipStream_t st) {
    static std::atomic<int> resident{0};
    auto kern = [] {
        if constexpr (WAVE_ROWS) return norm_fwd_wave_kernel<T, LN, MAXC>;
        else return norm_fwd_rows_kernel<T, LN, MAXC>;
    }();
    int grid = 0;
    hipError_t e = resident_workgroups(resident, kern, grid);
    if (e != hipSuccess) return e;
    const int all = WAVE_ROWS ? ceil_div(nrows, 4) : nrows, prep_blocks = prep ? token_prep_blocks(*prep) : 0;
    kern<<<prep_blocks + (all < grid ? all : grid), 256, 0, st>>>((const T *)x, (const T *)g, (const T *)b, (T *)out, mean, rstd, nrows, H,
                                                                  eps, prep ? *prep : TokenPrep{}, prep_blocks);
    return hipGetLastError();
}

hipError_t norm_fwd(int dtype, bool layernorm, const void *x, const void *g, const void *b, void *out,
                    float *mean, float *rstd, int T, int H, float eps, const TokenPrep *prep, hipStream_t st) {
    if (T == 0) return hipSuccess;
    if (H % 8 || H > 8192) return hipErrorInvalidValue;
#define R(TT, LNV, MC, WR) return launch_norm_fwd_rows<TT, LNV, MC, WR>(x, g, b, out, mean, rstd, T, H, eps, prep, st)
#define L(TT, LNV) do { if (H <= 512) R(TT, LNV, 1, true); else if (H <= 1024) R(TT, LNV, 2, true); else if (H <= 1536) R(TT, LNV, 3, true); \
                        else if (H <= 2048) R(TT, LNV, 4, true); else if (H <= 4096) R(TT, LNV, 2, false); else R(TT, LNV, 4, false); } while (0)
    if (dtype == DT_F32) { if (layernorm) L(float, true); else L(float, false); }
    else { if (layernorm) L(bf16_t, true); else L(bf16_t, false); }
#undef L
#undef R
    return hipGetLastError();
}

// ---- normalisation backward ----------------------------------------------------------
// With xhat = (x - mean) * r and ghat = d_out * g:
//   d_in = r * (ghat - mean_H(ghat) [LayerNorm only] - xhat * mean_H(ghat * xhat)) + d_res
//   dg = sum_t d_out * xhat,  db = sum_t d_out.
// A workgroup walks rows blockIdx.x, blockIdx.x + gridDim.x, ...; each thread owns the same
// columns in every row, so the gain/bias partial sums stay in registers and are written once
// per workgroup to part_g / part_b [gridDim.x, H].
constexpr int NORM_BWD_MAXC = 4;          // column chunks of 8 per thread: H <= 256 * 8 * 4 = 8192 (the kernel is also
                                          // built for 1 and 2 chunks: fewer registers per thread, more rows in flight)
constexpr int NORM_BWD_GRID = 512;

// Rows up to this width take a wavefront each (wider ones need more registers than leave room for two wavefronts per SIMD:
// 4111 rows of 1280 15.4 -> 22.5 us)
constexpr int NORM_BWD_WAVE_H = 1024;

// up to 4096 there are registers for more resident workgroups: twice the grid; narrow rows: four rows per workgroup at a time
int norm_bwd_blocks(int T, int H) {
    const int grid = H > NORM_BWD_WAVE_H && H <= 4096 ? 2 * NORM_BWD_GRID : NORM_BWD_GRID;
    const int all = H <= NORM_BWD_WAVE_H ? ceil_div(T, 4) : T;
    return all < grid ? (all > 0 ? all : 1) : grid;
}

// SPLIT: d_out comes as the fp32 partial products of the input gradient in front, cut along K, and is added up here, in order, instead
// of by a kernel that writes it and this one that reads it back: 1031 rows of 4096 in three parts, 14.2 + 11.6 -> 21.1 us.  The parts
// are not requested a row ahead (up to 1024 rows a workgroup has one, up to 2047 two).
template <typename T, bool LN, int NORM_BWD_MAXC, bool COLS, bool SPLIT = false>
__global__ __launch_bounds__(256) void norm_bwd_kernel(const T *__restrict__ d_out, const T *__restrict__ x,
                                                       const T *__restrict__ g, const float *__restrict__ mean,
                                                       const float *__restrict__ rstd, const T *__restrict__ d_res,
                                                       T *__restrict__ d_in, float *__restrict__ part_g,
                                                       float *__restrict__ part_b, float *__restrict__ part_din,
                                                       float *__restrict__ part_dres, int nrows, int H, NormParts parts) {
    __shared__ float red[4];
    float gv[NORM_BWD_MAXC][8], ag[NORM_BWD_MAXC][8], ab[NORM_BWD_MAXC][8];
    // COLS: column sums of the result and of the added gradient as well (the bias gradients of the two linears
    // that sit on either side of the normalisation's residual branch)
    float ad[COLS ? NORM_BWD_MAXC : 1][8], ae[COLS ? NORM_BWD_MAXC : 1][8];
#pragma unroll
    for (int i = 0; i < NORM_BWD_MAXC; ++i) {
        const int c = (threadIdx.x + i * 256) * 8;
        if (c < H) load8(g + c, gv[i]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            ag[i][j] = 0.f; ab[i][j] = 0.f;
            if (COLS) { ad[i][j] = 0.f; ae[i][j] = 0.f; }
        }
    }
    // All three inputs of a row are requested together, and a row ahead: while a row is reduced and stored the next one
    // is in flight (held as loaded, widened to fp32 when its turn comes).
    Raw8<T> pd[NORM_BWD_MAXC], px[NORM_BWD_MAXC], pr[NORM_BWD_MAXC];
    auto request = [&](size_t row) {
#pragma unroll
        for (int i = 0; i < NORM_BWD_MAXC; ++i) {
            const int c = (threadIdx.x + i * 256) * 8;
            if (c < H && row < (size_t)nrows) {
                if (!SPLIT) load_raw8(d_out + row * H + c, pd[i]);
                load_raw8(x + row * H + c, px[i]);
                load_raw8(d_res + row * H + c, pr[i]);
            }
        }
    };
    request(blockIdx.x);
    for (size_t row = blockIdx.x; row < (size_t)nrows; row += gridDim.x) {
        const float r = rstd[row];
        const float mu = LN ? mean[row] : 0.f;
        float dv[NORM_BWD_MAXC][8], xh[NORM_BWD_MAXC][8], rv[NORM_BWD_MAXC][8];
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int i = 0; i < NORM_BWD_MAXC; ++i) {
            if ((threadIdx.x + i * 256) * 8 < H) {
                if (!SPLIT) unpack8(pd[i], dv[i]);
                unpack8(px[i], xh[i]); unpack8(pr[i], rv[i]);
            }
        }
        if constexpr (SPLIT) {
            const size_t plane = (size_t)nrows * H;
            constexpr int BATCH = 4;                               // parts on their way together
#pragma unroll
            for (int i = 0; i < NORM_BWD_MAXC; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) dv[i][j] = 0.f;
            for (int s = 0; s < parts.n; s += BATCH) {
                f32x4 v[BATCH][NORM_BWD_MAXC][2];
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
#pragma unroll
                    for (int i = 0; i < NORM_BWD_MAXC; ++i) {
                        const int c = (threadIdx.x + i * 256) * 8;
                        v[u][i][0] = v[u][i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
                        if (c >= H || s + u >= parts.n) continue;
                        const f32x4 *q = reinterpret_cast<const f32x4 *>(parts.p + (s + u) * plane + row * H + c);
                        v[u][i][0] = q[0];
                        v[u][i][1] = q[1];
                    }
#pragma unroll
                for (int u = 0; u < BATCH; ++u)
#pragma unroll
                    for (int i = 0; i < NORM_BWD_MAXC; ++i)
#pragma unroll
                        for (int j = 0; j < 8; ++j) dv[i][j] += v[u][i][j >> 2][j & 3];
            }
        }
        request(row + gridDim.x);
#pragma unroll
        for (int i = 0; i < NORM_BWD_MAXC; ++i) {
            const int c = (threadIdx.x + i * 256) * 8;
            if (c < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    xh[i][j] = (xh[i][j] - mu) * r;
                    ag[i][j] += dv[i][j] * xh[i][j];
                    ab[i][j] += dv[i][j];
                    dv[i][j] *= gv[i][j];          // ghat
                    s0 += dv[i][j];
                    s1 += dv[i][j] * xh[i][j];
                }
            }
        }
        s1 = block_sum<4>(s1, red) / H;
        s0 = LN ? block_sum<4>(s0, red) / H : 0.f;
#pragma unroll
        for (int i = 0; i < NORM_BWD_MAXC; ++i) {
            const int c = (threadIdx.x + i * 256) * 8;
            if (c < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (COLS) ae[i][j] += rv[i][j];
                    rv[i][j] += r * (dv[i][j] - s0 - xh[i][j] * s1);
                    if (COLS) ad[i][j] += rv[i][j];
                }
                store8(d_in + row * H + c, rv[i]);      // a plain store: the streaming form is slower here (46 -> 49.5 us)
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NORM_BWD_MAXC; ++i) {
        const int c = (threadIdx.x + i * 256) * 8;
        if (c < H) {
            if (part_g) store8(part_g + (size_t)blockIdx.x * H + c, ag[i]);
            if (LN && part_b) store8(part_b + (size_t)blockIdx.x * H + c, ab[i]);
            if (COLS && part_din) store8(part_din + (size_t)blockIdx.x * H + c, ad[i]);
            if (COLS && part_dres) store8(part_dres + (size_t)blockIdx.x * H + c, ae[i]);
        }
    }
}

// The same for rows of at most 512 * MAXC elements, one wavefront per row (as in norm_fwd_wave_kernel): no barrier per row, all
// lanes at work on a 1024-wide row, and half the partial rows (or fewer).  9536 rows of 1024, with / without the column sums:
// 25.1 -> 20.1 / 23.0 -> 18.1 us, and their reduction 17.2 -> 12.0.
template <typename T, bool LN, int MAXC, bool COLS>
__global__ __launch_bounds__(256) void norm_bwd_wave_kernel(const T *__restrict__ d_out, const T *__restrict__ x,
                                                            const T *__restrict__ g, const float *__restrict__ mean,
                                                            const float *__restrict__ rstd, const T *__restrict__ d_res,
                                                            T *__restrict__ d_in, float *__restrict__ part_g,
                                                            float *__restrict__ part_b, float *__restrict__ part_din,
                                                            float *__restrict__ part_dres, int nrows, int H) {
    __shared__ __attribute__((aligned(16))) float red[4][512 * MAXC];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, step = gridDim.x * 4;
    float gv[MAXC][8], ag[MAXC][8], ab[LN ? MAXC : 1][8];
    float ad[COLS ? MAXC : 1][8], ae[COLS ? MAXC : 1][8];
    Raw8<T> pd[MAXC], px[MAXC], pr[MAXC];
    auto request = [&](int row) {
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = (lane + i * 64) * 8;
            if (c < H && row < nrows) {
                load_raw8(d_out + (size_t)row * H + c, pd[i]);
                load_raw8(x + (size_t)row * H + c, px[i]);
                load_raw8(d_res + (size_t)row * H + c, pr[i]);
            }
        }
    };
    int row = blockIdx.x * 4 + wave;
    request(row);
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
        const int c = (lane + i * 64) * 8;
        if (c < H) load8(g + c, gv[i]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            ag[i][j] = 0.f;
            if (LN) ab[i][j] = 0.f;
            if (COLS) { ad[i][j] = 0.f; ae[i][j] = 0.f; }
        }
    }
    for (; row < nrows; row += step) {
        const float r = rstd[row], mu = LN ? mean[row] : 0.f;
        float dv[MAXC][8], xh[MAXC][8], rv[MAXC][8], s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if ((lane + i * 64) * 8 < H) { unpack8(pd[i], dv[i]); unpack8(px[i], xh[i]); unpack8(pr[i], rv[i]); }
        request(row + step);
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if ((lane + i * 64) * 8 < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    xh[i][j] = (xh[i][j] - mu) * r;
                    ag[i][j] += dv[i][j] * xh[i][j];
                    if (LN) ab[i][j] += dv[i][j];
                    dv[i][j] *= gv[i][j];          // ghat
                    s0 += dv[i][j];
                    s1 += dv[i][j] * xh[i][j];
                }
            }
        s1 = wave_sum(s1) / H;
        s0 = LN ? wave_sum(s0) / H : 0.f;
#pragma unroll
        for (int i = 0; i < MAXC; ++i) {
            const int c = (lane + i * 64) * 8;
            if (c < H) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (COLS) ae[i][j] += rv[i][j];
                    rv[i][j] += r * (dv[i][j] - s0 - xh[i][j] * s1);
                    if (COLS) ad[i][j] += rv[i][j];
                }
                store8(d_in + (size_t)row * H + c, rv[i]);
            }
        }
    }
    // the four wavefronts' column sums, added in order, as one partial row
    auto flush = [&](const float (&v)[MAXC][8], float *part) {
        if (!part) return;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MAXC; ++i)
            if ((lane + i * 64) * 8 < H) store8(&red[wave][(lane + i * 64) * 8], v[i]);
        __syncthreads();
        for (int c = threadIdx.x * 4; c < H; c += 1024) {
            f32x4 s = *reinterpret_cast<const f32x4 *>(&red[0][c]);
#pragma unroll
            for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const f32x4 *>(&red[w][c]);
            *reinterpret_cast<f32x4 *>(part + (size_t)blockIdx.x * H + c) = s;
        }
    };
    flush(ag, part_g);
    if constexpr (LN) flush(ab, part_b);
    if constexpr (COLS) { flush(ad, part_din); flush(ae, part_dres); }
}

// Built for RMSNorm rows of more than NORM_BWD_WAVE_H and at most SPLIT_MAX_H columns; in front of other normalisations the parts are
// summed by a kernel of their own.  Backward of a frozen decoder layer, apart -> together, us: 4096 wide, 300, 700, 1031, 1400, 2047 tokens
// 244.4 -> 242.1, 363.3 -> 357.4, 474.4 -> 468.3, 636.3 -> 633.4, 807.8 -> 795.9; 2048 wide (ffn 11008), 300, 1400 154.2 -> 151.2, 355.6 ->
// 350.7.  Wider rows take four column chunks per thread, which leaves registers for one wavefront per SIMD (232 -> 352), and lose: 5120
// wide, 300, 1031 tokens 327.4 -> 330.8, 676.0 -> 681.7; 6144, 300 387.1 -> 390.3; 8192, 300 684.1 -> 688.4.
constexpr int SPLIT_MAX_H = 4096;
bool norm_bwd_adds_parts(int dtype, bool layernorm, int H) { return dtype == DT_BF16 && !layernorm && H > NORM_BWD_WAVE_H && H <= SPLIT_MAX_H; }

hipError_t norm_bwd(int dtype, bool layernorm, const void *d_out, const void *x, const void *g,
                    const float *mean, const float *rstd, const void *d_res, void *d_in, float *part_g,
                    float *part_b, float *part_din, float *part_dres, int T, int H, NormParts parts, hipStream_t st) {
    if (T == 0) return hipSuccess;
    if (H > 256 * 8 * NORM_BWD_MAXC) return hipErrorInvalidValue;
    const int grid = norm_bwd_blocks(T, H);
    const bool cols = part_din || part_dres;
    if (parts.n) {
        if (!norm_bwd_adds_parts(dtype, layernorm, H) || cols) return hipErrorInvalidValue;
        auto launch = [&](auto MAXC_) {
            norm_bwd_kernel<bf16_t, false, decltype(MAXC_)::value, false, true><<<grid, 256, 0, st>>>(
                nullptr, (const bf16_t *)x, (const bf16_t *)g, mean, rstd, (const bf16_t *)d_res, (bf16_t *)d_in, part_g, part_b, nullptr, nullptr, T, H, parts);
        };
        if (H <= 2048) launch(std::integral_constant<int, 1>{});
        else launch(std::integral_constant<int, 2>{});
        return hipGetLastError();
    }
#define L2(TT, LNV, MC, CV) norm_bwd_kernel<TT, LNV, MC, CV><<<grid, 256, 0, st>>>((const TT *)d_out, (const TT *)x, (const TT *)g, mean, rstd, (const TT *)d_res, (TT *)d_in, part_g, part_b, part_din, part_dres, T, H, parts)
#define L1(TT, LNV, MC) do { if (cols) L2(TT, LNV, MC, true); else L2(TT, LNV, MC, false); } while (0)
#define W2(TT, LNV, MC, CV) norm_bwd_wave_kernel<TT, LNV, MC, CV><<<grid, 256, 0, st>>>((const TT *)d_out, (const TT *)x, (const TT *)g, mean, rstd, (const TT *)d_res, (TT *)d_in, part_g, part_b, part_din, part_dres, T, H)
#define W1(TT, LNV, MC) do { if (cols) W2(TT, LNV, MC, true); else W2(TT, LNV, MC, false); } while (0)
#define L(TT, LNV) do { if (H <= 512) W1(TT, LNV, 1); else if (H <= NORM_BWD_WAVE_H) W1(TT, LNV, 2); \
                        else if (H <= 2048) L1(TT, LNV, 1); else if (H <= 4096) L1(TT, LNV, 2); else L1(TT, LNV, 4); } while (0)
    if (dtype == DT_F32) { if (layernorm) L(float, true); else L(float, false); }
    else { if (layernorm) L(bf16_t, true); else L(bf16_t, false); }
#undef L2
#undef L1
#undef W2
#undef W1
#undef L
    return hipGetLastError();
}

// ---- partial-sum reduction -----------------------------------------------------------
// 32 columns per workgroup.  Vector form (N a multiple of 4): 8 lanes cover the 32 columns with 16 bytes each and
// 32 row lanes walk the partial rows; scalar form: 32 column lanes, 8 row lanes.  Both combine through LDS in a
// fixed order.
template <typename T>
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float *__restrict__ part, int rows, int N,
                                                              T *__restrict__ out, bool accumulate) {
    __shared__ float red[8][33];
    const int c = blockIdx.x * 32 + (threadIdx.x & 31), rl = threadIdx.x >> 5;
    float s = 0.f;
    if (c < N)
        for (int r = rl; r < rows; r += 8) s += part[(size_t)r * N + c];
    red[rl][threadIdx.x & 31] = s;
    __syncthreads();
    if (rl == 0 && c < N) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) t += red[i][threadIdx.x];
        if (accumulate) t += Elem<T>::load(out + c);
        Elem<T>::store(out + c, t);
    }
}

template <typename T>
__global__ __launch_bounds__(256) void reduce_partials_vec_kernel(const float *__restrict__ part, int rows, int N,
                                                                  T *__restrict__ out, bool accumulate) {
    __shared__ float red[32][36];
    const int cl = threadIdx.x & 7, rl = threadIdx.x >> 3;
    const int c = blockIdx.x * 32 + cl * 4;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (c < N) {
        // eight rows in flight per thread: a thread's rows are 32 apart, and one load at a time leaves the kernel waiting
        // on memory latency (8 arrays of a few megabytes took 20 us)
        f32x4 t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = s;
        int r = rl;
        for (; r + 7 * 32 < rows; r += 256) {
            const float *q = part + (size_t)r * N + c;
            f32x4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4 *>(q + (size_t)(32 * u) * N);
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] += v[u];
        }
        for (; r < rows; r += 32) t[0] += *reinterpret_cast<const f32x4 *>(part + (size_t)r * N + c);
        s = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    }
    *reinterpret_cast<f32x4 *>(&red[rl][cl * 4]) = s;
    __syncthreads();
    const int oc = blockIdx.x * 32 + threadIdx.x;
    if (threadIdx.x < 32 && oc < N) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < 32; ++i) t += red[i][threadIdx.x];
        if (accumulate) t += Elem<T>::load(out + oc);
        Elem<T>::store(out + oc, t);
    }
}

hipError_t reduce_partials(int dtype, const float *part, int rows, int N, void *out, bool accumulate,
                           hipStream_t st) {
    if (N == 0) return hipSuccess;
    const int grid = ceil_div(N, 32);
    if (N % 4 == 0) {
        if (dtype == DT_F32) reduce_partials_vec_kernel<float><<<grid, 256, 0, st>>>(part, rows, N, (float *)out, accumulate);
        else reduce_partials_vec_kernel<bf16_t><<<grid, 256, 0, st>>>(part, rows, N, (bf16_t *)out, accumulate);
    } else {
        if (dtype == DT_F32) reduce_partials_kernel<float><<<grid, 256, 0, st>>>(part, rows, N, (float *)out, accumulate);
        else reduce_partials_kernel<bf16_t><<<grid, 256, 0, st>>>(part, rows, N, (bf16_t *)out, accumulate);
    }
    return hipGetLastError();
}

// one launch for a set of reductions (see reduce.h)
template <typename T>
__global__ __launch_bounds__(256) void reduce_jobs_kernel(ReduceJobSet set) {
    __shared__ float red[32][36];
    reduce_unit<T>(set, blockIdx.x, red, threadIdx.x);
}

bool reduce_job_set(const ReduceJob *jobs, int n, bool accumulate, ReduceJobSet &set) {
    set = {};
    set.accumulate = accumulate ? 1 : 0;
    int m = 0;
    for (int i = 0; i < n && m < 8; ++i) {
        if (!jobs[i].part || !jobs[i].out || jobs[i].N <= 0) continue;
        if (jobs[i].N % 4) return false;
        set.part[m] = jobs[i].part; set.out[m] = jobs[i].out; set.rows[m] = jobs[i].rows; set.N[m] = jobs[i].N;
        set.units[m + 1] = set.units[m] + ceil_div(jobs[i].N, 32);
        ++m;
    }
    for (int i = m + 1; i <= 8; ++i) set.units[i] = set.units[m];
    return m > 0;
}

hipError_t reduce_jobs(int dtype, const ReduceJob *jobs, int n, bool accumulate, hipStream_t st) {
    ReduceJobSet set;
    if (!reduce_job_set(jobs, n, accumulate, set)) {               // the vector form needs whole quads: one launch each
        for (int i = 0; i < n; ++i) {
            if (!jobs[i].part || !jobs[i].out || jobs[i].N <= 0) continue;
            hipError_t e = reduce_partials(dtype, jobs[i].part, jobs[i].rows, jobs[i].N, jobs[i].out, accumulate, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    if (dtype == DT_F32) reduce_jobs_kernel<float><<<set.units[8], 256, 0, st>>>(set);
    else reduce_jobs_kernel<bf16_t><<<set.units[8], 256, 0, st>>>(set);
    return hipGetLastError();
}

// ---- column sums (bias gradients) ----------------------------------------------------
// Rows per workgroup: short slabs, so that a [T, N] pass has enough workgroups (T N / 32768 at 16 rows), and shorter ones on
// short packs, where a slab's rows one after the other are the kernel's time (GELU backward, us: 2304 x 4096 24.6 at 16 rows,
// 15.5 at 4; 4111 x 5120 35.9 at 16, 29.8 at 8; 9536 x 4096 46.1 at 16, 48.3 at 8).  The pack's length alone decides: against 16 rows
// throughout, 33 sizes of 300 to 12000 rows and 1024 to 16384 columns take from 0.38 (1000 x 1024) to 1.04 of the time (3000 x 10240 39.1 ->
// 40.6, 3000 x 16384 68.6 -> 59.9).
int colsum_rows(int T) { return T > 6144 ? 16 : T > 3072 ? 8 : 4; }
int colsum_slabs(int T) { return T > 0 ? ceil_div(T, colsum_rows(T)) : 1; }
int colsum_slabs_max(int T) { return std::max({colsum_slabs(T), colsum_slabs(std::min(T, 3072)), colsum_slabs(std::min(T, 6144))}); }

template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(const T *__restrict__ in, int nrows, int N, int ld, int slab,
                                                     float *__restrict__ part) {
    const int c = (blockIdx.x * 256 + threadIdx.x) * 8;
    if (c >= N) return;
    const int r0 = blockIdx.y * slab, r1 = min(nrows, r0 + slab);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int r = r0; r < r1; r += 8) {              // 8 rows requested before the first is added
        float v[8][8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (r + k < r1) load8(in + (size_t)(r + k) * ld + c, v[k]);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (r + k < r1) {
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += v[k][j];
            }
    }
    store8(part + (size_t)blockIdx.y * N + c, acc);
}

hipError_t colsum_partials(int dtype, const void *in, int T, int N, int ld, float *part, hipStream_t st) {
    if (T == 0 || N == 0) return hipSuccess;
    dim3 grid(ceil_div(N, 2048), colsum_slabs(T));
    if (dtype == DT_F32) colsum_kernel<float><<<grid, 256, 0, st>>>((const float *)in, T, N, ld, colsum_rows(T), part);
    else colsum_kernel<bf16_t><<<grid, 256, 0, st>>>((const bf16_t *)in, T, N, ld, colsum_rows(T), part);
    return hipGetLastError();
}

// ---- rotary embedding, in place ------------------------------------------------------
// Heads [0, n_rot_heads) of every row (the q heads then the k heads) are rotated on the pair
// (i, i + d/2) by the tabulated angle of the token's position in its segment.  inverse = the
// transposed rotation (backward pass).
template <typename T>
__global__ __launch_bounds__(256) void rope_kernel(T *__restrict__ qkv, int ld, int ntok, int n_rot_heads, int d,
                                                   const float2 *__restrict__ cs, float sgn) {
    const int half = d >> 1, cpp = half >> 3;                    // 8-wide chunks per half head
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    const long total = (long)ntok * n_rot_heads * cpp;
    if (idx >= total) return;
    const int ch = (int)(idx % cpp);
    const int h = (int)((idx / cpp) % n_rot_heads);
    const long t = idx / ((long)cpp * n_rot_heads);
    T *p = qkv + t * ld + h * d + ch * 8;
    float lo[8], hi[8];
    load8(p, lo);
    load8(p + half, hi);
    const float2 *c = cs + t * half + ch * 8;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float co = c[j].x, si = sgn * c[j].y;
        const float a = lo[j] * co - hi[j] * si, b = hi[j] * co + lo[j] * si;
        lo[j] = a; hi[j] = b;
    }
    store8(p, lo);
    store8(p + half, hi);
}

hipError_t rope_inplace(int dtype, void *qkv, int ld, int T, int n_rot_heads, int d, const float2 *rope_cs,
                        bool inverse, hipStream_t st) {
    const long total = (long)T * n_rot_heads * (d / 16);
    if (total == 0) return hipSuccess;
    const float sgn = inverse ? -1.f : 1.f;
    if (dtype == DT_F32) rope_kernel<float><<<ceil_div(total, 256), 256, 0, st>>>((float *)qkv, ld, T, n_rot_heads, d, rope_cs, sgn);
    else rope_kernel<bf16_t><<<ceil_div(total, 256), 256, 0, st>>>((bf16_t *)qkv, ld, T, n_rot_heads, d, rope_cs, sgn);
    return hipGetLastError();
}

// ---- SwiGLU --------------------------------------------------------------------------
// gu[T, 2F] = [gate | up];  m = gate * sigmoid(gate) * up.
template <typename T>
__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const T *__restrict__ gu, T *__restrict__ m, long nchunks, int F) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= nchunks) return;
    const int cpr = F >> 3;
    const long t = idx / cpr;
    const int c = (int)(idx % cpr) * 8;
    float g[8], u[8];
    load8_stream(gu + t * 2 * F + c, g);
    load8_stream(gu + t * 2 * F + F + c, u);
#pragma unroll
    for (int j = 0; j < 8; ++j) g[j] = g[j] * sigmoid_fast(g[j]) * u[j];
    store8_stream(m + t * F + c, g);
}

template <typename T>
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const T *__restrict__ d_m, const T *__restrict__ gu,
                                                         T *__restrict__ d_gu, long nchunks, int F) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= nchunks) return;
    const int cpr = F >> 3;
    const long t = idx / cpr;
    const int c = (int)(idx % cpr) * 8;
    float g[8], u[8], dm[8];
    load8_stream(gu + t * 2 * F + c, g);
    load8_stream(gu + t * 2 * F + F + c, u);
    load8_stream(d_m + t * F + c, dm);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float2 d = swiglu_gradient(dm[j], g[j], u[j]);
        g[j] = d.x;
        u[j] = d.y;
    }
    store8_stream(d_gu + t * 2 * F + c, g);
    store8_stream(d_gu + t * 2 * F + F + c, u);
}

hipError_t swiglu_fwd(int dtype, const void *gu, void *m, int T, int F, hipStream_t st) {
    const long n = (long)T * (F / 8);
    if (n == 0) return hipSuccess;
    if (dtype == DT_F32) swiglu_fwd_kernel<float><<<ceil_div(n, 256), 256, 0, st>>>((const float *)gu, (float *)m, n, F);
    else swiglu_fwd_kernel<bf16_t><<<ceil_div(n, 256), 256, 0, st>>>((const bf16_t *)gu, (bf16_t *)m, n, F);
    return hipGetLastError();
}
hipError_t swiglu_bwd(int dtype, const void *d_m, const void *gu, void *d_gu, int T, int F, hipStream_t st) {
    const long n = (long)T * (F / 8);
    if (n == 0) return hipSuccess;
    if (dtype == DT_F32) swiglu_bwd_kernel<float><<<ceil_div(n, 256), 256, 0, st>>>((const float *)d_m, (const float *)gu, (float *)d_gu, n, F);
    else swiglu_bwd_kernel<bf16_t><<<ceil_div(n, 256), 256, 0, st>>>((const bf16_t *)d_m, (const bf16_t *)gu, (bf16_t *)d_gu, n, F);
    return hipGetLastError();
}

// ---- GELU (erf form) -----------------------------------------------------------------
// Phi(v) and phi(v) of the standard normal distribution.  The library erff costs some forty vector instructions, which
// made these kernels bound by the vector ALUs (GELU backward ran at 3.6 TB/s); this is the five-term rational
// approximation of Abramowitz & Stegun 7.1.26, erf(x) = 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p x), x >= 0,
// absolute error 1.5e-7, whose exponential exp(-v^2 / 2) is phi's as well: a dozen instructions for both.  In fp32
// arithmetic Phi comes out within 3e-7 (absolute; an fp32 rounding of a value near 1 is 6e-8).
__device__ __forceinline__ void normal_cdf_pdf(float v, float &cdf, float &pdf) {
    const float e = __builtin_amdgcn_exp2f(v * v * -0.72134752044448170f);            // exp(-v^2 / 2)
    const float t = __builtin_amdgcn_rcpf(fmaf(0.23164189f, fabsf(v), 1.f));              // p / sqrt(2) = 0.3275911 / 1.41421356
    const float poly = ((((1.061405429f * t - 1.453152027f) * t + 1.421413741f) * t - 0.284496736f) * t + 0.254829592f) * t;
    const float h = 0.5f * poly * e;                                                     // the smaller tail
    cdf = v >= 0.f ? 1.f - h : h;
    pdf = 0.3989422804014327f * e;
}
template <typename T>
__global__ __launch_bounds__(256) void gelu_fwd_kernel(const T *__restrict__ z, T *__restrict__ a, long nchunks) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= nchunks) return;
    float v[8];
    load8(z + idx * 8, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float cdf, pdf;
        normal_cdf_pdf(v[j], cdf, pdf);
        v[j] *= cdf;
    }
    store8(a + idx * 8, v);
}
// gelu'(z) = Phi(z) + z * phi(z)
template <typename T>
__global__ __launch_bounds__(256) void gelu_bwd_kernel(const T *__restrict__ d_a, const T *__restrict__ z,
                                                       T *__restrict__ d_z, long nchunks) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= nchunks) return;
    float v[8], g[8];
    load8(z + idx * 8, v);
    load8(d_a + idx * 8, g);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float cdf, pdf;
        normal_cdf_pdf(v[j], cdf, pdf);
        v[j] = g[j] * (cdf + v[j] * pdf);
    }
    store8(d_z + idx * 8, v);
}

// The same over [nrows, N] with the column sums of d_z (the bias gradient of the linear in front of the activation):
// a thread owns 8 columns of a slab of rows; part[slab, N] receives the slab's sums.
template <typename T>
__global__ __launch_bounds__(256) void gelu_bwd_colsum_kernel(const T *__restrict__ d_a, const T *__restrict__ z,
                                                              T *__restrict__ d_z, int nrows, int N, int slab,
                                                              float *__restrict__ part) {
    const int c = (blockIdx.x * 256 + threadIdx.x) * 8;
    if (c >= N) return;
    const int r0 = blockIdx.y * slab, r1 = min(nrows, r0 + slab);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int r = r0; r < r1; r += 4) {
        float v[4][8], g[4][8];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (r + k < r1) { load8(z + (size_t)(r + k) * N + c, v[k]); load8(d_a + (size_t)(r + k) * N + c, g[k]); }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (r + k < r1) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    float cdf, pdf;
                    normal_cdf_pdf(v[k][j], cdf, pdf);
                    v[k][j] = g[k][j] * (cdf + v[k][j] * pdf);
                }
                store8(d_z + (size_t)(r + k) * N + c, v[k]);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += v[k][j];
            }
    }
    store8(part + (size_t)blockIdx.y * N + c, acc);
}

hipError_t gelu_fwd(int dtype, const void *z, void *a, long n, hipStream_t st) {
    const long nc = n / 8;
    if (nc == 0) return hipSuccess;
    if (dtype == DT_F32) gelu_fwd_kernel<float><<<ceil_div(nc, 256), 256, 0, st>>>((const float *)z, (float *)a, nc);
    else gelu_fwd_kernel<bf16_t><<<ceil_div(nc, 256), 256, 0, st>>>((const bf16_t *)z, (bf16_t *)a, nc);
    return hipGetLastError();
}
hipError_t gelu_bwd_colsum(int dtype, const void *d_a, const void *z, void *d_z, int T, int N, float *part, hipStream_t st) {
    if (T == 0 || N == 0) return hipSuccess;
    dim3 grid(ceil_div(N, 2048), colsum_slabs(T));
    if (dtype == DT_F32) gelu_bwd_colsum_kernel<float><<<grid, 256, 0, st>>>((const float *)d_a, (const float *)z, (float *)d_z, T, N, colsum_rows(T), part);
    else gelu_bwd_colsum_kernel<bf16_t><<<grid, 256, 0, st>>>((const bf16_t *)d_a, (const bf16_t *)z, (bf16_t *)d_z, T, N, colsum_rows(T), part);
    return hipGetLastError();
}
hipError_t gelu_bwd(int dtype, const void *d_a, const void *z, void *d_z, long n, hipStream_t st) {
    const long nc = n / 8;
    if (nc == 0) return hipSuccess;
    if (dtype == DT_F32) gelu_bwd_kernel<float><<<ceil_div(nc, 256), 256, 0, st>>>((const float *)d_a, (const float *)z, (float *)d_z, nc);
    else gelu_bwd_kernel<bf16_t><<<ceil_div(nc, 256), 256, 0, st>>>((const bf16_t *)d_a, (const bf16_t *)z, (bf16_t *)d_z, nc);
    return hipGetLastError();
}

// ---- zeros (the gradients of an empty pack) --------------------------------------------
__global__ void fill_zero_kernel(uint32_t *p, size_t nwords) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nwords) p[i] = 0u;
}
hipError_t fill_zero(void *p, size_t elems, int dtype, hipStream_t st) {
    if (!p || elems == 0) return hipSuccess;
    const size_t bytes = elems * (dtype == DT_F32 ? 4 : 2);
    const size_t words = bytes / 4;            // all parameter tensors have an even element count
    fill_zero_kernel<<<ceil_div((long)words, 256), 256, 0, st>>>((uint32_t *)p, words);
    return hipGetLastError();
}

}  // namespace mmt
