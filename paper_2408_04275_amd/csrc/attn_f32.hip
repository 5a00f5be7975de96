// Segment-masked attention, forward and backward, on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32): the fp32 storage
// path.  fp32 products, fp32 accumulation, the library's expf: the arithmetic of the vector-ALU kernels in another order.
//
// The fp32 packs are small (512 tokens, 4 heads), so latency bounds these kernels.  A workgroup owns 16 queries (forward, dQ)
// or 16 keys (dK/dV) of one head; its wavefronts share out the 16-row blocks of the other side (times the query heads of
// the group, dK/dV) and their partial results are combined through LDS in a fixed order.  One wavefront per (token, head) and
// one key at a time, as before, took 57 / 58 / 47 us (forward / dQ / dK,dV) on that pack.
//
// As in the bf16 kernels the score tile is [streamed rows x owned rows]: a lane holds one owned row (lane & 15) and the four
// streamed rows 4 (lane >> 4) .. + 3, so P and dS are already the column operand of the product that contracts over the
// streamed rows -- MFMA j of such a product takes the streamed rows 4 (lane >> 4) + j.  Operands come straight from global
// memory in two forms: a row's 16-byte pieces where the features are contracted (feature 16 b + 4 (lane >> 4) + j for MFMA j),
// four neighbouring features of a row where they are the result's rows (fragment 4 c + f holds features 64 c + 4 x + f).
//
// A streamed row that an owned row may not see must not reach it, not even as 0 * NaN: blocks that are partly masked check the
// rows they are about to multiply and take a select per element if one of them is not finite.
#include "kernels.h"

namespace mmt {

namespace {

constexpr int END_MASK = 0x3fffffff;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)bytes, 0x00020000);
}
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
    return *reinterpret_cast<const f32x4 *>(&w);
}
__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// rows of a [T, ld] tensor as the kernels read them; rows at or beyond T read as zero
template <int D>
struct Tensor {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t ld4, col4;                            // bytes per row; byte offset of the head's first feature
    __device__ __forceinline__ Tensor(const void *p, int T, int ld, int col)
        : rs(rsrc(p, (size_t)T * ld * 4)), ld4((uint32_t)ld * 4u), col4((uint32_t)col * 4u) {}
    // features contracted: row row0 + (lane & 15)
    __device__ __forceinline__ void pieces(int row0, f32x4 (&v)[D / 16]) const {
        const uint32_t o = (uint32_t)(row0 + (threadIdx.x & 15)) * ld4 + col4 + ((threadIdx.x & 48) >> 4) * 16u;
#pragma unroll
        for (int b = 0; b < D / 16; ++b) v[b] = load4(rs, o + 64u * b);
    }
    // rows contracted: rows row0 + 4 (lane >> 4) + j, features 64 c + 4 (lane & 15) ..
    __device__ __forceinline__ void columns(int row0, f32x4 (&v)[4][D / 64]) const {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t o = (uint32_t)(row0 + ((threadIdx.x & 48) >> 4) * 4 + j) * ld4 + col4 + (threadIdx.x & 15) * 16u;
#pragma unroll
            for (int c = 0; c < D / 64; ++c) v[j][c] = load4(rs, o + 256u * c);
        }
    }
};

// score-shaped product: [streamed row 4 (lane >> 4) + e][owned row lane & 15], contracted over the features
template <int D>
__device__ __forceinline__ f32x4 dot_rows(const f32x4 (&streamed)[D / 16], const f32x4 (&owned)[D / 16]) {
    f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};       // two chains: an MFMA's result is several cycles away
#pragma unroll
    for (int b = 0; b < D / 16; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j & 1] = mfma(streamed[b][j], owned[b][j], s[j & 1]);
    return s[0] + s[1];
}

// acc[feature][owned row] += sum over the 16 streamed rows of x[row][feature] * w[row][owned row].  `seen`: bit e set if the
// lane's owned row may see the streamed row 4 (lane >> 4) + e (its w is zero otherwise); partial: some lane has a bit clear.
template <int D>
__device__ __forceinline__ void add_rows(f32x4 (&acc)[D / 16], const f32x4 (&x)[4][D / 64], const f32x4 &w, uint32_t seen, bool partial) {
    if (partial) {
        float t = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < D / 64; ++c)
#pragma unroll
                for (int f = 0; f < 4; ++f) t += x[j][c][f] * 0.f;
        if (__any(t != 0.f)) {                     // an infinity or NaN among the rows (t is NaN then)
            const int r = threadIdx.x & 15, q = (threadIdx.x & 48) >> 4;
            for (int g = 0; g < 4; ++g) {
                const uint32_t bits = __shfl(seen, 16 * g + r, 64);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float wj = __shfl(w[j], 16 * g + r, 64);
                    // acc[4 c + f][e] is feature 64 c + 4 (4 q + e) + f: lane 16 g + 4 q + e holds it of row 4 g + j
#pragma unroll
                    for (int c = 0; c < D / 64; ++c)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int f = 0; f < 4; ++f) {
                                const float v = __shfl(x[j][c][f], 16 * g + 4 * q + e, 64);
                                if ((bits >> j) & 1) acc[4 * c + f][e] += wj * v;
                            }
                }
            }
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
#pragma unroll
            for (int f = 0; f < 4; ++f) acc[4 * c + f] = mfma(x[j][c][f], w[j], acc[4 * c + f]);
}

template <int D, int NW>
struct Partials {                                  // the wavefronts' [16 owned rows][D] results
    static constexpr int PITCH = D + 4;
    float v[NW][16][PITCH];
    __device__ __forceinline__ void put(int wave, const f32x4 (&acc)[D / 16]) {
        const int r = threadIdx.x & 15, q = (threadIdx.x & 48) >> 4;
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *reinterpret_cast<f32x4 *>(&v[wave][r][64 * c + 16 * q + 4 * e]) =
                    f32x4{acc[4 * c][e], acc[4 * c + 1][e], acc[4 * c + 2][e], acc[4 * c + 3][e]};
    }
    __device__ __forceinline__ f32x4 sum(int row, int col) const {
        f32x4 s = *reinterpret_cast<const f32x4 *>(&v[0][row][col]);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *reinterpret_cast<const f32x4 *>(&v[w][row][col]);
        return s;
    }
    // the sums times `scale` into rows row0 .. of out (row length ld); cs: rotate back by the rows' angles ([T, D / 2] cos, sin)
    __device__ __forceinline__ void store(float *out, int ld, int row0, int T, float scale, const float2 *cs) const {
        if (!cs) {
            for (int i = threadIdx.x; i < 16 * D / 4; i += 64 * NW) {
                const int row = i / (D / 4), col = i % (D / 4) * 4;
                if (row0 + row < T) *reinterpret_cast<f32x4 *>(out + (size_t)(row0 + row) * ld + col) = sum(row, col) * scale;
            }
            return;
        }
        for (int i = threadIdx.x; i < 16 * D / 8; i += 64 * NW) {
            const int row = i / (D / 8), col = i % (D / 8) * 4;
            if (row0 + row >= T) continue;
            const f32x4 lo = sum(row, col) * scale, hi = sum(row, col + D / 2) * scale;
            const float2 *a = cs + (size_t)(row0 + row) * (D / 2) + col;
            f32x4 x, y;
#pragma unroll
            for (int e = 0; e < 4; ++e) { x[e] = lo[e] * a[e].x + hi[e] * a[e].y; y[e] = hi[e] * a[e].x - lo[e] * a[e].y; }
            *reinterpret_cast<f32x4 *>(out + (size_t)(row0 + row) * ld + col) = x;
            *reinterpret_cast<f32x4 *>(out + (size_t)(row0 + row) * ld + col + D / 2) = y;
        }
    }
};

struct Range { int lo, hi; };                      // streamed rows an owned row may see
__device__ __forceinline__ Range keys_of(const int2 *info, int q, int T) {
    if (q >= T) return {0, 0};
    const int2 v = info[q];
    return {v.x, (v.y >> 30) ? (v.y & END_MASK) : q + 1};
}
__device__ __forceinline__ Range queries_of(const int2 *info, int k, int T) {
    if (k >= T) return {0, 0};
    const int2 v = info[k];
    return {(v.y >> 30) ? v.x : k, v.y & END_MASK};
}
__device__ __forceinline__ uint32_t seen_bits(const Range &me, int row0) {
    const int k = row0 + ((threadIdx.x & 48) >> 4) * 4;
    uint32_t b = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) b |= (k + e >= me.lo && k + e < me.hi ? 1u : 0u) << e;
    return b;
}

// a lane's value for its owned row: combined over the four lanes that hold that row
__device__ __forceinline__ float row_sum(float v) { v += __shfl_xor(v, 16, 64); return v + __shfl_xor(v, 32, 64); }
__device__ __forceinline__ float row_max(float v) { v = fmaxf(v, __shfl_xor(v, 16, 64)); return fmaxf(v, __shfl_xor(v, 32, 64)); }

template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_fwd_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) Partials<D, NW> part;
    __shared__ float stat_m[NW][16], stat_l[NW][16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = threadIdx.x & 15;
    const int q0 = blockIdx.x * 16, h = blockIdx.y, g = h / (a.nh / a.nkv), T = a.T, nq = a.nh * D, nk = a.nkv * D;
    const Tensor<D> Q(a.qkv, T, a.ld_qkv, h * D), K(a.qkv, T, a.ld_qkv, nq + g * D), V(a.qkv, T, a.ld_qkv, nq + nk + g * D);
    const Range me = keys_of(a.tok_info, q0 + r, T);
    const int kbeg = keys_of(a.tok_info, q0, T).lo, kend = keys_of(a.tok_info, min(q0 + 16, T) - 1, T).hi;   // monotonic bounds
    f32x4 qf[D / 16], acc[D / 16];
    Q.pieces(q0, qf);
#pragma unroll
    for (int i = 0; i < D / 16; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    for (int k0 = kbeg + 16 * wave; k0 < kend; k0 += 16 * NW) {
        f32x4 kf[D / 16], vf[4][D / 64];
        K.pieces(k0, kf);
        V.columns(k0, vf);
        const uint32_t seen = seen_bits(me, k0);
        f32x4 p = dot_rows<D>(kf, qf) * a.scale;
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) { if (!((seen >> e) & 1)) p[e] = -INFINITY; mx = fmaxf(mx, p[e]); }
        const float mn = fmaxf(m, row_max(mx)), base = mn == -INFINITY ? 0.f : mn, corr = expf(m - base);
        l *= corr;
#pragma unroll
        for (int e = 0; e < 4; ++e) { p[e] = expf(p[e] - base); l += p[e]; }
#pragma unroll
        for (int i = 0; i < D / 16; ++i) acc[i] *= corr;
        m = mn;
        add_rows<D>(acc, vf, p, seen, __any(seen != 15u));
    }
    l = row_sum(l);
    if (threadIdx.x % 64 < 16) { stat_m[wave][r] = m; stat_l[wave][r] = l; }
    __syncthreads();
    float top = stat_m[0][r], total = 0.f;
#pragma unroll
    for (int w = 1; w < NW; ++w) top = fmaxf(top, stat_m[w][r]);
    const float base = top == -INFINITY ? 0.f : top;
#pragma unroll
    for (int w = 0; w < NW; ++w) total += stat_l[w][r] * expf(stat_m[w][r] - base);
    const float f = expf(m - base) / total;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) acc[i] *= f;
    part.put(wave, acc);
    __syncthreads();
    part.store((float *)a.o + h * D, nq, q0, T, 1.f, nullptr);
    if (threadIdx.x < 16 && q0 + r < T) a.lse[(size_t)h * T + q0 + r] = base + logf(total);
}

// D_i = dO_i . O_i of the rows row0 + (lane & 15)
template <int D>
__device__ __forceinline__ float row_dots(const Tensor<D> &O, int row0, const f32x4 (&gf)[D / 16]) {
    f32x4 of[D / 16];
    O.pieces(row0, of);
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < D / 16; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) d += gf[i][e] * of[i][e];
    return row_sum(d);
}

// dQ_i = scale * sum_j dS_ij k_j,  dS_ij = P_ij (dO_i . v_j - D_i),  P_ij = exp(s_ij - lse_i).  KEEP_D: D goes to a.Dsum as well
template <int D, int NW, bool KEEP_D>
__device__ __forceinline__ void dq_rows(const AttnArgs &a, Partials<D, NW> &part, int h) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = threadIdx.x & 15;
    const int q0 = blockIdx.x * 16, g = h / (a.nh / a.nkv), T = a.T, nq = a.nh * D, nk = a.nkv * D;
    const Tensor<D> Q(a.qkv, T, a.ld_qkv, h * D), K(a.qkv, T, a.ld_qkv, nq + g * D), V(a.qkv, T, a.ld_qkv, nq + nk + g * D);
    const Tensor<D> dO(a.d_o, T, nq, h * D), O(a.o, T, nq, h * D);
    const Range me = keys_of(a.tok_info, q0 + r, T);
    const int kbeg = keys_of(a.tok_info, q0, T).lo, kend = keys_of(a.tok_info, min(q0 + 16, T) - 1, T).hi;
    f32x4 qf[D / 16], gf[D / 16], acc[D / 16];
    Q.pieces(q0, qf);
    dO.pieces(q0, gf);
#pragma unroll
    for (int i = 0; i < D / 16; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float Di = row_dots<D>(O, q0, gf);
    const float lse = q0 + r < T ? a.lse[(size_t)h * T + q0 + r] : 0.f;
    if (KEEP_D && threadIdx.x < 16 && q0 + r < T) a.Dsum[(size_t)h * T + q0 + r] = Di;
    for (int k0 = kbeg + 16 * wave; k0 < kend; k0 += 16 * NW) {
        f32x4 kf[D / 16], vf[D / 16], kc[4][D / 64];
        K.pieces(k0, kf);
        V.pieces(k0, vf);
        K.columns(k0, kc);
        const uint32_t seen = seen_bits(me, k0);
        const f32x4 s = dot_rows<D>(kf, qf) * a.scale, dp = dot_rows<D>(vf, gf);
        f32x4 ds;
#pragma unroll
        for (int e = 0; e < 4; ++e) ds[e] = (seen >> e) & 1 ? expf(s[e] - lse) * (dp[e] - Di) : 0.f;
        add_rows<D>(acc, kc, ds, seen, __any(seen != 15u));
    }
    part.put(wave, acc);
    __syncthreads();
    part.store((float *)a.d_qkv + h * D, a.ld_qkv, q0, T, a.scale, a.rope_cs);
}

// dK_j = scale * sum_{h in group} sum_i dS_ij q_i,   dV_j = sum_{h in group} sum_i P_ij dO_i.  KEPT_D: D is in a.Dsum; otherwise it is
// formed again for every block of keys, to the same bits
template <int D, int NW, bool KEPT_D>
__device__ __forceinline__ void dkv_rows(const AttnArgs &a, Partials<D, NW> &part, int g) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = threadIdx.x & 15, q4 = ((threadIdx.x & 48) >> 4) * 4;
    const int k0 = blockIdx.x * 16, group = a.nh / a.nkv, T = a.T, nq = a.nh * D, nk = a.nkv * D;
    const Tensor<D> K(a.qkv, T, a.ld_qkv, nq + g * D), V(a.qkv, T, a.ld_qkv, nq + nk + g * D);
    const Range me = queries_of(a.tok_info, k0 + r, T);
    const int qbeg = queries_of(a.tok_info, k0, T).lo, qend = queries_of(a.tok_info, min(k0 + 16, T) - 1, T).hi;
    f32x4 kf[D / 16], vf[D / 16], dk[D / 16], dv[D / 16];
    K.pieces(k0, kf);
    V.pieces(k0, vf);
#pragma unroll
    for (int i = 0; i < D / 16; ++i) dk[i] = dv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int blocks = (qend - qbeg + 15) / 16;
    for (int item = wave; item < blocks * group; item += NW) {
        const int h = g * group + item / blocks, q0 = qbeg + 16 * (item % blocks);
        const Tensor<D> Q(a.qkv, T, a.ld_qkv, h * D), dO(a.d_o, T, nq, h * D), O(a.o, T, nq, h * D);
        f32x4 qf[D / 16], gf[D / 16], qc[4][D / 64], gc[4][D / 64];
        Q.pieces(q0, qf);
        dO.pieces(q0, gf);
        Q.columns(q0, qc);
        dO.columns(q0, gc);
        f32x4 lse, Ds, p, ds;
#pragma unroll
        for (int e = 0; e < 4; ++e) lse[e] = a.lse[(size_t)h * T + min(q0 + q4 + e, T - 1)];
        if constexpr (KEPT_D) {
#pragma unroll
            for (int e = 0; e < 4; ++e) Ds[e] = a.Dsum[(size_t)h * T + min(q0 + q4 + e, T - 1)];
        } else {
            const float d = row_dots<D>(O, q0, gf);
#pragma unroll
            for (int e = 0; e < 4; ++e) Ds[e] = __shfl(d, q4 + e, 64);
        }
        const uint32_t seen = seen_bits(me, q0);
        const f32x4 s = dot_rows<D>(qf, kf) * a.scale, dp = dot_rows<D>(gf, vf);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            p[e] = (seen >> e) & 1 ? expf(s[e] - lse[e]) : 0.f;
            ds[e] = (seen >> e) & 1 ? p[e] * (dp[e] - Ds[e]) : 0.f;
        }
        const bool partial = __any(seen != 15u);
        add_rows<D>(dv, gc, p, seen, partial);
        add_rows<D>(dk, qc, ds, seen, partial);
    }
    float *out = (float *)a.d_qkv;
    part.put(wave, dk);
    __syncthreads();
    part.store(out + nq + g * D, a.ld_qkv, k0, T, a.scale, a.rope_cs);
    __syncthreads();
    part.put(wave, dv);
    __syncthreads();
    part.store(out + nq + nk + g * D, a.ld_qkv, k0, T, 1.f, nullptr);
}

// Both in one launch, the dK/dV workgroups (longer with grouped heads) first; see one_launch.  Rows first .. of the nkv + nh rows of
// workgroups (a grid holds 65535).
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_bwd_kernel(AttnArgs a, int first) {
    __shared__ __attribute__((aligned(16))) Partials<D, NW> part;
    const int y = first + blockIdx.y;
    if (y < a.nkv) dkv_rows<D, NW, false>(a, part, y);
    else dq_rows<D, NW, false>(a, part, y - a.nkv);
}
// ... or one after the other
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_dq_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) Partials<D, NW> part;
    dq_rows<D, NW, true>(a, part, blockIdx.y);
}
template <int D, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_dkv_kernel(AttnArgs a) {
    __shared__ __attribute__((aligned(16))) Partials<D, NW> part;
    dkv_rows<D, NW, true>(a, part, blockIdx.y);
}

}  // namespace

// 32-bit byte offsets, one grid row per head
bool attn_f32_supported(const AttnArgs &a) {
    return (a.d == 64 || a.d == 128) && ((size_t)a.T + 64) * a.ld_qkv * 4 < 0xfff00000ull && a.nh <= 65535;
}

// 64-wide heads: eight wavefronts; 128-wide ones: four, whose partial results are as large
hipError_t attn_f32_fwd(const AttnArgs &a, hipStream_t st) {
    if (a.T == 0) return hipSuccess;
    const dim3 grid(ceil_div(a.T, 16), a.nh);
    if (a.d == 64) attn_f32_fwd_kernel<64, 8><<<grid, 512, 0, st>>>(a);
    else attn_f32_fwd_kernel<128, 4><<<grid, 256, 0, st>>>(a);
    return hipGetLastError();
}

// One launch where dK/dV alone leaves the chip part empty: dQ fills it, and D from the rows at hand costs dK/dV one more read and spares it
// the wait for dQ (512 tokens and 4 heads of 64 in four segments, 128 workgroups: 18.1 -> 11.2 us).  With more workgroups of 64-wide heads
// that read is work on a full chip.  One launch against two, mean over 3 to 21 packs of one to eight segments each (dK/dV workgroups:
// ratio): 192: 0.88, 256: 0.96, 320: 0.87, 384: 0.90, 448: 0.97, 512: 1.05, 640: 0.99, 768: 1.01, 1024: 1.09; 16 heads, 8192 tokens in one
// segment 6547 us against 5679. Single packs scatter around these: of 273 the rule is 8 % faster on average than two launches, and seven
// are 2.5 % or more slower, 16 heads on 4 over 1019 tokens in eight segments (48.4 -> 55.9 us) the most. 128-wide heads, four wavefronts
// per workgroup, gain at every length (32 heads, 96 tokens 27.2 -> 22.8 us, 8192 38629 -> 36478).
constexpr long ONE_LAUNCH_WORKGROUPS = 448;
static bool one_launch(int T, int nkv, int d) { return d != 64 || (long)ceil_div(T, 16) * nkv <= ONE_LAUNCH_WORKGROUPS; }
int attn_f32_bwd_launches(int T, int nh, int nkv, int d) { return one_launch(T, nkv, d) ? ceil_div(nkv + nh, 65535) : 2; }

hipError_t attn_f32_bwd(const AttnArgs &a, hipStream_t st) {
    if (a.T == 0) return hipSuccess;
    const int blocks = ceil_div(a.T, 16);
    if (!one_launch(a.T, a.nkv, a.d)) {
        attn_f32_dq_kernel<64, 8><<<dim3(blocks, a.nh), 512, 0, st>>>(a);
        attn_f32_dkv_kernel<64, 8><<<dim3(blocks, a.nkv), 512, 0, st>>>(a);
        return hipGetLastError();
    }
    for (int first = 0, rows; (rows = a.nkv + a.nh - first) > 0; first += 65535) {
        const dim3 grid(blocks, rows < 65535 ? rows : 65535);
        if (a.d == 64) attn_f32_bwd_kernel<64, 8><<<grid, 512, 0, st>>>(a, first);
        else attn_f32_bwd_kernel<128, 4><<<grid, 256, 0, st>>>(a, first);
    }
    return hipGetLastError();
}

}  // namespace mmt
