// Optimizer step of mixed-precision training on one rank's shard of the parameters (ZeRO-1 gives every
// data-parallel rank 1/DP of the optimizer state): fp32 master weights and Adam moments, fp32 accumulated
// gradients, bf16 (or fp32) working copy of the weights written in the same pass.  Decoupled weight decay
// (AdamW).  Memory-bound: per element it reads 16 bytes and writes 12 + the working copy (+ 4 when the
// gradient is cleared for the next accumulation), 16 bytes per lane per access.
#include "kernels.h"

namespace mmt {

// Streaming pays where the arrays do not fit the memory-side cache (256 MB) together.  us, plain -> streaming, on repeated
// passes / after all inputs were written / after the gradient was / from HBM: 12.6 M elements with a bf16 copy (216 MiB)
// 62 -> 65 / 63 -> 68 / 71 -> 65 / 92 -> 82, 16.8 M (288 MiB) 88 -> 85 / 85 -> 89 / 90 -> 84 / 119 -> 109, 21.0 M (360 MiB)
// 135 -> 102 / 110 -> 108 / 117 -> 103 / 148 -> 127, 25.3 M 172 -> 124 / 144 -> 137 / 149 -> 124 / 174 -> 159, 41.9 M
// 281 -> 202 / 255 -> 227 / 256 -> 213 / 278 -> 260.  With the gradient's load nontemporal too it was behind plain accesses
// up to 33 M elements wherever an input was fresh (25.3 M: 152, 157).
bool adam_streams(size_t n, size_t param_bytes) { return n * (16 + param_bytes) >= (size_t)360 << 20; }

namespace {

__device__ __forceinline__ void update(float &w, float g, float &m, float &v, const AdamArgs &a) {
    const float gr = g * a.grad_scale;
    m = a.beta1 * m + a.omb1 * gr;
    v = a.beta2 * v + a.omb2 * gr * gr;
    const float upd = (m * a.inv_bias1) / (sqrtf(v * a.inv_bias2) + a.eps) + a.weight_decay * w;
    w -= a.lr * upd;
}

template <bool STREAM, typename V>
__device__ __forceinline__ V load(const float *p) {
    return STREAM ? __builtin_nontemporal_load(reinterpret_cast<const V *>(p)) : *reinterpret_cast<const V *>(p);
}
template <bool STREAM, typename V, typename T>
__device__ __forceinline__ void store(T *p, V v) {
    if (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<V *>(p));
    else *reinterpret_cast<V *>(p) = v;
}

// QUADS groups of four elements per thread, all requested before the first is updated.  STREAM: nontemporal accesses, except for
// the gradient's load: the backward pass has just written it, so the memory-side cache may still hold it.
template <typename TP, bool STREAM, int QUADS>
__global__ __launch_bounds__(256) void adam_kernel(size_t n, float *__restrict__ w, float *__restrict__ g,
                                                   float *__restrict__ m, float *__restrict__ v, TP *__restrict__ p,
                                                   AdamArgs a) {
    const size_t first = ((size_t)blockIdx.x * QUADS * 256 + threadIdx.x) * 4;
    f32x4 wv[QUADS], gv[QUADS], mv[QUADS], vv[QUADS];
#pragma unroll
    for (int k = 0; k < QUADS; ++k) {
        const size_t i = first + k * 1024;
        if (i + 4 > n) continue;
        wv[k] = load<STREAM, f32x4>(w + i); gv[k] = load<false, f32x4>(g + i);
        mv[k] = load<STREAM, f32x4>(m + i); vv[k] = load<STREAM, f32x4>(v + i);
    }
#pragma unroll
    for (int k = 0; k < QUADS; ++k) {
        const size_t i = first + k * 1024;
        if (i + 4 <= n) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float we = wv[k][e], me = mv[k][e], ve = vv[k][e];
                update(we, gv[k][e], me, ve, a);
                wv[k][e] = we; mv[k][e] = me; vv[k][e] = ve;
            }
            store<STREAM>(w + i, wv[k]);
            store<STREAM>(m + i, mv[k]);
            store<STREAM>(v + i, vv[k]);
            if (a.zero_grad) store<STREAM>(g + i, f32x4{0.f, 0.f, 0.f, 0.f});
            if (p) {
                if constexpr (sizeof(TP) == 2) store<STREAM>(p + i, u32x2{pack_bf16x2(wv[k][0], wv[k][1]), pack_bf16x2(wv[k][2], wv[k][3])});
                else store<STREAM>(p + i, wv[k]);
            }
        } else {
            for (size_t j = i; j < n; ++j) {
                float wj = w[j], mj = m[j], vj = v[j];
                update(wj, g[j], mj, vj, a);
                w[j] = wj; m[j] = mj; v[j] = vj;
                if (a.zero_grad) g[j] = 0.f;
                if (p) Elem<TP>::store(p + j, wj);
            }
        }
    }
}

template <typename TP>
hipError_t launch(size_t n, float *w, float *g, float *m, float *v, TP *p, const AdamArgs &a, hipStream_t st) {
    if (adam_streams(n, p ? sizeof(TP) : 0)) adam_kernel<TP, true, 2><<<(unsigned)((n + 2047) / 2048), 256, 0, st>>>(n, w, g, m, v, p, a);
    else adam_kernel<TP, false, 1><<<(unsigned)((n + 1023) / 1024), 256, 0, st>>>(n, w, g, m, v, p, a);
    return hipGetLastError();
}

}  // namespace

hipError_t adam_step(int param_dtype, size_t n, float *w, float *g, float *m, float *v, void *p, const AdamArgs &a,
                     hipStream_t st) {
    if (n == 0) return hipSuccess;
    return param_dtype == DT_F32 ? launch(n, w, g, m, v, (float *)p, a, st) : launch(n, w, g, m, v, (bf16_t *)p, a, st);
}

}  // namespace mmt
