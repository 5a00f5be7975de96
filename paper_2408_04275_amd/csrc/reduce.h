// Sums of the rows of fp32 arrays: what a backward pass leaves behind as partial sums.
#pragma once
#include "kernels.h"

namespace mmt {

// Up to eight reductions of different shapes: gain and bias gradients of both normalisations, the bias gradients of the four linears.
// They are added up together at the end of the pass instead of by one launch where each array is produced.  A unit of work is 32
// columns of one array; units[j] .. units[j + 1] - 1 belong to array j.
struct ReduceJobSet {
    const float *part[8];
    void *out[8];
    int rows[8], N[8], units[9];
    int accumulate;
};
// false: nothing to reduce, or an array whose rows are not whole quads
bool reduce_job_set(const ReduceJob *jobs, int n, bool accumulate, ReduceJobSet &set);

constexpr int REDUCE_LDS = 32 * 36 * 4;
// one unit, by 256 threads of a workgroup (tid); red: REDUCE_LDS bytes; has a barrier
template <typename T>
__device__ __forceinline__ void reduce_unit(const ReduceJobSet &set, int unit, float (*red)[36], int tid) {
    int j = 0;
#pragma unroll
    for (int i = 1; i < 8; ++i) j += unit >= set.units[i];
    const int N = set.N[j], rows = set.rows[j], c0 = (unit - set.units[j]) * 32;
    const float *part = set.part[j];
    T *out = (T *)set.out[j];
    const int cl = tid & 7, rl = tid >> 3;
    const int c = c0 + cl * 4;
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
    const int oc = c0 + tid;
    if (tid < 32 && oc < N) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < 32; ++i) t += red[i][tid];
        if (set.accumulate) t += Elem<T>::load(out + oc);
        Elem<T>::store(out + oc, t);
    }
}

}  // namespace mmt
