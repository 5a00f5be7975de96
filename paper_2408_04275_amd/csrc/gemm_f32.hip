// fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products, fp32 accumulation) for the fp32 storage path.
//
//   C[M,N] (+)= opA(A) . opB(B) (+ bias[N]) (+ residual[M,N])
//
// The fp32 layers are small (512 x 768 x 256), so what bounds a product is latency and how many compute units take part, not
// the matrix cores' rate.  A workgroup owns a 32 x 32 tile of C and its eight wavefronts take every eighth 16-deep block of K
// each: eight times the loads in flight and an eighth of the serial chain (four wavefronts with twice the look-ahead take 0 to
// 15 % longer).  Large products run in 64 x 64 tiles with four wavefronts.  The partial tiles are added through LDS in a fixed
// order.  512 x 768 x 256: 47.6 -> 7.3 us against the vector-ALU kernel; 512 x 256 x 1376: 257 -> 11.9 us.
//
// No operand goes through LDS: a fragment of the MFMA is 16 rows x 4 k, lane l holding row l & 15, k = l >> 4, and which k of
// a block an MFMA takes is free as long as both operands agree.  MFMA j of a block takes k = 4 (l >> 4) + j:
//   * K-contiguous operand: a lane's four k of a row are 16 contiguous bytes, one load for the block's four MFMAs;
//   * K-strided operand: a lane loads 2 or 4 neighbouring rows of one k, one load per MFMA; fragment f then holds the rows
//     (fragments) x (l & 15) + f, which only the epilogue has to know.
// Rows and k outside the matrix read as zero (the buffer descriptor's bounds check).
#include "kernels.h"
#include "reduce.h"

namespace mmt {

namespace {

struct GemmF32 {
    int M, N, K;
    const float *A; int lda;
    const float *B; int ldb;
    float *C; int ldc;
    const float *bias, *residual;
    int accumulate;
    // what an epilogue other than PLAIN needs
    float *extra;              // SWIGLU: [M, pair], silu(gate) up
    const float *gu;           // SWIGLU_BWD: [M, 2 N], gate and up side by side
    const float2 *cs;          // ROPE: [M, pair], cosine and sine
    int pair;                  // SWIGLU, ROPE: distance of the two columns that belong together
    int rotated;               // ROPE: heads that are rotated; those behind them are stored as they are
};
// Elementwise work on a product that its epilogue does, instead of a launch behind it.  A decoder layer forward and backward with the launch back,
// us, 256 features: 300, 512, 2048, 4096 tokens 104.4, 122.3, 309.6, 627.5 -> SwiGLU 106.4, 124.5, 313.4, 633.7; rotation 106.6, 124.5, 312.0, 632.3; SwiGLU's
// gradient 106.6, 124.6, 314.1, 633.7; the sums that ride along below 107.6, 125.9, 314.7, 633.1; all four 114.2, 132.5, 326.0, 648.0.  Each gained in every layer
// measured (256 to 1024 features, 96 to 4096 tokens).
//   SWIGLU      C = [gate | up], and silu(gate) up next to it.  A tile takes half of its columns from the gate and the same ones from up.
//   ROPE        the rotary embedding of heads of 2 pair features; a tile's columns are `half a tile` of a head's first half and their partners.
//   SWIGLU_BWD  the product is the gradient of silu(gate) up and is not stored: C = [d_gate | d_up], 2 N wide.
enum { PLAIN, SWIGLU, ROPE, SWIGLU_BWD };

constexpr uint32_t OOB = 0xfffffff0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)bytes, 0x00020000);
}

// One operand's fragments of a 16-deep K block: v[f][j] = fragment f's element for MFMA j.
template <int TB, bool KC>
struct Operand {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t off[KC ? TB : 4], step;
    int kq, K;
    // fragments TB / 2 .. of a K-contiguous operand: rows from row0 + second on
    __device__ __forceinline__ void init(const float *X, int ld, int row0, int nrows, int K_, int second = 8 * TB) {
        const int r = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
        K = K_;
        kq = 4 * q;
        if constexpr (KC) {
            rs = rsrc(X, ((size_t)(nrows - 1) * ld + K_) * 4);
            step = 64;
#pragma unroll
            for (int f = 0; f < TB; ++f) off[f] = (uint32_t)(((size_t)(row0 + (f < TB / 2 ? 0 : second) + 16 * (f % (TB / 2)) + r) * ld + kq) * 4);
        } else {
            rs = rsrc(X, ((size_t)(K_ - 1) * ld + nrows) * 4);
            step = (uint32_t)ld * 64u;
#pragma unroll
            for (int j = 0; j < 4; ++j) off[j] = (uint32_t)(((size_t)(kq + j) * ld + row0 + TB * r) * 4);
        }
    }
    __device__ __forceinline__ void load(int kb, float (&v)[TB][4]) const {
        const uint32_t base = (uint32_t)kb * step;
        if constexpr (KC) {
#pragma unroll
            for (int f = 0; f < TB; ++f) {
                const uint32_t o = kb * 16 + kq < K ? off[f] + base : OOB;
                const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o, 0, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[f][j] = __uint_as_float(w[j]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t o = kb * 16 + kq + j < K ? off[j] + base : OOB;
                if constexpr (TB == 4) {
                    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o, 0, 0);
#pragma unroll
                    for (int f = 0; f < 4; ++f) v[f][j] = __uint_as_float(w[f]);
                } else {
                    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, 0, 0);
#pragma unroll
                    for (int f = 0; f < 2; ++f) v[f][j] = __uint_as_float(w[f]);
                }
            }
        }
    }
};

// AHEAD: K blocks of a wavefront in flight while one is multiplied
template <int TB, int NW, int AHEAD, bool A_KC, bool B_KC, int EPI = PLAIN>
__device__ __forceinline__ void gemm_f32_tile(const GemmF32 &p, int n0, int m0) {
    constexpr int TILE = 16 * TB, PITCH = TILE + 4;
    constexpr bool PAIRED = EPI == SWIGLU || EPI == ROPE;
    constexpr int WIDTH = PAIRED ? TILE / 2 : TILE;             // columns that the epilogue walks over
    static_assert(!PAIRED || B_KC, "pairs are rows of a K-contiguous B");
    __shared__ __attribute__((aligned(16))) float red[NW / 2][TILE][PITCH];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, q = lane >> 4;
    Operand<TB, A_KC> la;
    Operand<TB, B_KC> lb;
    la.init(p.A, p.lda, m0, p.M, p.K);
    lb.init(p.B, p.ldb, n0, p.N, p.K, PAIRED ? p.pair : 8 * TB);

    f32x4 acc[TB][TB];
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // blocks wave, wave + NW, ... of K; those beyond the end read as zero
    const int nkb = (p.K + 15) / 16;
    float a[AHEAD][TB][4], b[AHEAD][TB][4];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) { la.load(wave + NW * s, a[s]); lb.load(wave + NW * s, b[s]); }
    for (int kb = wave; kb < nkb; kb += NW * AHEAD) {
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            // operands swapped: a lane holds four neighbouring columns of one row of C
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int fa = 0; fa < TB; ++fa)
#pragma unroll
                    for (int fb = 0; fb < TB; ++fb)
                        acc[fa][fb] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[s][fb][j], a[s][fa][j], acc[fa][fb], 0, 0, 0);
            la.load(kb + NW * (s + AHEAD), a[s]);
            lb.load(kb + NW * (s + AHEAD), b[s]);
        }
    }

    // what the epilogue reads besides the product, requested in front of the sum over the wavefronts
    constexpr int ITEMS = (TILE * WIDTH + 256 * NW - 1) / (256 * NW);
    f32x4 in[EPI == SWIGLU_BWD || EPI == ROPE ? ITEMS : 1][2];
    if constexpr (EPI == SWIGLU_BWD || EPI == ROPE) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int c = threadIdx.x + 64 * NW * i, row = c / (WIDTH / 4), m = m0 + row, n = n0 + c % (WIDTH / 4) * 4;
            in[i][0] = in[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (row >= TILE || m >= p.M || n >= p.N) continue;
            const float *at = EPI == ROPE ? reinterpret_cast<const float *>(p.cs + (size_t)m * p.pair + n % (2 * p.pair)) : p.gu + (size_t)m * 2 * p.N + n;
            in[i][0] = *reinterpret_cast<const f32x4 *>(at);
            in[i][1] = *reinterpret_cast<const f32x4 *>(at + (EPI == ROPE ? 4 : p.N));
        }
    }

    // sum of the wavefronts' partial tiles: the upper half is added to the lower until two are left, those in the epilogue
    auto row_of = [&](int fa) { return A_KC ? 16 * fa + r : TB * r + fa; };
    auto put = [&](float (&t)[TILE][PITCH]) {
#pragma unroll
        for (int fa = 0; fa < TB; ++fa)
#pragma unroll
            for (int fb = 0; fb < TB; ++fb) {
                if constexpr (B_KC) *reinterpret_cast<f32x4 *>(&t[row_of(fa)][16 * fb + 4 * q]) = acc[fa][fb];
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[row_of(fa)][TB * (4 * q + e) + fb] = acc[fa][fb][e];
                }
            }
    };
    if (wave >= NW / 2) put(red[wave - NW / 2]);
    __syncthreads();
#pragma unroll
    for (int left = NW / 2; left >= 2; left /= 2) {
        if (wave < left) {
            const int from = left == NW / 2 ? wave : wave + left;
#pragma unroll
            for (int fa = 0; fa < TB; ++fa)
#pragma unroll
                for (int fb = 0; fb < TB; ++fb) {
                    if constexpr (B_KC) acc[fa][fb] += *reinterpret_cast<const f32x4 *>(&red[from][row_of(fa)][16 * fb + 4 * q]);
                    else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[fa][fb][e] += red[from][row_of(fa)][TB * (4 * q + e) + fb];
                    }
                }
            if (left == 2 || wave >= left / 2) put(red[wave]);      // slot `wave` has been read by this wavefront alone
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int c = threadIdx.x + 64 * NW * i, row = c / (WIDTH / 4), col = c % (WIDTH / 4) * 4;
        const int m = m0 + row, n = n0 + col;
        if (row >= TILE || m >= p.M || n >= (EPI == SWIGLU ? p.pair : p.N)) continue;        // N is a multiple of 4
        auto sum = [&](int at) { return *reinterpret_cast<const f32x4 *>(&red[0][row][at]) + *reinterpret_cast<const f32x4 *>(&red[1][row][at]); };
        f32x4 v = sum(col);
        const size_t o = (size_t)m * p.ldc + n;
        if constexpr (EPI == PLAIN) {
            if (p.bias) v += *reinterpret_cast<const f32x4 *>(p.bias + n);
            if (p.residual) v += *reinterpret_cast<const f32x4 *>(p.residual + o);
            if (p.accumulate) v += *reinterpret_cast<const f32x4 *>(p.C + o);
            *reinterpret_cast<f32x4 *>(p.C + o) = v;
        } else if constexpr (EPI == SWIGLU_BWD) {
            f32x4 dg, du;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 d = swiglu_gradient(v[e], in[i][0][e], in[i][1][e]);
                dg[e] = d.x;
                du[e] = d.y;
            }
            *reinterpret_cast<f32x4 *>(p.C + o) = dg;
            *reinterpret_cast<f32x4 *>(p.C + o + p.N) = du;
        } else {
            f32x4 w = sum(col + TILE / 2);
            if constexpr (EPI == SWIGLU) {
                f32x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = v[e] * sigmoid_fast(v[e]) * w[e];
                *reinterpret_cast<f32x4 *>(p.extra + (size_t)m * p.pair + n) = x;
            } else if (n0 < p.rotated * 2 * p.pair) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float co = in[i][e >> 1][2 * (e & 1)], si = in[i][e >> 1][2 * (e & 1) + 1], lo = v[e], hi = w[e];
                    v[e] = lo * co - hi * si;
                    w[e] = hi * co + lo * si;
                }
            }
            *reinterpret_cast<f32x4 *>(p.C + o) = v;
            *reinterpret_cast<f32x4 *>(p.C + o + p.pair) = w;
        }
    }
}

template <int TB, int NW, int AHEAD, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmF32 p) {
    int n0 = blockIdx.x * 16 * TB;
    if constexpr (EPI == SWIGLU) n0 /= 2;
    if constexpr (EPI == ROPE) {                       // pair / (half a tile) tiles per head
        const int per_head = p.pair / (8 * TB), head = blockIdx.x / per_head;
        n0 = head * 2 * p.pair + (blockIdx.x - head * per_head) * 8 * TB;
    }
    gemm_f32_tile<TB, NW, AHEAD, A_KC, B_KC, EPI>(p, n0, blockIdx.y * 16 * TB);
}

// Several weight gradients in one launch: problem i has the workgroups [first[i], first[i + 1]), row by row of tiles.  Those behind the last one's
// add up sums that ride along, two units each: in a launch of their own these took 3.9 us at the end of a pass.
constexpr int MAX_GROUP = 4;
struct GroupF32 {
    GemmF32 p[MAX_GROUP];
    int first[MAX_GROUP + 1];
    ReduceJobSet reduce;
};
__global__ __launch_bounds__(512) void gemm_f32_group_kernel(GroupF32 g) {
    if ((int)blockIdx.x >= g.first[MAX_GROUP]) {
        __shared__ float sums[2][32][36];
        const int half = threadIdx.x >> 8;             // (a unit behind the last one has no columns)
        reduce_unit<float>(g.reduce, 2 * (blockIdx.x - g.first[MAX_GROUP]) + half, sums[half], threadIdx.x & 255);
        return;
    }
    int i = 0;
#pragma unroll
    for (int j = 1; j < MAX_GROUP; ++j) i += (int)blockIdx.x >= g.first[j] ? 1 : 0;
    const GemmF32 p = i == 0 ? g.p[0] : i == 1 ? g.p[1] : i == 2 ? g.p[2] : g.p[3];
    const int first = i == 0 ? 0 : i == 1 ? g.first[1] : i == 2 ? g.first[2] : g.first[3];
    const int tile = blockIdx.x - first, across = (p.N + 31) / 32;
    gemm_f32_tile<2, 8, 2, false, false>(p, tile % across * 32, tile / across * 32);
}

bool few_tiles(int M, int N) { return (long)ceil_div(M, 64) * ceil_div(N, 64) < 384; }

template <bool A_KC, bool B_KC, int EPI = PLAIN>
hipError_t launch(const GemmF32 &p, hipStream_t st) {
    // 64 x 64 tiles read half the operand bytes; they pay once there are enough of them (2048^3: 233 -> 150 us; 1024 x 2560 x
    // 512, 640 tiles: 43.5 -> 37.9; at 264 tiles both take 20 us; 512 x 256 x 688, 32 tiles: 7.0 -> 19.2)
    if (!few_tiles(p.M, p.N))
        gemm_f32_kernel<4, 4, 2, A_KC, B_KC, EPI><<<dim3(ceil_div(p.N, 64), ceil_div(p.M, 64)), 256, 0, st>>>(p);
    else
        gemm_f32_kernel<2, 8, 2, A_KC, B_KC, EPI><<<dim3(ceil_div(p.N, 32), ceil_div(p.M, 32)), 512, 0, st>>>(p);
    return hipGetLastError();
}

}  // namespace

// 16-byte accesses throughout: leading dimensions, N, and whatever index is contiguous in an operand multiples of 4, all
// pointers 16-byte aligned, 32-bit byte offsets.  A K of a few 16-deep blocks occupies only a few of a workgroup's wavefronts; where
// there are tiles enough for the vector-ALU kernel to fill the chip too, that one is ahead up to K = 64 (NN) and 80 (TN), us there ->
// here: NN 1352 x 3288 x 8 12.7 -> 17.0, 5652 x 3396 x 64 61 -> 69, x 72 ahead here; TN 772 x 2540 x 16 8.8 -> 15.2, 5504 x 1024 x 64 22 ->
// 30, 5652 x 3396 x 80 75 -> 82, x 96 ahead here (NT 1456 x 2408 x 8 10.9 -> 11.2).
bool gemm_f32_supported(const GemmArgs &g) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
    if (!few_tiles(g.M, g.N) && g.K < (g.layout == GEMM_TN ? 96 : g.layout == GEMM_NN ? 72 : 0)) return false;
    if ((g.lda | g.ldb | g.ldc | g.N) & 3) return false;
    const bool a_kc = g.layout != GEMM_TN, b_kc = g.layout == GEMM_NT;
    if ((a_kc || b_kc) && (g.K & 3)) return false;
    if (!a_kc && (g.M & 3)) return false;
    const size_t rows_a = a_kc ? g.M : g.K, rows_b = b_kc ? g.N : g.K;
    if ((rows_a + 256) * (size_t)g.lda * 4 >= 0xfff00000ull || (rows_b + 256) * (size_t)g.ldb * 4 >= 0xfff00000ull) return false;
    const uintptr_t bits = (uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C | (uintptr_t)g.bias | (uintptr_t)g.residual;
    return (bits & 15) == 0 && ceil_div(g.M, 32) <= 65535;
}

static GemmF32 params(const GemmArgs &g) {
    return {g.M, g.N, g.K, (const float *)g.A, g.lda, (const float *)g.B, g.ldb, (float *)g.C, g.ldc,
            (const float *)g.bias, (const float *)g.residual, g.accumulate ? 1 : 0, nullptr, nullptr, nullptr, 0, 0};
}

bool gemm_f32_few_tiles(const GemmArgs &g) { return g.layout == GEMM_TN && gemm_f32_supported(g) && few_tiles(g.M, g.N); }

// The weight gradients of a small layer together: 64 to 344 tiles each on the 512-token layer, 7.1 + 9.6 + 7.0 + 7.1 us one by one.
hipError_t gemm_f32_group(const GemmArgs *gs, int n, const ReduceJobSet *reduce, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (n > MAX_GROUP) return hipErrorInvalidValue;
    GroupF32 grp = {};
    int total = 0;
    for (int i = 0; i < MAX_GROUP; ++i) {
        grp.first[i] = total;
        if (i >= n) continue;
        if (!gemm_f32_few_tiles(gs[i])) return hipErrorInvalidValue;
        grp.p[i] = params(gs[i]);
        total += ceil_div(gs[i].M, 32) * ceil_div(gs[i].N, 32);
    }
    grp.first[MAX_GROUP] = total;
    if (reduce) grp.reduce = *reduce;
    gemm_f32_group_kernel<<<total + ceil_div(grp.reduce.units[8], 2), 512, 0, st>>>(grp);
    return hipGetLastError();
}

static bool product_alone(const GemmArgs &g) { return !g.bias && !g.residual && !g.accumulate && gemm_f32_supported(g); }

bool gemm_f32_swiglu_supported(const GemmArgs &g) { return g.layout == GEMM_NT && g.N % 8 == 0 && g.ldc == g.N && product_alone(g); }
hipError_t gemm_f32_swiglu(const GemmArgs &g, void *m, hipStream_t st) {
    GemmF32 p = params(g);
    p.extra = (float *)m; p.pair = g.N / 2;
    return launch<true, true, SWIGLU>(p, st);
}

// (heads of whole tiles, whichever size of tile is taken)
bool gemm_f32_rope_supported(const GemmArgs &g, int d) { return g.layout == GEMM_NT && d % 64 == 0 && g.N % d == 0 && product_alone(g); }
hipError_t gemm_f32_rope(const GemmArgs &g, int d, int rotated, const float2 *cs, hipStream_t st) {
    GemmF32 p = params(g);
    p.cs = cs; p.pair = d / 2; p.rotated = rotated;
    return launch<true, true, ROPE>(p, st);
}

bool gemm_f32_swiglu_bwd_supported(const GemmArgs &g) { return g.layout == GEMM_NN && g.ldc == 2 * g.N && product_alone(g); }
hipError_t gemm_f32_swiglu_bwd(const GemmArgs &g, const void *gu, hipStream_t st) {
    GemmF32 p = params(g);
    p.gu = (const float *)gu;
    return launch<true, false, SWIGLU_BWD>(p, st);
}

hipError_t gemm_f32(const GemmArgs &g, hipStream_t st) {
    const GemmF32 p = params(g);
    switch (g.layout) {
        case GEMM_NT: return launch<true, true>(p, st);
        case GEMM_NN: return launch<true, false>(p, st);
        default: return launch<false, false>(p, st);
    }
}

}  // namespace mmt
