// Segment-masked flash attention on the gfx950 matrix cores (bf16 in, fp32 accumulate),
// forward and backward, for packed variable-length segments.
//
// Tiling is on the GLOBAL token index, not per segment: a workgroup owns a run of consecutive queries
// (256 or 128 in the forward and dQ kernels, one query per lane of 8 or 4 wavefronts; both lane halves of a wavefront
// mirror the same 32 queries) or keys (128 in the dK/dV kernel).  Every query carries its own key range
// [lo, hi) = [segment start, causal ? q + 1 : segment end), so a tile may straddle any number of
// segment boundaries and a pack of many short segments still fills whole tiles.  The key loop of
// a workgroup runs over [lo(first query), hi(last query)) only: tiles that are fully masked for
// the workgroup are never loaded, and 32-key blocks that are fully masked for one wavefront are
// skipped by that wavefront (causal lower triangle, other segments).  The tiles of a launch differ a lot
// in work (a query tile at the end of a long causal segment walks many more keys than one at its start):
// they are dispatched heaviest first, with the head index fastest, from a table the host computes
// (longest-first scheduling as in the paper's Algorithm 1, applied to the GPU's work items).
//
// All score tiles are computed TRANSPOSED (keys x queries): S^T = K . Q^T with the MFMA's row
// operand = keys and column operand = queries.  A lane then holds 16 keys of ONE query per
// 32-key block, so the softmax row reductions are in-lane plus one cross-half exchange, the
// running max / sum / log-sum-exp / D are per-lane scalars, and P^T (or dS^T) is already laid
// out as the column operand of the next MFMA: O^T = V^T . P^T, dQ^T = K^T . dS^T.  The row
// operand of those products is the K or V tile transposed ([feature][key]), its keys in the order in
// which the accumulator registers hold them: all kernels keep the tiles row-major in LDS, as they are copied, and form
// the transposed fragments with the transposing LDS read.
//
// The backward pass is two kernels: dQ (same roles as forward; also writes -D, D = rowsum(dO * O), for the second),
// then dK/dV with one KEY per lane, looping over the query tiles that can see the workgroup's
// keys and over the query heads of the key/value head's group, so grouped-query gradients are
// summed in registers and nothing needs atomics: results are deterministic.  The dK/dV kernel has two forms: for
// heads wider than 64 features one in which two wavefronts share the work on their keys (scores and softmax, products),
// for 64-wide heads a plain one that leaves room for two workgroups per compute unit.
//
// Head dimensions: tiles in LDS are 64 or 128 features wide; a head of another width (a multiple of 16, e.g. 80) uses the
// next wider ones with the missing features read as zero and never stored.  Template parameters: D the tiles' width, KS the
// 16-feature slices that scores are contracted over, CB the 32-feature blocks of a result; heads of up to 80 and 96
// features have kernels that leave the zero slices and blocks out (80: 5 of 8 and 3 of 4, 11 MFMAs per 32 x 32 block
// instead of 16 forward, 16 of 24 in dQ, 22 of 32 in dK/dV).
#include "kernels.h"
#include <atomic>
#include <algorithm>
#include <type_traits>
#include <utility>

namespace mmt {

namespace {

constexpr int BQ = 128;        // keys per workgroup of the dK/dV kernel
constexpr int END_MASK = 0x3fffffff;
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// Swizzle of the 16-byte units of a tile row in LDS: unit u of row `row` stands at position u ^ swz_unit<D>(row).
// What it has to achieve was measured with a microbenchmark of LDS read patterns: a 16-byte-per-lane read is served
// 16 lanes at a time, lanes 0-7 together with 24-31, 8-15 with 16-23 (and the same in the upper half), an 8-byte
// transposing read 32 lanes at a time, lanes 0-31 and 32-63, each at full rate when its lanes fall into distinct slots modulo 256
// bytes.  A fragment read covers 32 consecutive rows at one unit: rows 0-7 and 24-31 have to differ, and rows 8-23.  A transposing
// read covers, with half a wavefront, four consecutive rows at four consecutive units (8 bytes a lane): the four rows have to differ in
// the unit bits above the lowest two.  With 256-byte rows (D = 128) the row's two lowest bits go there and its next two below them;
// with 128-byte rows (D = 64) the lowest bit is in the address as it is.  (With the lowest bit alone above, half of the lanes of a
// transposing read were served at a time, and LDS was what the dK/dV kernel waited for.)
template <int D>
__device__ __forceinline__ int swz_unit(int row) {
    if constexpr (D == 128) return (row & 2) << 2 | (row & 1) << 2 | (row >> 1 & 2) | (row >> 3 & 1);
    else return (row & 2) << 1 | (row >> 1 & 2) | (row >> 3 & 1);
}

__device__ __forceinline__ bf16x8 pack8(const float *v) {
    bf16x8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = (__bf16)v[i];
    return r;
}

__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    return z;
}

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

// The same MFMA written as assembly, with its result in VECTOR registers and its column operand in ACCUMULATION registers.
// In a kernel that needs more than 256 registers the compiler gives every MFMA builtin an accumulation-register result,
// and a result the vector ALU reads next (a score) then costs one copy instruction per element; operands that only MFMAs
// read (a wavefront's own K and V rows) can live in the accumulation half instead.  The compiler does not know what
// these statements are: whoever uses them keeps a result away from the vector ALU until the MFMA has retired
// (mfma_results_settle, or enough other work in between), and never lets two of them in a row depend on each other's result.
__device__ __forceinline__ void mfma_v_first(f32x16 &acc, const bf16x8 &rows, const bf16x8 &cols_acc) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(rows), "a"(cols_acc));
}
__device__ __forceinline__ void mfma_v(f32x16 &acc, const bf16x8 &rows, const bf16x8 &cols_acc) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(rows), "a"(cols_acc));
}
// more wait states than the eight passes of the MFMA above plus its write-back take
__device__ __forceinline__ void mfma_results_settle() { asm volatile("s_nop 15\n\ts_nop 7" ::: "memory"); }


// Per-compute-unit busy time (measurement aid): a workgroup adds its run time, in ticks of the constant 100 MHz
// counter, to the entry of the compute unit it ran on: minus the time at its start, plus the time at its end
// (unsigned wrap-around), so that nothing has to be kept in a register in between.
__device__ __forceinline__ void add_busy(unsigned long long *row, bool end) {
    if (row && threadIdx.x == 0) {
        const unsigned long long t = wall_clock64();
        atomicAdd(row + (__smid() & 1023u), end ? t : 0ull - t);
    }
}

struct RowInfo { int lo, hi; };   // allowed partner range of one token

// Smallest and largest range bounds over the 32 consecutive tokens base .. base + 31 that a wavefront holds one per
// lane (lanes 32 .. 63 repeat them), as scalars.  Both bounds are non-decreasing in the token index (segments follow
// one another in the pack; a causal bound moves with the token), so the first and the last token in range have them.
// No token in range: empty (lo_min = hi_min = INT_MAX, lo_max = hi_max = 0).
struct WaveBounds { int lo_min, lo_max, hi_min, hi_max; };
__device__ __forceinline__ WaveBounds wave_bounds(const RowInfo &me, int base, int T) {
    WaveBounds w = {0x7fffffff, 0, 0x7fffffff, 0};
    const int n = min(T - base, 32);
    if (n > 0) {
        w.lo_min = __builtin_amdgcn_readfirstlane(me.lo);
        w.hi_min = __builtin_amdgcn_readfirstlane(me.hi);
        w.lo_max = __builtin_amdgcn_readlane(me.lo, n - 1);
        w.hi_max = __builtin_amdgcn_readlane(me.hi, n - 1);
    }
    return w;
}

// Allowed partner ranges (KEYS: the queries that see a key; else the keys that a query sees) of this lane's token, one of the 32 from base
// on, and of the first and last of the workgroup's `rows` tokens from tile0 on.  Without the token table (AttnArgs::tok_info) they come from
// the segments themselves, one per lane: the same single trip to memory, and a call of attention alone saves the launch that fills the
// table (4.5 us; 64 heads on 8, 2047 tokens, forward and backward, where it stood twice: 220.5 -> 217.1).
template <bool KEYS>
__device__ __forceinline__ void ranges(const AttnArgs &a, int tile0, int rows, int base, RowInfo &me, RowInfo &first, RowInfo &last) {
    const int T = a.T, lane = threadIdx.x & 63, t = base + (lane & 31), end = min(tile0 + rows, T) - 1;
    int2 vm = {0, 0}, vf, vl;
    if (a.tok_info) {
        if (t < T) vm = a.tok_info[t];
        vf = a.tok_info[tile0];
        vl = a.tok_info[end];
    } else {
        int start = 0x7fffffff, info = 0;              // lane s: segment s
        if (lane < a.S) {
            start = a.cu[lane];
            info = a.cu[lane + 1] | ((a.modes ? (int)a.modes[lane] : a.default_mode) == MASK_BIDIR ? 1 << 30 : 0);
        }
        // the last segment that starts at or in front of token u (uniform)
        auto index = [&](int u) { return max(__popcll(__builtin_amdgcn_ballot_w64(start <= u)) - 1, 0); };
        auto segment = [&](int s) { return make_int2(__builtin_amdgcn_readlane(start, s), __builtin_amdgcn_readlane(info, s)); };
        vf = segment(index(tile0));
        vl = segment(index(end));
        const int to = index(base + 31);
        for (int s = index(base); s <= to; ++s) {
            const int2 v = segment(s);
            if (v.x <= t && t < T) vm = v;
        }
    }
    auto range = [&](const int2 &v, int u) {
        const bool bidir = v.y >> 30;
        RowInfo r = {0, 0};
        if (u < T) { r.lo = KEYS && !bidir ? u : v.x; r.hi = KEYS || bidir ? v.y & END_MASK : u + 1; }
        return r;
    };
    me = range(vm, t);
    first = range(vf, tile0);
    last = range(vl, end);
}

// ------------------------------------------------------------------------------------------
// shared pieces
// ------------------------------------------------------------------------------------------
constexpr int FQ = 256;         // queries per tile of the dispatch order of the forward and dQ kernels (8 wavefronts x 32)

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((ext_vector_type(4))) uint32_t rawx4;

__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// fragment of a row-major [rows][D] tile (row bytes 2 D): row, k-slice ks (16 features), lane half
template <int D>
__device__ __forceinline__ bf16x8 frag_k(const uint8_t *tile, int row, int ks, int half) {
    constexpr int UPR = D / 8;
    return *reinterpret_cast<const bf16x8 *>(tile + (row * UPR + ((ks * 2 + half) ^ swz_unit<D>(row))) * 16);
}

// ------------------------------------------------------------------------------------------
// backward
// ------------------------------------------------------------------------------------------
// Both backward kernels walk 64-row tiles that are copied global -> LDS directly, row-major ([row][D],
// 16-byte units XOR-swizzled by row), into two slots, the next tile being in flight while the current one
// is multiplied.  A product whose contraction runs over the tile's rows (dQ^T = K^T dS^T, dV^T = dO^T P,
// dK^T = Q^T dS) needs the tile transposed as its row operand; that fragment is formed from the same
// row-major tile by the transposing LDS read (ds_read_b64_tr_b16), with the rows taken in the order in
// which the accumulator registers of the score tile hold them.
constexpr int BT2 = 64;

typedef __attribute__((ext_vector_type(4))) short shortx4;
typedef __attribute__((ext_vector_type(8))) short shortx8;

// One wavefront's share of the copies of [64][D] tiles out of a row-major tensor: N copies of 1 KiB per tile, copy
// (first + i) of a tile covering its rows (first + i) * 512 / D ...  What depends on the lane is computed once
// (init); a copy then costs one addition.  Rows at or beyond the end of the tensor read as zero (the descriptor's
// bounds check), and so do the columns from row_elems on (a head narrower than the tile): their lanes carry an
// offset of 2 GiB, which no tensor reaches (the launchers check), and the sum with the offset of a tile that starts in front of the
// tensor's end cannot wrap.  The forward kernel's K tile may start up to 31 rows behind it: with rows of over 1024 elements and a tensor just under
// 2 GiB those columns wrap around to its first rows, which exist, and the scores of such keys are masked.
template <int D, int N>
struct RowCopier {
    static constexpr int UPR = D / 8, ROWS_PER_COPY = 1024 / (2 * D);
    uint32_t off[N];
    int first;
    __device__ __forceinline__ void init(int first_, long ld, int row_elems) {
        first = first_;
        const int lane = threadIdx.x & 63;
        const int lrow = lane / UPR, pos = lane % UPR;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int row = (first + i) * ROWS_PER_COPY + lrow;
            const int unit = pos ^ swz_unit<D>(row);
            off[i] = unit * 8 < row_elems ? (uint32_t)((row * ld + unit * 8) * 2) : 0x80000000u;
        }
    }
    // the tile whose first row is row0 and whose first column is col0 of the tensor rs describes (row length ld)
    __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, uint8_t *tile, long row0, long ld, long col0) const {
        const uint32_t base = (uint32_t)((row0 * ld + col0) * 2);
#pragma unroll
        for (int i = 0; i < N; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(tile + (first + i) * ROWS_PER_COPY * 2 * D), 16,
                                                     (int)(off[i] + base), 0, 0, 0);
    }
};
constexpr size_t MAX_TENSOR_BYTES = 0x7fff0000ull;      // what RowCopier's offsets allow

// Transposing reads.  Lane constants: 16-lane group gq = lane >> 4 forms the fragment rows (features)
// 16 (gq & 1) .. + 15 for lane half h = gq >> 1; as a source, lane j = lane & 15 of the group supplies
// the address of tile row 4 h + (j >> 2) (+ a multiple of 8), features 4 (j & 3) .. + 3 of the group's 16.
// off[2 C + SEC] holds that address for feature block C and the first or second 8 rows of 16, whose bit is in the swizzle.
template <int D>
struct TrReader {
    static constexpr int N = D / 16;
    uint32_t off[N];
    __device__ __forceinline__ void init(uint32_t lds_base) {
        const int lane = threadIdx.x & 63, gq = lane >> 4, j = lane & 15, qd = j & 3, t = j >> 2, h = gq >> 1;
        const int L = (2 * (gq & 1) + (qd >> 1)) ^ swz_unit<D>(4 * h + t);
#pragma unroll
        for (int x = 0; x < N; ++x) off[x] = lds_base + (4 * h + t) * 2 * D + (qd & 1) * 8 + ((L ^ (4 * (x >> 1)) ^ (x & 1)) << 4);
    }
    // half SEC (elements 4 SEC .. 4 SEC + 3) of the fragment of 32-row block B, MFMA M of the block, feature
    // block C of a tile at byte offset `tile` from lds_base: rows 32 B + 16 M + 8 SEC + 4 h + (0..3)
    template <int B, int M, int C, int SEC>
    __device__ __forceinline__ shortx4 read(uint32_t tile) const {
        shortx4 v;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(off[2 * C + SEC] + tile), "n"((32 * B + 16 * M + 8 * SEC) * 2 * D));
        return v;
    }
    // the same with the tile's offset already added to the addresses (base) and a constant offset on top
    template <int B, int M, int C, int SEC, int EXTRA>
    static __device__ __forceinline__ shortx4 read_at(const uint32_t (&base)[N]) {
        constexpr int IMM = (32 * B + 16 * M + 8 * SEC) * 2 * D + EXTRA;
        static_assert(IMM < 65536, "LDS offset field");
        shortx4 v;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(base[2 * C + SEC]), "n"(IMM));
        return v;
    }
};
__device__ __forceinline__ bf16x8 join(shortx4 lo, shortx4 hi) {
    const shortx8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return *reinterpret_cast<const bf16x8 *>(&v);
}
// The transposing reads are written as assembly because the compiler makes the builtin wait for every
// direct-to-LDS copy in flight; their results may be used only after this wait, which names them.
#define TR_WAIT4(x) "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])
#define TR_WAIT3(x) "+v"(x[0]), "+v"(x[1]), "+v"(x[2])
#define TR_WAIT2(x) "+v"(x[0]), "+v"(x[1])
// four arrays of CB transposing reads each have landed
template <int CB, int N>
__device__ __forceinline__ void tr_wait(shortx4 (&a)[N], shortx4 (&b)[N], shortx4 (&c)[N], shortx4 (&d)[N]) {
    if constexpr (CB == 4) asm volatile("s_waitcnt lgkmcnt(0)" : TR_WAIT4(a), TR_WAIT4(b), TR_WAIT4(c), TR_WAIT4(d));
    else if constexpr (CB == 3) asm volatile("s_waitcnt lgkmcnt(0)" : TR_WAIT3(a), TR_WAIT3(b), TR_WAIT3(c), TR_WAIT3(d));
    else asm volatile("s_waitcnt lgkmcnt(0)" : TR_WAIT2(a), TR_WAIT2(b), TR_WAIT2(c), TR_WAIT2(d));
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}
// LDS read of the dK/dV kernel's first wavefronts.  A read written as assembly may only be waited for in one place of the program: where two
// branches follow it, each with a wait of its own, the compiler copied the result in one of them in front of that branch's wait.
template <typename V>
__device__ __forceinline__ V lds_load(uint32_t addr) {
    return *(volatile __attribute__((address_space(3))) const V *)(uintptr_t)addr;
}
// LDS reads of its second wavefronts, written as assembly together with their waits: the compiler makes reads wait for copies in flight
// and does not count the transposing reads, so its waits come out stricter than needed.  All of them are volatile, so they are issued
// in source order, and the kernel counts that order.
template <int IMM, typename V>
__device__ __forceinline__ void lds_read16(V &dst, uint32_t addr) {
    static_assert(sizeof(V) == 16 && IMM >= 0 && IMM < 65536, "ds_read_b128");
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(IMM));
}
// Inverse rotary embedding of a gradient held in accumulator layout (the backward pass of the rotation that
// was applied to q and k before the attention): feature f < D/2 pairs with f + D/2, which sit in the same
// lane and register index of accumulators c and c + CB/2.  cs = the (cos, sin) row of this lane's token.
template <int CB>
__device__ __forceinline__ void unrotate(f32x16 (&g)[CB], const float2 *cs, int half) {
#pragma unroll
    for (int c = 0; c < CB / 2; ++c)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const float4 *p4 = reinterpret_cast<const float4 *>(cs + 32 * c + 8 * gq + 4 * half);
            const float4 a = p4[0], b = p4[1];
            const float co[4] = {a.x, a.z, b.x, b.z}, si[4] = {a.y, a.w, b.y, b.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float lo = g[c][4 * gq + e], hi = g[c + CB / 2][4 * gq + e];
                g[c][4 * gq + e] = lo * co[e] + hi * si[e];
                g[c + CB / 2][4 * gq + e] = hi * co[e] - lo * si[e];
            }
        }
}

// Stores a wavefront's 32 x D result (accumulator layout: lane = row, registers = features; 4 consecutive features
// per lane and register quad) as bf16 rows of a row-major tensor.  The rows go through LDS so that a store
// instruction writes 16 bytes per lane and D / 8 lanes cover a row, whole cache lines, instead of 8 bytes into
// each of 32 rows.  stage: STAGE_BYTES<D> bytes of LDS that belong to this wavefront alone and that no wavefront still
// reads as a tile (the callers put a barrier in front).  dst: row 0, feature 0; rows_valid rows and dh features exist.
template <int D>
constexpr int STAGE_BYTES = 32 * (2 * D + 16);
template <int D>
constexpr int ROWS32_BYTES = 32 * D * 2;              // 32 rows of one operand, staged in the tile layout
template <int D>
constexpr int DKV_STAGE_BYTES = 4 * ROWS32_BYTES<D>;  // the rows of one operand of the plain dK/dV kernel's 4 wavefronts
// the dQ kernel: first slot, then the Q and dO rows of 8 wavefronts (the second slot lies there later), or two slots, the second
// of which holds the rows of one operand at a time of 4 wavefronts
template <int D, int WAVES>
constexpr int DQ_LDS_BYTES = WAVES == 8 ? 2 * BT2 * D * 2 + 8 * 2 * ROWS32_BYTES<D> : 2 * 2 * BT2 * D * 2;
// the forward kernel: two slots of a K and a V tile; with 8 wavefronts their Q rows (of 4: in the second slot) and the first 32 K rows
template <int D, int WAVES>
constexpr int FWD_LDS_BYTES = 2 * 2 * BT2 * D * 2 + (WAVES == 8 ? 9 * ROWS32_BYTES<D> : 0);
// the plain dK/dV kernel: two slots of a Q tile, a dO tile and their log-sum-exps and D values, and the K and V rows of 4 wavefronts
template <int D>
constexpr int DKV_PLAIN_LDS = 2 * (2 * BT2 * D * 2 + 2 * BT2 * 4) + 2 * DKV_STAGE_BYTES<D>;
// colsum: when not null, receives the sums of the stored rows' columns (bias gradients of the linear behind them), from the rounded values.
// A pass of its own over d_qkv for these took 12.7 us on 9536 x 3072, 5.9 on 2304 x 3072.  Not for heads wider than 96, whose dQ kernel has no
// register left for them.
template <int D, int CB>
__device__ __forceinline__ void store_rows(uint8_t *stage, const f32x16 (&acc)[CB], float scale, bf16_t *dst, long ld,
                                           int rows_valid, int dh, float *colsum = nullptr) {
    constexpr bool SUMS = 32 * CB <= COLSUM_HEAD;
    constexpr int RS = 2 * D + 16, LPR = D / 8, RPI = 64 / LPR;    // row stride in LDS (2-way bank conflicts at most)
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            uint2 w;
            w.x = pack_bf16x2(acc[c][4 * gq] * scale, acc[c][4 * gq + 1] * scale);
            w.y = pack_bf16x2(acc[c][4 * gq + 2] * scale, acc[c][4 * gq + 3] * scale);
            *reinterpret_cast<uint2 *>(stage + l32 * RS + (32 * c + 8 * gq + 4 * half) * 2) = w;
        }
    const int r0 = lane / LPR, cb = (lane % LPR) * 16;
    uint4 v[32 / RPI];                                 // read and stored without a branch in between: callers without sums paid up to 3 % for one
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int r = i * RPI + r0;
        v[i] = *reinterpret_cast<const uint4 *>(stage + r * RS + cb);
        if (r < rows_valid && cb / 2 < dh) *reinterpret_cast<uint4 *>(dst + (long)r * ld + cb / 2) = v[i];
    }
    if (SUMS && colsum) {
        float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) {
            const bool valid = i * RPI + r0 < rows_valid;
            const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sum[2 * e] += valid ? __uint_as_float(w[e] << 16) : 0.f;
                sum[2 * e + 1] += valid ? __uint_as_float(w[e] & 0xffff0000u) : 0.f;
            }
        }
#pragma unroll
        for (int o = LPR; o < 64; o *= 2)
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[e] += __shfl_xor(sum[e], o, 64);
        if (r0 == 0 && cb / 2 < dh && rows_valid > 0) {
            f32x4 *out = reinterpret_cast<f32x4 *>(colsum + cb / 2);
            out[0] = f32x4{sum[0], sum[1], sum[2], sum[3]};
            out[1] = f32x4{sum[4], sum[5], sum[6], sum[7]};
        }
    }
}

// The same rows as fp32, unscaled, for partial sums: every row of the tensor has ld floats, all D features are stored.
template <int D>
constexpr int STAGE32_BYTES = 32 * (4 * D + 16);
template <int D, int CB>
__device__ __forceinline__ void store_rows_f32(uint8_t *stage, const f32x16 (&acc)[CB], float *dst, long ld, int rows_valid, int dh) {
    constexpr int RS = 4 * D + 16, LPR = D / 4, RPI = 64 / LPR;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq)
            *reinterpret_cast<f32x4 *>(stage + l32 * RS + (32 * c + 8 * gq + 4 * half) * 4) =
                f32x4{acc[c][4 * gq], acc[c][4 * gq + 1], acc[c][4 * gq + 2], acc[c][4 * gq + 3]};
    const int r0 = lane / LPR, cb = (lane % LPR) * 16;
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int r = i * RPI + r0;
        const f32x4 v = *reinterpret_cast<const f32x4 *>(stage + r * RS + cb);
        if (r < rows_valid && cb / 4 < dh) *reinterpret_cast<f32x4 *>(dst + (long)r * ld + cb / 4) = v;
    }
}

// Two wavefronts of a workgroup that share a row block (PARTS = 2): the second leaves its N values per lane in LDS, the first
// picks them up after the barrier in between.  box: XCHG_BYTES<N> bytes that belong to the pair.
template <int N>
constexpr int XCHG_BYTES = (N + 3) / 4 * 1024;
template <int CB>
__device__ __forceinline__ void put_acc(uint8_t *box, const f32x16 (&acc)[CB]) {
    f32x4 *p = reinterpret_cast<f32x4 *>(box) + (threadIdx.x & 63);
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) p[(4 * c + i) * 64] = f32x4{acc[c][4 * i], acc[c][4 * i + 1], acc[c][4 * i + 2], acc[c][4 * i + 3]};
}
// acc = acc * w_own + what the other wavefront put * w_other
template <int CB>
__device__ __forceinline__ void merge_acc(const uint8_t *box, f32x16 (&acc)[CB], float w_own, float w_other) {
    const f32x4 *p = reinterpret_cast<const f32x4 *>(box) + (threadIdx.x & 63);
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 v = p[(4 * c + i) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[c][4 * i + e] = acc[c][4 * i + e] * w_own + v[e] * w_other;
        }
}

// End of both dK/dV kernels: a wavefront's 32 keys' dV and dK (unscaled) as rows of d_qkv, or, where the query heads of a
// group are shared out over several workgroups, as this workgroup's fp32 partial sums.
template <int D, int CB>
__device__ __forceinline__ void store_dkv(const AttnArgs &a, uint8_t *smem, int wave, int half, int g, int key0, int key, bool valid,
                                          f32x16 (&dk)[CB], f32x16 (&dv)[CB]) {
    const int dh = a.d, nk = a.nkv * dh, rows = a.T - key0;
    if (a.dkv_parts > 1) {
        float *out = a.dkv_part + ((size_t)blockIdx.z * a.T + key0) * 2 * nk + g * dh;
        uint8_t *stage = smem + wave * STAGE32_BYTES<D>;
        store_rows_f32<D, CB>(stage, dk, out, 2 * nk, rows, dh);
        store_rows_f32<D, CB>(stage, dv, out + nk, 2 * nk, rows, dh);
        return;
    }
    bf16_t *okp = (bf16_t *)a.d_qkv + (long)key0 * a.ld_qkv + a.nh * dh + g * dh;
    uint8_t *stage = smem + wave * STAGE_BYTES<D>;
    float *const sums = a.colsum ? a.colsum + (size_t)(key0 / 32) * a.ld_qkv + a.nh * dh + g * dh : nullptr;
    store_rows<D, CB>(stage, dv, 1.f, okp + nk, a.ld_qkv, rows, dh, sums ? sums + nk : nullptr);
    if constexpr (CB == D / 32)
        if (valid && a.rope_cs) unrotate<CB>(dk, a.rope_cs + (long)key * (D / 2), half);
    store_rows<D, CB>(stage, dk, a.scale, okp, a.ld_qkv, rows, dh, sums);
}

// The partial sums of the workgroups that share a group's query heads, added in order: dK scaled and rotated back, dV, as bf16
// rows of d_qkv.  A thread owns four features below d / 2 and the four they are rotated with.
__global__ __launch_bounds__(256) void dkv_reduce_kernel(AttnArgs a) {
    const int dh = a.d, nk = a.nkv * dh, quads = dh / 8, per_row = 2 * a.nkv * quads;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)a.T * per_row) return;
    const int t = (int)(idx / per_row), r = (int)(idx % per_row), head = r / quads, f = r % quads * 4;
    const bool is_k = head < a.nkv;
    const size_t stride = (size_t)a.T * 2 * nk;
    const float *p = a.dkv_part + (size_t)t * 2 * nk + head * dh + f;
    f32x4 lo = *reinterpret_cast<const f32x4 *>(p), hi = *reinterpret_cast<const f32x4 *>(p + dh / 2);
    for (int i = 1; i < a.dkv_parts; ++i) {
        lo += *reinterpret_cast<const f32x4 *>(p + i * stride);
        hi += *reinterpret_cast<const f32x4 *>(p + i * stride + dh / 2);
    }
    if (is_k) {
        if (a.rope_cs) {
            const float2 *cs = a.rope_cs + (size_t)t * (dh / 2) + f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = lo[e], y = hi[e];
                lo[e] = x * cs[e].x + y * cs[e].y;
                hi[e] = y * cs[e].x - x * cs[e].y;
            }
        }
        lo *= a.scale; hi *= a.scale;
    }
    bf16_t *out = (bf16_t *)a.d_qkv + (size_t)t * a.ld_qkv + a.nh * dh + head * dh + f;      // k heads, then v heads
    *reinterpret_cast<uint2 *>(out) = make_uint2(pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]));
    *reinterpret_cast<uint2 *>(out + dh / 2) = make_uint2(pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3]));
}

// ------------------------------------------------------------------------------------------
// backward: dQ (and -D, D = rowsum(dO * O)).  Same roles as the forward kernel: 8 or 4 wavefronts x 32 queries, or two groups of 4.
// ------------------------------------------------------------------------------------------
template <int D, int KS, int CB, int WAVES, int PARTS>
__global__ __launch_bounds__(WAVES * PARTS * 64, 2) void attn_dq_kernel(AttnArgs a) {
    static_assert(PARTS == 1 || WAVES == 4, "the key range is shared by two groups of four wavefronts");
    constexpr int FQW = WAVES * 32;                                // queries per workgroup
    constexpr int TILE = BT2 * D * 2, SLOT = 2 * TILE;             // K tile, then V tile
    constexpr int COPIES = BT2 * D * 2 / 1024 / 4;                 // per wavefront (4 wavefronts per tile)
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_all[];
    // grid: x = head, y = position in the dispatch order of the query tiles (heaviest first)
    const int head = blockIdx.x, g = head / (a.nh / a.nkv);
    // (of FQ-query tiles: the workgroups of one tile, two with four wavefronts each, follow each other)
    constexpr int PER_TILE = FQ / FQW;
    const int q0 = (a.use_order ? a.order_q[blockIdx.y / PER_TILE] * PER_TILE + blockIdx.y % PER_TILE : blockIdx.y) * FQW;
    if (q0 >= a.T) return;                                         // second half of a last tile that the pack only half fills
    add_busy(a.cu_busy ? a.cu_busy + 1024 : nullptr, false);
    // the wavefront's index as a scalar: what is derived from it (copy destinations, buffer descriptors) stays uniform
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5, l32 = lane & 31;
    const int part = PARTS == 1 ? 0 : wv / WAVES, wave = PARTS == 1 ? wv : wv % WAVES;
    uint8_t *const smem = smem_all + part * 2 * SLOT;
    const int T = a.T;
    const bf16_t *qkv = (const bf16_t *)a.qkv;
    const long ld = a.ld_qkv;
    const int dh = a.d;                                 // head dimension in memory (<= D: LDS tiles and fragments are zero-padded to D)
    const int nq = a.nh * dh, nk = a.nkv * dh;

    const int q = q0 + wave * 32 + l32;
    RowInfo me, first, last;
    ranges<false>(a, q0, FQW, q0 + wave * 32, me, first, last);
    const bool valid = q < T;
    const WaveBounds wb = wave_bounds(me, q0 + wave * 32, T);
    const int w_lo_min = wb.lo_min, w_lo_max = wb.lo_max, w_hi_max = wb.hi_max, w_hi_min = wb.hi_min;
    const int kbeg = first.lo, kend = last.hi;

    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(qkv), 0, (int)(uint32_t)((size_t)T * ld * 2), 0x00020000);
    // eight wavefronts: 4..7 copy the K tile, 0..3 the V tile; four wavefronts: each copies its quarter of both
    RowCopier<D, COPIES> cp;
    cp.init((wave & 3) * COPIES, ld, dh);
    auto copy_kv = [&](uint8_t *slot, int kt) {
        if (WAVES == 4 || wave >= 4) cp.issue(rs, slot, kt, ld, nq + g * dh);
        if (WAVES == 4 || wave < 4) cp.issue(rs, slot + TILE, kt, ld, nq + nk + g * dh);
    };
    TrReader<D> tr;
    tr.init((uint32_t)(uintptr_t)(lds_void *)smem);

    // This wavefront's 32 rows of Q, dO and O: copied into LDS the way tiles are (whole rows per instruction, rows
    // beyond the pack and features beyond the head's width as zeros) and read back in the fragment layout; loading
    // them straight into that layout takes 24 loads of 16 bytes per row and a fifth of the kernel's time on packs
    // of short segments.  They stand behind the first slot (Q and dO side by side, O then in Q's place); the second
    // slot, which they cover, is first written after the first step's barrier.
    bf16x8 qf[KS], dof[KS];
    float Dq = 0.f;
    {
        const __amdgpu_buffer_rsrc_t rs_do = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<bf16_t *>((const bf16_t *)a.d_o), 0, (int)(uint32_t)((size_t)T * nq * 2), 0x00020000);
        const __amdgpu_buffer_rsrc_t rs_o = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<bf16_t *>((const bf16_t *)a.o), 0, (int)(uint32_t)((size_t)T * nq * 2), 0x00020000);
        RowCopier<D, ROWS32_BYTES<D> / 1024> cp_q, cp_o;
        cp_q.init(0, ld, dh);
        cp_o.init(0, nq, dh);
        uint8_t *st_q = smem + SLOT + wave * (WAVES == 8 ? 2 : 1) * ROWS32_BYTES<D>;
        if constexpr (WAVES == 8) {
            uint8_t *st_do = st_q + ROWS32_BYTES<D>;
            cp_q.issue(rs, st_q, q0 + wave * 32, ld, head * dh);
            cp_o.issue(rs_do, st_do, q0 + wave * 32, nq, head * dh);
            if (part == 0 || kbeg + BT2 < kend) copy_kv(smem, kbeg + part * BT2);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                qf[ks] = frag_k<D>(st_q, l32, ks, half);
                dof[ks] = frag_k<D>(st_do, l32, ks, half);
            }
        } else {                                                     // one operand after the other in the same place
            cp_q.issue(rs, st_q, q0 + wave * 32, ld, head * dh);
            if (part == 0 || kbeg + BT2 < kend) copy_kv(smem, kbeg + part * BT2);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[ks] = frag_k<D>(st_q, l32, ks, half);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            cp_o.issue(rs_do, st_q, q0 + wave * 32, nq, head * dh);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) dof[ks] = frag_k<D>(st_q, l32, ks, half);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // read: O may take the place
        cp_o.issue(rs_o, st_q, q0 + wave * 32, nq, head * dh);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 of = frag_k<D>(st_q, l32, ks, half);
            const uint4 w = *reinterpret_cast<const uint4 *>(&dof[ks]), x = *reinterpret_cast<const uint4 *>(&of);
            const uint32_t dw[4] = {w.x, w.y, w.z, w.w}, ow[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                Dq += __uint_as_float(dw[e] << 16) * __uint_as_float(ow[e] << 16);
                Dq += __uint_as_float(dw[e] & 0xffff0000u) * __uint_as_float(ow[e] & 0xffff0000u);
            }
        }
    }
    Dq += __shfl_xor(Dq, 32, 64);
    float lse2 = 0.f;                                  // log-sum-exp in log2 units
    if (valid) {
        lse2 = a.lse[(long)head * T + q] * LOG2E;
        if (half == 0 && part == 0) a.Dsum[(long)head * T + q] = -Dq;                // the dK/dV kernels add it
    }
    // With 64-wide heads dP - D comes out of the matrix core: the dP product of every block starts from -D instead of
    // from zero (a lane holds keys of ONE query, so the 16 accumulator registers of a lane all start from that query's
    // -D).  The 128-wide kernel has no 16 registers to hold that operand and subtracts D element by element.
    constexpr bool D_IN_MFMA = D <= 64;
    f32x16 negD;
#pragma unroll
    for (int i = 0; i < 16; ++i) negD[i] = D_IN_MFMA ? -Dq : 0.f;
    f32x16 dq[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) dq[c] = zero16();
    const float sl2 = a.scale * LOG2E;

    int slot = 0;
    for (int kt = kbeg + part * BT2; kt - part * BT2 < kend; kt += PARTS * BT2, slot ^= 1) {
        const uint8_t *sK = smem + slot * SLOT, *sV = sK + TILE;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this step's tiles have landed
        lds_barrier();                                               // ... and everyone is done with the other slot
        if (kt + PARTS * BT2 < kend) copy_kv(smem + (slot ^ 1) * SLOT, kt + PARTS * BT2);
        auto block = [&](auto B_) {
            constexpr int b = decltype(B_)::value;
            const int kb = kt + 32 * b;
            if (!((kb < w_hi_max) && (kb + 32 > w_lo_min))) return;
            f32x16 s = zero16(), dp = negD;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                s = MFMA(frag_k<D>(sK, 32 * b + l32, ks, half), qf[ks], s);
                dp = MFMA(frag_k<D>(sV, 32 * b + l32, ks, half), dof[ks], dp);
            }
            // K^T fragments of this block: [MFMA m][feature block c], two halves each
            shortx4 t0[4], t1[4], t2[4], t3[4];                      // (m, sec) = (0,0), (0,1), (1,0), (1,1)
            const uint32_t tile = slot * SLOT;
            t0[0] = tr.template read<b, 0, 0, 0>(tile); t1[0] = tr.template read<b, 0, 0, 1>(tile);
            t2[0] = tr.template read<b, 1, 0, 0>(tile); t3[0] = tr.template read<b, 1, 0, 1>(tile);
            t0[1] = tr.template read<b, 0, 1, 0>(tile); t1[1] = tr.template read<b, 0, 1, 1>(tile);
            t2[1] = tr.template read<b, 1, 1, 0>(tile); t3[1] = tr.template read<b, 1, 1, 1>(tile);
            if constexpr (CB > 2) {
                t0[2] = tr.template read<b, 0, 2, 0>(tile); t1[2] = tr.template read<b, 0, 2, 1>(tile);
                t2[2] = tr.template read<b, 1, 2, 0>(tile); t3[2] = tr.template read<b, 1, 2, 1>(tile);
            }
            if constexpr (CB > 3) {
                t0[3] = tr.template read<b, 0, 3, 0>(tile); t1[3] = tr.template read<b, 0, 3, 1>(tile);
                t2[3] = tr.template read<b, 1, 3, 0>(tile); t3[3] = tr.template read<b, 1, 3, 1>(tile);
            }
            const bool inside = kb >= w_lo_max && kb + 32 <= w_hi_min;
            const unsigned span = (unsigned)(me.hi - me.lo);
            const int rel = kb + 4 * half - me.lo;
            float ds[16];
            // two copies of the loop, so that a block no key of which is masked pays nothing for the mask
            auto softmax = [&](auto MASK_) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    float p = __builtin_amdgcn_exp2f(fmaf(s[i], sl2, -lse2));
                    if (decltype(MASK_)::value) p = (unsigned)(rel + 8 * (i >> 2) + (i & 3)) < span ? p : 0.f;
                    ds[i] = D_IN_MFMA ? p * dp[i] : p * (dp[i] - Dq);
                }
            };
            if (inside) softmax(std::false_type{});
            else softmax(std::true_type{});
            tr_wait<CB>(t0, t1, t2, t3);
            const bf16x8 ds0 = pack8(ds), ds1 = pack8(ds + 8);
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                dq[c] = MFMA(join(t0[c], t1[c]), ds0, dq[c]);
                dq[c] = MFMA(join(t2[c], t3[c]), ds1, dq[c]);
            }
        };
        block(std::integral_constant<int, 0>{});
        block(std::integral_constant<int, 1>{});
    }
    lds_barrier();                                     // the tiles are done with: LDS now stages the output rows
    uint8_t *stage = smem_all + wave * STAGE_BYTES<D>;
    if constexpr (PARTS == 2) {
        uint8_t *box = smem_all + wave * XCHG_BYTES<16 * CB>;
        stage += WAVES * XCHG_BYTES<16 * CB>;
        if (part == 1) put_acc(box, dq);
        lds_barrier();
        if (part == 1) return;
        merge_acc(box, dq, 1.f, 1.f);
    }
    if constexpr (CB == D / 32)                        // (narrower heads are rotated back by a pass of their own)
        if (valid && a.rope_cs) unrotate<CB>(dq, a.rope_cs + (long)q * (D / 2), half);
    store_rows<D, CB>(stage, dq, a.scale, (bf16_t *)a.d_qkv + (long)(q0 + wave * 32) * ld + head * dh, ld, T - (q0 + wave * 32), dh,
                      a.colsum ? a.colsum + (size_t)(q0 / 32 + wave) * ld + head * dh : nullptr);
    add_busy(a.cu_busy ? a.cu_busy + 1024 : nullptr, true);
}

// Exchange between lane l and lane l ^ 32 in one vector instruction (the two halves of a wavefront hold the two halves of
// every query's keys): after the swap the first result holds the lower half's values in both halves, the second the upper's.
__device__ __forceinline__ float max_across_halves(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_across_halves(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The forward kernel's running maximum is lazy: the reference the exponentials are taken against moves only when a
// block's maximum exceeds it by more than 2^LAZY_LOG2 (in units of the exponent), so the output accumulators are rescaled
// a few times per query instead of at almost every block; exponentials stay below 2^LAZY_LOG2, far inside fp32 and bf16 range.
// From the first block to the second it moves by any amount: the exponential of the maximum is 1 and has no rounding error, and of 64
// keys the first reference is more often the row's maximum than of 32 (l2 error of the output, 1100 causal tokens of 64 heads: 2.051e-3; lazy
// there too 2.079e-3; the maximum over 64 keys at once 2.058e-3).
constexpr float LAZY_LOG2 = 8.f;

// LDS reads of items lo .. hi - 1 of a forward block of KS items with one read each and NI - KS with two
template <int KS, int NI>
constexpr int lds_ops(int lo, int hi) {
    int n = 0;
    for (int x = lo; x < hi && x < NI; ++x) n += x < KS ? 1 : 2;
    return n;
}

// ------------------------------------------------------------------------------------------
// forward.  WAVES wavefronts x 32 queries per workgroup, two wavefronts per SIMD either way (so that one can run its
// softmax on the vector ALUs while the other occupies the matrix core): 8 wavefronts = 256 queries, one workgroup per
// compute unit (every K / V tile is fetched once for 256 queries), or 4 wavefronts = 128 queries, two workgroups per
// compute unit (see four_waves).  PARTS = 2: two groups of 4 wavefronts with the same 128 queries, the keys of every other step and
// LDS slots each (see two_parts).  The keys are walked 64 at a time through two LDS slots of {K tile, V tile}, both copied global -> LDS
// directly in their memory order (wavefronts 4..7 copy K, 0..3 copy V).  O^T = V^T . P^T takes V^T from the row-major tile by the
// transposing LDS read, the same scheme as dQ^T = K^T . dS^T above.  One barrier per step: after it every wavefront has finished the
// previous step, so the slot that step used may be refilled.
// LOOK_AHEAD: with eight wavefronts each works one block of 32 keys ahead: the scores of the next block are multiplied between the
// exponentials of the current one, neither of which needs the other, and a K tile therefore stands one block further on than its V tile.
// Taken one after the other, a block's scores, maxima, exponentials and products wait for each other and for their LDS reads, and two
// wavefronts per SIMD overlap only part of that (an issue benchmark of the same mix: 980 cycles per block for one wavefront, 620 in turn).
// What bounds it: LDS reads (half of its cycles) and MFMAs together, the barrier (the ramp behind it and the wavefront that comes last), and
// power: a tenth fewer cycles come with 4 % less clock.  128 keys per step, reads 3, 5 or 6 items ahead change nothing.  us without ->
// with it: 32 heads of 128, 8192 tokens in one long document 490 -> 446, in spans 138 -> 128.  Four wavefronts, whose workgroups walk
// fewer steps, run the longer program from a cold instruction cache and lose as much there as they gain: alone, 2047 tokens of 64 heads on 8 48.4 ->
// 46.5, but in a row of other kernels the same, one image of 576 patches through a layer 63.5 -> 64.4.
// ------------------------------------------------------------------------------------------
template <int D, int KS, int CB, int WAVES, int PARTS>
__global__ __launch_bounds__(WAVES * PARTS * 64, 2) void attn_fwd_kernel(AttnArgs a) {
    static_assert(PARTS == 1 || WAVES == 4, "the key range is shared by two groups of four wavefronts");
    constexpr int FQW = WAVES * 32;                                // queries per workgroup
    constexpr int TILE = BT2 * D * 2, SLOT = 2 * TILE;             // K tile, then V tile
    constexpr int COPIES = BT2 * D * 2 / 1024 / 4;                 // per wavefront and tile (four wavefronts copy a tile)
    constexpr bool LOOK_AHEAD = WAVES == 8;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_all[];
    const int head = blockIdx.x, g = head / (a.nh / a.nkv);
    // the dispatch order is kept per FQ-query tile; the workgroups of one tile (two, with four wavefronts each) follow each other
    constexpr int PER_TILE = FQ / FQW;
    const int q0 = (a.use_order ? a.order_q[blockIdx.y / PER_TILE] * PER_TILE + blockIdx.y % PER_TILE : blockIdx.y) * FQW;
    if (q0 >= a.T) return;                                         // second half of a last tile that the pack only half fills
    add_busy(a.cu_busy, false);
    // the wavefront's index as a scalar: what is derived from it (copy destinations, buffer descriptors) stays uniform
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5, l32 = lane & 31;
    const int part = PARTS == 1 ? 0 : wv / WAVES, wave = PARTS == 1 ? wv : wv % WAVES;
    uint8_t *const smem = smem_all + part * 2 * SLOT;
    const int T = a.T;
    const bf16_t *qkv = (const bf16_t *)a.qkv;
    const long ld = a.ld_qkv;
    const int dh = a.d;
    const int nq = a.nh * dh, nk = a.nkv * dh;

    const int q = q0 + wave * 32 + l32;
    RowInfo me, first, last;
    ranges<false>(a, q0, FQW, q0 + wave * 32, me, first, last);
    const bool valid = q < T;
    const WaveBounds wb = wave_bounds(me, q0 + wave * 32, T);
    const int w_lo_min = wb.lo_min, w_lo_max = wb.lo_max, w_hi_max = wb.hi_max, w_hi_min = wb.hi_min;
    const int kbeg = first.lo, kend = last.hi;

    bf16x8 qf[KS];                                     // this wavefront's Q rows as the MFMA's column operand (filled below)
    f32x16 oacc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) oacc[c] = zero16();
    // the reference of the exponentials (raw score), the same in the exponent's units, the row sum
    float m_run = -INFINITY, msc = 0.f, l_run = 0.f;
    const float sl2 = a.scale * LOG2E;

    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(qkv), 0, (int)(uint32_t)((size_t)T * ld * 2), 0x00020000);
    // eight wavefronts: 4..7 copy the K tile, 0..3 the V tile; four wavefronts: each copies its quarter of both.  With the look ahead a
    // step's K tile stands one block of 32 keys further on than its V tile, and the first block's K rows have a place of their own
    RowCopier<D, COPIES> cp;
    cp.init((wave & 3) * COPIES, ld, dh);
    auto copy_kv = [&](uint8_t *slot, int kt) {
        if (WAVES == 4 || wave >= 4) cp.issue(rs, slot, kt + (LOOK_AHEAD ? 32 : 0), ld, nq + g * dh);
        if (WAVES == 4 || wave < 4) cp.issue(rs, slot + TILE, kt, ld, nq + nk + g * dh);
    };
    constexpr int K_FIRST = 2 * SLOT + WAVES * ROWS32_BYTES<D>;

    // The Q rows go through LDS like the dQ kernel's Q, dO and O rows (see there): behind the two slots, or, with four
    // wavefronts (whose Q rows fill a slot exactly), in the second slot, which is first written after the first barrier.
    {
        RowCopier<D, ROWS32_BYTES<D> / 1024> cp_q;
        cp_q.init(0, ld, dh);
        uint8_t *st_q = smem + (WAVES == 4 ? SLOT : 2 * SLOT) + wave * ROWS32_BYTES<D>;
        cp_q.issue(rs, st_q, q0 + wave * 32, ld, head * dh);
        if (LOOK_AHEAD && (wave == 4 || wave == 5)) cp.issue(rs, smem + K_FIRST, kbeg, ld, nq + g * dh);
        if (part == 0 || kbeg + BT2 < kend) copy_kv(smem, kbeg + part * BT2);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = frag_k<D>(st_q, l32, ks, half);
    }
    TrReader<D> tr;
    tr.init((uint32_t)(uintptr_t)(lds_void *)smem);
    if constexpr (LOOK_AHEAD) {
        // LDS addresses in the first slot: K rows l32, 16-byte unit 2 ks + half; the V tile's transposing reads
        uint32_t kadr[KS];
        const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kadr[ks] = lds0 + (l32 * (D / 8) + ((2 * ks + half) ^ swz_unit<D>(l32))) * 16;
        const unsigned span = (unsigned)(me.hi - me.lo);
        f32x16 s[2];                                       // scores of the blocks of either parity
        uint32_t pp[8];
        // element i of a block: its exponential, the row sum, packed in pairs.  Register i  <->  key kb + 8 (i >> 2) + 4 half + (i & 3)
        auto element = [&](auto I_, const f32x16 &cur, float &keep) {
            constexpr int i = decltype(I_)::value;
            const float p = __builtin_amdgcn_exp2f(fmaf(cur[i], sl2, -msc));
            l_run += p;
            asm volatile("" : "+v"(l_run));               // (here, between the MFMAs: the compiler would collect the additions behind them)
            if constexpr (i & 1) pp[i >> 1] = pack_bf16x2(keep, p);
            else keep = p;
        };
        auto p_frag = [&](auto M_) {
            constexpr int m = decltype(M_)::value;
            const rawx4 w = {pp[4 * m], pp[4 * m + 1], pp[4 * m + 2], pp[4 * m + 3]};
            return *reinterpret_cast<const bf16x8 *>(&w);
        };
        auto mask = [&](f32x16 &x, int kb) {
            const int rel = kb + 4 * half - me.lo;
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = (unsigned)(rel + 8 * (i >> 2) + (i & 3)) < span ? x[i] : -INFINITY;
        };
        auto max16 = [&](const f32x16 &x) {
            float mx = x[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, x[i]);
            return mx;
        };
        float m_limit = -INFINITY;                         // the maximum that moves the reference
        const float lazy = LAZY_LOG2 / sl2;
        // move the reference only where a block's maximum (of this lane's keys, or of its other half's) is more than 2^LAZY_LOG2 above it;
        // STRICT (a wavefront's first block): the next one moves it by any amount
        auto follow = [&](float mx, auto STRICT_) {
            if (__builtin_amdgcn_ballot_w64(mx > m_limit) == 0) return;
            mx = max_across_halves(mx);
            const bool need = mx > m_limit;
            const float corr = need ? __builtin_amdgcn_exp2f((m_run - mx) * sl2) : 1.f;
            m_run = need ? mx : m_run;
            m_limit = decltype(STRICT_)::value ? m_run : m_run + lazy;
            msc = m_run == -INFINITY ? 0.f : m_run * sl2;
            l_run *= corr;
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[c][i] *= corr;
        };
        // Block b of a step, whose scores are in s[b]: its exponentials and products with V, and the scores of the block behind it (keys
        // nb ..), whose MFMAs have nothing to do with the exponentials and stand between them.  Items 0 .. KS - 1 are the score MFMAs, the
        // others those with V (16 keys m, 32 features c); each needs one LDS read (K: 16 bytes, V: two transposing ones), issued AHEAD
        // items in front of it.
        auto block = [&](auto SLOT_, auto B_, int nb) {
            constexpr int b = decltype(B_)::value, NI = KS + 2 * CB, AHEAD = 4, AT = decltype(SLOT_)::value * SLOT;
            const f32x16 &cur = s[b];
            f32x16 &nxt = s[b ^ 1];
            bf16x8 fr[KS];
            shortx4 v0[2 * CB], v1[2 * CB];
            auto issue = [&](auto X_) {
                constexpr int x = decltype(X_)::value;
                if constexpr (x < KS) lds_read16<AT + b * 64 * D>(fr[x], kadr[x]);
                else if constexpr (x < NI) {
                    constexpr int m = (x - KS) / CB, c = (x - KS) % CB;
                    v0[x - KS] = TrReader<D>::template read_at<b, m, c, 0, AT + TILE>(tr.off);
                    v1[x - KS] = TrReader<D>::template read_at<b, m, c, 1, AT + TILE>(tr.off);
                }
            };
            float keep = 0.f, mx = -INFINITY;
            static_for<0, AHEAD>([&](auto X_) { issue(X_); });
            __builtin_amdgcn_sched_barrier(0);
            // two elements while the first reads are on their way, the others spread over the items in front of the second 16 keys' products
            constexpr int E0 = 2, SPAN = KS + CB;
            static_for<0, E0>([&](auto I_) { element(I_, cur, keep); });
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, NI>([&](auto X_) {
                constexpr int x = decltype(X_)::value;
                constexpr int behind = lds_ops<KS, NI>(x + 1, x + AHEAD);       // reads issued behind item x's
                if constexpr (x < KS) {
                    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[x]) : "n"(behind));
                    if constexpr (x == 0) nxt = MFMA(fr[x], qf[x], zero16());
                    else nxt = MFMA(fr[x], qf[x], nxt);
                } else {
                    constexpr int m = (x - KS) / CB, c = (x - KS) % CB;
                    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(v0[x - KS]), "+v"(v1[x - KS]) : "n"(behind));
                    oacc[c] = MFMA(join(v0[x - KS], v1[x - KS]), p_frag(std::integral_constant<int, m>{}), oacc[c]);
                }
                issue(std::integral_constant<int, x + AHEAD>{});
                constexpr int lo = x < SPAN ? E0 + (16 - E0) * x / SPAN : 16, hi = x + 1 < SPAN ? E0 + (16 - E0) * (x + 1) / SPAN : 16;
                static_for<lo, hi>([&](auto I_) { element(I_, cur, keep); });
                if constexpr (x > KS) {
                    constexpr int d0 = 16 * (x - KS - 1) / (2 * CB - 1), d1 = 16 * (x - KS) / (2 * CB - 1);
                    static_for<d0, d1>([&](auto I_) { mx = fmaxf(mx, nxt[decltype(I_)::value]); });
                    asm volatile("" : "+v"(mx));
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if (!(nb >= w_lo_max && nb + 32 <= w_hi_min)) {
                mask(nxt, nb);
                mx = max16(nxt);
            }
            follow(mx, std::false_type{});
        };
        auto active = [&](int kb) { return kb < w_hi_max && kb + 32 > w_lo_min; };
        // The first block that has keys for this wavefront, numbered from kbeg on: its scores are computed one block earlier, by
        // themselves.  (Its blocks follow one another: both bounds of the ranges are non-decreasing.)
        const int lead = max(w_lo_min - kbeg, 0), lead_steps = lead / BT2, lead_rest = lead % BT2;
        const int n_first = 2 * lead_steps + (lead_rest < 32 ? 0 : lead_rest < 64 ? 1 : 2);
        const int kb_first = kbeg + (n_first >> 1) * BT2 + (n_first & 1) * 32;
        const int kt_head = active(kb_first) ? (n_first == 0 ? kbeg : kbeg + ((n_first - 1) >> 1) * BT2) : -1;
        // one step, its tiles in the given slot: written out per slot, so that every LDS address is a lane's constant and an immediate offset
        auto step = [&](auto SLOT_, int kt) {
            constexpr int slot = decltype(SLOT_)::value;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this step's tiles have landed
            lds_barrier();                                               // ... and everyone is done with the other slot
            if (kt == kt_head) {
                const uint32_t at = n_first == 0 ? K_FIRST : slot * SLOT + ((n_first - 1) & 1) * 64 * D;
                f32x16 x = zero16();
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) x = MFMA(lds_load<bf16x8>(kadr[ks] + at), qf[ks], x);
                if (!(kb_first >= w_lo_max && kb_first + 32 <= w_hi_min)) mask(x, kb_first);
                if (n_first & 1) s[1] = x;
                else s[0] = x;
                follow(max16(x), std::true_type{});
            }
            if (active(kt)) block(SLOT_, std::integral_constant<int, 0>{}, kt + 32);
            // (behind the first block: right behind the barrier all wavefronts would wait for each other at the copies)
            if (kt + BT2 < kend) copy_kv(smem + (slot ^ 1) * SLOT, kt + BT2);
            if (active(kt + 32)) block(SLOT_, std::integral_constant<int, 1>{}, kt + BT2);
        };
        for (int kt = kbeg; kt < kend; kt += 2 * BT2) {
            step(std::integral_constant<int, 0>{}, kt);
            if (kt + BT2 >= kend) break;
            step(std::integral_constant<int, 1>{}, kt + BT2);
        }
    } else {
        int slot = 0;
        for (int kt = kbeg + part * BT2; kt - part * BT2 < kend; kt += PARTS * BT2, slot ^= 1) {
            const uint8_t *sK = smem + slot * SLOT;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this step's tiles have landed
            lds_barrier();                                               // ... and everyone is done with the other slot
            if (kt + PARTS * BT2 < kend) copy_kv(smem + (slot ^ 1) * SLOT, kt + PARTS * BT2);
            bool act[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) act[b] = (kt + 32 * b < w_hi_max) && (kt + 32 * b + 32 > w_lo_min);
            if (!(act[0] || act[1])) continue;
            f32x16 s[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                s[b] = zero16();
                if (act[b]) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) s[b] = MFMA(frag_k<D>(sK, 32 * b + l32, ks, half), qf[ks], s[b]);
                }
            }
            // online softmax on the raw scores (the scale is folded into the exponent);
            // register i of block b  <->  key kt + 32 b + 8 (i >> 2) + 4 half + (i & 3)
            float mx = -INFINITY;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                if (!act[b]) continue;
                const int kb = kt + 32 * b;
                if (!(kb >= w_lo_max && kb + 32 <= w_hi_min)) {            // some lane needs masking
                    const unsigned span = (unsigned)(me.hi - me.lo);
                    const int rel = kb + 4 * half - me.lo;
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        s[b][i] = (unsigned)(rel + 8 * (i >> 2) + (i & 3)) < span ? s[b][i] : -INFINITY;
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[b][i]);
            }
            mx = max_across_halves(mx);
            // move the reference only where the step's maximum is more than 2^LAZY_LOG2 above it (always from -inf)
            const bool need = (mx - m_run) * sl2 > LAZY_LOG2;
            if (__builtin_amdgcn_ballot_w64(need) != 0) {
                const float corr = need ? __builtin_amdgcn_exp2f((m_run - mx) * sl2) : 1.f;
                m_run = need ? mx : m_run;
                l_run *= corr;
#pragma unroll
                for (int c = 0; c < CB; ++c)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[c][i] *= corr;
            }
            msc = m_run == -INFINITY ? 0.f : m_run * sl2;
            const uint32_t tv = slot * SLOT + TILE;
            auto block = [&](auto B_) {
                constexpr int b = decltype(B_)::value;
                if (!act[b]) return;
                // V^T fragments of this block: [MFMA m][feature block c], two halves each; in flight during the exponentials
                shortx4 t0[4], t1[4], t2[4], t3[4];
                t0[0] = tr.template read<b, 0, 0, 0>(tv); t1[0] = tr.template read<b, 0, 0, 1>(tv);
                t2[0] = tr.template read<b, 1, 0, 0>(tv); t3[0] = tr.template read<b, 1, 0, 1>(tv);
                t0[1] = tr.template read<b, 0, 1, 0>(tv); t1[1] = tr.template read<b, 0, 1, 1>(tv);
                t2[1] = tr.template read<b, 1, 1, 0>(tv); t3[1] = tr.template read<b, 1, 1, 1>(tv);
                if constexpr (CB > 2) {
                    t0[2] = tr.template read<b, 0, 2, 0>(tv); t1[2] = tr.template read<b, 0, 2, 1>(tv);
                    t2[2] = tr.template read<b, 1, 2, 0>(tv); t3[2] = tr.template read<b, 1, 2, 1>(tv);
                }
                if constexpr (CB > 3) {
                    t0[3] = tr.template read<b, 0, 3, 0>(tv); t1[3] = tr.template read<b, 0, 3, 1>(tv);
                    t2[3] = tr.template read<b, 1, 3, 0>(tv); t3[3] = tr.template read<b, 1, 3, 1>(tv);
                }
                float p[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    p[i] = __builtin_amdgcn_exp2f(fmaf(s[b][i], sl2, -msc));
                    l_run += p[i];
                }
                tr_wait<CB>(t0, t1, t2, t3);
                const bf16x8 p0 = pack8(p), p1 = pack8(p + 8);
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    oacc[c] = MFMA(join(t0[c], t1[c]), p0, oacc[c]);
                    oacc[c] = MFMA(join(t2[c], t3[c]), p1, oacc[c]);
                }
            };
            block(std::integral_constant<int, 0>{});
            block(std::integral_constant<int, 1>{});
        }
    }

    lds_barrier();                                     // the tiles are done with: LDS now stages the output rows
    uint8_t *stage = smem_all + wave * STAGE_BYTES<D>;
    if constexpr (PARTS == 2) {                        // two partial softmaxes over disjoint keys become one
        uint8_t *box = smem_all + wave * XCHG_BYTES<16 * CB + 2>;
        float2 *ml = reinterpret_cast<float2 *>(box + 16 * CB * 256) + lane;
        stage += WAVES * XCHG_BYTES<16 * CB + 2>;
        if (part == 1) {
            put_acc(box, oacc);
            *ml = make_float2(m_run, l_run);
        }
        lds_barrier();
        if (part == 1) return;
        const float m1 = ml->x, m = fmaxf(m_run, m1);
        const float w0 = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run - m) * sl2);
        const float w1 = m1 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m1 - m) * sl2);
        merge_acc(box, oacc, w0, w1);
        l_run = l_run * w0 + ml->y * w1;
        m_run = m;
    }
    const float l_tot = sum_across_halves(l_run);
    store_rows<D, CB>(stage, oacc, valid ? 1.f / l_tot : 0.f, (bf16_t *)a.o + (long)(q0 + wave * 32) * nq + head * dh,
                      nq, T - (q0 + wave * 32), dh);
    if (valid && half == 0) a.lse[(long)head * T + q] = (m_run * sl2 + __builtin_amdgcn_logf(l_tot)) * LN2;
    add_busy(a.cu_busy, true);
}

// ------------------------------------------------------------------------------------------
// backward: dK, dV for heads wider than 64 features.  32 keys belong to a pair of wavefronts on one SIMD: the first holds their K and
// V rows and turns 32 queries at a time into P and dS (two score products of KS MFMAs and the softmax), the second holds dK and dV
// and adds dO^T P and Q^T dS (4 CB MFMAs).  Neither fits a SIMD twice (the accumulators alone take 128 registers), but the two
// halves do, and they need different units at the same time: while the first is in its softmax the second keeps the matrix core busy.
// P and dS go through LDS, 4 KiB per block of 32 queries, in the layout in which both wavefronts hold them (lane by lane, no
// conflicts), two buffers; the second wavefront works one block behind the first, with one barrier per block.  Q and dO tiles of 64
// queries go round three slots: a tile is copied by the second wavefronts during the three blocks in front of its first use.
// What bounds it: issue slots and power.  A block of 32 queries takes 1.62 k cycles (all keys visible), at about 1.7 GHz.  Left out one at a
// time: the second wavefront's work 1.52 k (and 2.0 GHz: a quarter of the time), the exponentials 1.50 k, the score fragments' reads 1.59 k, the
// transposing reads 1.61 k; nothing that is left gives much by itself.  Computing the next block's scores under the exponentials, or giving dP
// and dS to the second wavefront, moved cost and did not lower it.  dQ + dK/dV in us, against one wavefront per 32 keys with the next block's
// scores under the exponentials of this one and transposing reads at half rate: 32 heads of 128, 8192 tokens in one long document 1616 -> 1502; in
// bidirectional segments of 700 471 -> 411; 1031 tokens in four segments 45.8 -> 40.9; 64 heads on 8, 2047 tokens 334 -> 299; 16 heads of 80, 4111
// bidirectional tokens in twelve segments 78.7 -> 69.6.
// ------------------------------------------------------------------------------------------
template <int D>
constexpr int DKV_SLOT = 2 * BT2 * D * 2 + 2 * BT2 * 4;            // Q tile, dO tile, lse[64], D[64]
constexpr int PDS_BYTES = 4 * 1024;                                // P and dS of one block of one pair
template <int D>
constexpr int DKV_PAIR_LDS = 3 * DKV_SLOT<D> + 2 * 4 * PDS_BYTES;

template <int D, int KS, int CB>
__global__ __launch_bounds__(512, 2) void attn_dkv_kernel(AttnArgs a) {
    constexpr int TILE = BT2 * D * 2, SLOT = DKV_SLOT<D>, COPIES = BT2 * D * 2 / 1024 / 4;      // copies per second wavefront and tile
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    add_busy(a.cu_busy ? a.cu_busy + 2048 : nullptr, false);

    // grid: x = key/value head, y = position in the dispatch order of the key tiles (heaviest first), z = this workgroup's share
    // of the group's query heads
    const int g = blockIdx.x, group_heads = a.nh / a.nkv;
    const int h_first = g * group_heads + blockIdx.z * group_heads / a.dkv_parts;
    const int group = g * group_heads + (blockIdx.z + 1) * group_heads / a.dkv_parts - h_first;
    const int k0 = (a.use_order ? a.order_k[blockIdx.y] : blockIdx.y) * BQ;
    // the wavefront's index as a scalar: what is derived from it (copy destinations, buffer descriptors) stays uniform
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5, l32 = lane & 31;
    const int pair = wv & 3;                            // wavefronts i and i + 4 of a workgroup share a SIMD
    const bool first_of_pair = wv < 4;
    const int T = a.T;
    const bf16_t *qkv = (const bf16_t *)a.qkv;
    const bf16_t *dO = (const bf16_t *)a.d_o;
    const long ld = a.ld_qkv;
    const int dh = a.d;                                 // head dimension in memory (<= D: LDS tiles and fragments are zero-padded to D)
    const int nq = a.nh * dh, nk = a.nkv * dh;

    const int key = k0 + pair * 32 + l32;
    RowInfo me, first, last;                                // queries [lo, hi) see this key
    ranges<true>(a, k0, BQ, k0 + pair * 32, me, first, last);
    const bool valid = key < T;
    const WaveBounds wb = wave_bounds(me, k0 + pair * 32, T);
    const int w_lo_min = wb.lo_min, w_lo_max = wb.lo_max, w_hi_max = wb.hi_max, w_hi_min = wb.hi_min;
    const int qbeg = first.lo, qend = last.hi;              // (never empty: a key sees itself)

    const __amdgpu_buffer_rsrc_t rs_q =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(qkv), 0, (int)(uint32_t)((size_t)T * ld * 2), 0x00020000);
    // The (head, query tile) pairs form one sequence of steps, every step two blocks of 32 queries.
    const int n_steps = group * ((qend - qbeg + BT2 - 1) / BT2);
    auto next_tile = [&](int qt) { return qt + BT2 >= qend ? qbeg : qt + BT2; };
    auto next_slot = [](uint32_t tile) { return tile == 2 * SLOT ? 0u : tile + SLOT; };
    // whether any of the pair's keys is seen by queries qb .. qb + 31: both wavefronts skip the block otherwise
    auto active = [&](int qb) { return qb < w_hi_max && qb + 32 > w_lo_min; };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
    const uint32_t box0 = lds0 + 3 * SLOT + pair * PDS_BYTES + lane * 16;        // this lane's part of the pair's first buffer

    if (first_of_pair) {
        bf16x8 kf[KS], vf[KS];                         // K and V rows as the MFMA's column operands
        // copied into LDS the way tiles are (whole rows per instruction, rows beyond the pack and features beyond the head's width as
        // zeros) and read back as fragments; loading them straight into the fragment layout takes 16 loads of 16 bytes per row.  The
        // V rows stand in the third slot, which is first written behind the second barrier, the K rows where P and dS go later.
        {
            static_assert(4 * ROWS32_BYTES<D> <= SLOT && 4 * ROWS32_BYTES<D> <= 8 * PDS_BYTES, "room for the staged K and V rows");
            RowCopier<D, ROWS32_BYTES<D> / 1024> cp_kv;
            cp_kv.init(0, ld, dh);
            uint8_t *stage_k = smem + 3 * SLOT + pair * ROWS32_BYTES<D>, *stage_v = smem + 2 * SLOT + pair * ROWS32_BYTES<D>;
            cp_kv.issue(rs_q, stage_k, k0 + pair * 32, ld, nq + g * dh);
            cp_kv.issue(rs_q, stage_v, k0 + pair * 32, ld, nq + nk + g * dh);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                kf[ks] = frag_k<D>(stage_k, l32, ks, half);
                vf[ks] = frag_k<D>(stage_v, l32, ks, half);
            }
        }
        const float sl2 = a.scale * LOG2E;
        const unsigned span = (unsigned)(me.hi - me.lo);
        // LDS addresses, shared by all blocks: row l32 of a tile's first 32, 16-byte unit 2 ks + half; the block's 32 rows are an
        // immediate offset, as the swizzle does not see them
        uint32_t f0[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) f0[ks] = lds0 + (l32 * (D / 8) + ((2 * ks + half) ^ swz_unit<D>(l32))) * 16;
        const uint32_t l0 = lds0 + 2 * TILE + half * 16;
        uint32_t tile = 0;                              // LDS offset of the step's slot
        // block b of the step whose first query is qt
        auto block = [&](auto B_, int qt) {
            constexpr int b = decltype(B_)::value;
            const int qb = qt + 32 * b;
            if (!active(qb)) return;
            // LDS reads in the order they are issued: the score fragments (slice ks of Q, of dO), then the log-sum-exps and D values of
            // the lane's four quads of queries.  AHEAD of them are out at any time; volatile keeps their order, the compiler writes the waits.
            constexpr int NF = 2 * KS, AHEAD = 8;
            bf16x8 fr[NF];
            f32x4 l4[4], d4[4];
            uint32_t fa, la = l0 + tile;
            asm volatile("" : "+v"(la));
            auto issue = [&](auto I_) {
                constexpr int i = decltype(I_)::value;
                if constexpr (i < NF) {
                    if constexpr ((i & 1) == 0) { fa = f0[i >> 1] + tile; asm volatile("" : "+v"(fa)); }      // (one address for both reads)
                    fr[i] = lds_load<bf16x8>(fa + ((i & 1) * TILE + b * 64 * D));
                } else if constexpr (((i - NF) & 1) == 0) l4[(i - NF) / 2] = lds_load<f32x4>(la + (b * 128 + (i - NF) / 2 * 32));
                else d4[(i - NF) / 2] = lds_load<f32x4>(la + (b * 128 + (i - NF) / 2 * 32 + BT2 * 4));
            };
            static_for<0, AHEAD>([&](auto I_) { issue(I_); });
            __builtin_amdgcn_sched_barrier(0);
            f32x16 s = zero16(), dp = zero16();
            static_for<0, NF>([&](auto J_) {
                constexpr int j = decltype(J_)::value;
                if constexpr ((j & 1) == 0) s = MFMA(fr[j], kf[j >> 1], s);
                else dp = MFMA(fr[j], vf[j >> 1], dp);
                issue(std::integral_constant<int, j + AHEAD>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            const bool inside = qb >= w_lo_max && qb + 32 <= w_hi_min;
            const int rel = qb + 4 * half - me.lo;
            uint32_t pp[8], dd[8];
            // two copies of the loop, so that a block no key of which is masked pays nothing for the mask
            auto softmax = [&](auto MASK_) {
                static_for<0, 4>([&](auto Q_) {
                    constexpr int gq = decltype(Q_)::value;
                    float p[4], ds[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        p[e] = __builtin_amdgcn_exp2f(fmaf(s[4 * gq + e], sl2, -l4[gq][e] * LOG2E));
                        if (decltype(MASK_)::value) p[e] = (unsigned)(rel + 8 * gq + e) < span ? p[e] : 0.f;
                        ds[e] = p[e] * (dp[4 * gq + e] + d4[gq][e]);             // the D array holds -D
                    }
                    pp[2 * gq] = pack_bf16x2(p[0], p[1]); pp[2 * gq + 1] = pack_bf16x2(p[2], p[3]);
                    dd[2 * gq] = pack_bf16x2(ds[0], ds[1]); dd[2 * gq + 1] = pack_bf16x2(ds[2], ds[3]);
                });
            };
            if (inside) softmax(std::false_type{});
            else softmax(std::true_type{});
            auto *box = reinterpret_cast<__attribute__((address_space(3))) rawx4 *>((uintptr_t)(box0 + b * 4 * PDS_BYTES));
            box[0] = rawx4{pp[0], pp[1], pp[2], pp[3]};
            box[64] = rawx4{pp[4], pp[5], pp[6], pp[7]};
            box[128] = rawx4{dd[0], dd[1], dd[2], dd[3]};
            box[192] = rawx4{dd[4], dd[5], dd[6], dd[7]};
        };
        int qt = qbeg;
        for (int step = 0; step < n_steps; ++step) {
            lds_barrier();
            block(std::integral_constant<int, 0>{}, qt);
            lds_barrier();
            block(std::integral_constant<int, 1>{}, qt);
            tile = next_slot(tile);
            qt = next_tile(qt);
        }
        lds_barrier();                                 // the last block's P and dS are there
        lds_barrier();                                 // the tiles are done with
        return;
    }

    // ---- the second wavefront of a pair
    f32x16 dk[CB], dv[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) { dk[c] = zero16(); dv[c] = zero16(); }
    const __amdgpu_buffer_rsrc_t rs_do =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(dO), 0, (int)(uint32_t)((size_t)T * nq * 2), 0x00020000);
    // each copies a quarter of the Q tile and of the dO tile; the first two also fetch the 64 log-sum-exps and the 64 D values of the
    // tile's queries (4 bytes per lane; queries >= T read as 0)
    RowCopier<D, COPIES> cp_q, cp_do;
    cp_q.init(pair * COPIES, ld, dh);
    cp_do.init(pair * COPIES, nq, dh);
    // the tile of queries qt .. of `head`, its two halves one after the other
    auto copy_q = [&](uint32_t slot, int head, int qt) { cp_q.issue(rs_q, smem + slot, qt, ld, head * dh); };
    auto copy_do = [&](uint32_t slot, int head, int qt) {
        cp_do.issue(rs_do, smem + slot + TILE, qt, nq, head * dh);
        if (pair < 2) {
            const float *src = (pair == 0 ? a.lse : a.Dsum) + (long)head * T;
            const __amdgpu_buffer_rsrc_t rs_f =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(src), 0, (int)(uint32_t)((size_t)T * 4), 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_f, (lds_void *)(smem + slot + 2 * TILE + pair * BT2 * 4), 4,
                                                     (int)((qt + lane) * 4), 0, 0, 0);
        }
    };
    TrReader<D> tr;
    tr.init(lds0);
    // block b (first query qb) of the tile at LDS offset `tile`
    auto block = [&](auto B_, int qb, uint32_t tile) {
        constexpr int b = decltype(B_)::value;
        if (!active(qb)) return;
        // LDS reads in the order they are issued: P and dS, then groups of four transposing reads, group 4 m + c (m: 16 queries, c: 32
        // features) for one dV and one dK MFMA; three groups are out in front of the first MFMA of each
        constexpr int NG = 2 * CB;
        bf16x8 pf[2], dsf[2];
        shortx4 o[NG][2], q[NG][2];
        const uint32_t box = box0 + b * 4 * PDS_BYTES;
        uint32_t trc[TrReader<D>::N];
#pragma unroll
        for (int x = 0; x < TrReader<D>::N; ++x) trc[x] = tr.off[x] + tile;
        lds_read16<0>(pf[0], box); lds_read16<2048>(dsf[0], box);
        lds_read16<1024>(pf[1], box); lds_read16<3072>(dsf[1], box);
        auto issue = [&](auto G_) {
            constexpr int gi = decltype(G_)::value, m = gi / CB, c = gi % CB;
            o[gi][0] = TrReader<D>::template read_at<b, m, c, 0, TILE>(trc); o[gi][1] = TrReader<D>::template read_at<b, m, c, 1, TILE>(trc);
            q[gi][0] = TrReader<D>::template read_at<b, m, c, 0, 0>(trc); q[gi][1] = TrReader<D>::template read_at<b, m, c, 1, 0>(trc);
        };
        static_for<0, 3>([&](auto G_) { issue(G_); });
        static_for<0, NG>([&](auto G_) {
            constexpr int gi = decltype(G_)::value, m = gi / CB, c = gi % CB, LEFT = NG - 1 - gi < 2 ? NG - 1 - gi : 2;
            asm volatile("s_waitcnt lgkmcnt(%4)" : TR_WAIT2(o[gi]), TR_WAIT2(q[gi]) : "n"(4 * LEFT));
            if constexpr (gi == 0) asm volatile("" : "+v"(pf[0]), "+v"(dsf[0]), "+v"(pf[1]), "+v"(dsf[1]));
            dv[c] = MFMA(join(o[gi][0], o[gi][1]), pf[m], dv[c]);
            dk[c] = MFMA(join(q[gi][0], q[gi][1]), dsf[m], dk[c]);
            if constexpr (gi + 3 < NG) issue(std::integral_constant<int, gi + 3>{});
        });
    };
    int head = h_first, qt_copy = qbeg;                // of the tile that is copied next
    auto copied = [&]() {
        if (qt_copy + BT2 >= qend) ++head;
        qt_copy = next_tile(qt_copy);
    };
    copy_q(0, head, qt_copy); copy_do(0, head, qt_copy);
    copied();
    if (n_steps > 1) { copy_q(SLOT, head, qt_copy); copy_do(SLOT, head, qt_copy); copied(); }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // Barrier 2 t stands in front of the first wavefront's block 0 of step t (tile t has landed, block 1 of step t - 1 is in its
    // buffer), barrier 2 t + 1 in front of its block 1.  Behind the latter nobody reads tile t - 1 any more: its slot is tile t + 2's,
    // whose Q rows are requested there and whose dO rows behind the next barrier.
    uint32_t tile = 0, before = 2 * SLOT;              // slots of tiles t and t - 1 (which is tile t + 2's)
    int qt_now = qbeg, qt_before = qbeg;
    for (int step = 0; step < n_steps; ++step) {
        lds_barrier();
        if (step > 0) {
            if (step + 1 < n_steps) { copy_do(next_slot(tile), head, qt_copy); copied(); }
            block(std::integral_constant<int, 1>{}, qt_before + 32, before);
        }
        lds_barrier();
        if (step + 2 < n_steps) copy_q(before, head, qt_copy);
        block(std::integral_constant<int, 0>{}, qt_now, tile);
        // tile t + 1 has landed; the copies of Q for tile t + 2 may be in flight (memory operations retire in order)
        if (step + 2 < n_steps) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        before = tile;
        tile = next_slot(tile);
        qt_before = qt_now;
        qt_now = next_tile(qt_now);
    }
    lds_barrier();
    block(std::integral_constant<int, 1>{}, qt_before + 32, before);
    lds_barrier();                                     // the tiles are done with: LDS now stages the output rows
    store_dkv<D, CB>(a, smem, pair, half, g, k0 + pair * 32, key, valid, dk, dv);
    if (a.cu_busy && wv == 4 && lane == 0) atomicAdd(a.cu_busy + 2048 + (__smid() & 1023u), wall_clock64());
}

// ------------------------------------------------------------------------------------------
// backward: dK, dV, the plain form: a block's scores, its softmax and its products one after the other, two LDS
// slots.  Used for the 64-wide head, where it fits 256 registers, so that two workgroups share a compute unit
// and overlap each other's phases.  PARTS = 2: two
// groups of 4 wavefronts with the same 128 keys and every other (head, query tile) step each (see two_parts).
// ------------------------------------------------------------------------------------------
template <int D, int PARTS>
__global__ __launch_bounds__(PARTS * 256, PARTS) void attn_dkv_plain_kernel(AttnArgs a) {
    constexpr int KS = D / 16, CB = D / 32;
    constexpr int TILE = BT2 * D * 2, SLOT = 2 * TILE + 2 * BT2 * 4;   // Q tile, dO tile, lse[64], D[64]
    constexpr int COPIES = BT2 * D * 2 / 1024 / 4;                     // per wavefront and tile
    extern __shared__ __attribute__((aligned(16))) uint8_t smem_all[];
    add_busy(a.cu_busy ? a.cu_busy + 2048 : nullptr, false);

    // grid: x = key/value head, y = position in the dispatch order of the key tiles (heaviest first), z = this workgroup's share
    // of the group's query heads
    const int g = blockIdx.x, group_heads = a.nh / a.nkv;
    const int h_first = g * group_heads + blockIdx.z * group_heads / a.dkv_parts;
    const int group = g * group_heads + (blockIdx.z + 1) * group_heads / a.dkv_parts - h_first;
    const int k0 = (a.use_order ? a.order_k[blockIdx.y] : blockIdx.y) * BQ;
    // the wavefront's index as a scalar: what is derived from it (copy destinations, buffer descriptors) stays uniform
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5, l32 = lane & 31;
    const int part = PARTS == 1 ? 0 : wv >> 2, wave = PARTS == 1 ? wv : wv & 3;
    uint8_t *const smem = smem_all + part * DKV_PLAIN_LDS<D>;
    const int T = a.T;
    const bf16_t *qkv = (const bf16_t *)a.qkv;
    const bf16_t *dO = (const bf16_t *)a.d_o;
    const long ld = a.ld_qkv;
    const int dh = a.d;                                 // head dimension in memory (<= D: LDS tiles and fragments are zero-padded to D)
    const int nq = a.nh * dh, nk = a.nkv * dh;

    const int key = k0 + wave * 32 + l32;
    RowInfo me, first, last;                                // queries [lo, hi) see this key
    ranges<true>(a, k0, BQ, k0 + wave * 32, me, first, last);
    const bool valid = key < T;
    const WaveBounds wb = wave_bounds(me, k0 + wave * 32, T);
    const int w_lo_min = wb.lo_min, w_lo_max = wb.lo_max, w_hi_max = wb.hi_max, w_hi_min = wb.hi_min;
    const int qbeg = first.lo, qend = last.hi;

    bf16x8 kf[KS], vf[KS];                             // this wavefront's K and V rows as MFMA operands (filled below)
    f32x16 dk[CB], dv[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) { dk[c] = zero16(); dv[c] = zero16(); }
    const float sl2 = a.scale * LOG2E;

    const __amdgpu_buffer_rsrc_t rs_q =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(qkv), 0, (int)(uint32_t)((size_t)T * ld * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_do =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(dO), 0, (int)(uint32_t)((size_t)T * nq * 2), 0x00020000);
    // every wavefront copies a quarter of the Q tile and of the dO tile; wavefronts 0 and 1 also fetch the
    // 64 log-sum-exps and the 64 D values of the tile's queries (4 bytes per lane; queries >= T read as 0)
    RowCopier<D, COPIES> cp_q, cp_do;
    cp_q.init(wave * COPIES, ld, dh);
    cp_do.init(wave * COPIES, nq, dh);
    auto copy_tile = [&](uint8_t *slot, int head, int qt) {
        cp_q.issue(rs_q, slot, qt, ld, head * dh);
        cp_do.issue(rs_do, slot + TILE, qt, nq, head * dh);
        if (wave < 2) {
            const float *src = (wave == 0 ? a.lse : a.Dsum) + (long)head * T;
            const __amdgpu_buffer_rsrc_t rs_f =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(src), 0, (int)(uint32_t)((size_t)T * 4), 0x00020000);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_f, (lds_void *)(slot + 2 * TILE + wave * BT2 * 4), 4,
                                                     (int)((qt + lane) * 4), 0, 0, 0);
        }
    };
    TrReader<D> tr;
    tr.init((uint32_t)(uintptr_t)(lds_void *)smem);

    if (qbeg >= qend) goto done;      // no query sees these keys (cannot happen for a key of a segment: it sees itself)
    {
    // the (head, query tile) pairs form one sequence; the copy of the next pair is in flight during this one
    const int tiles_per_head = (qend - qbeg + BT2 - 1) / BT2, n_steps = group * tiles_per_head;
    // the K and V rows go through LDS as in the kernel above, behind the two slots
    {
        RowCopier<D, ROWS32_BYTES<D> / 1024> cp_kv;
        cp_kv.init(0, ld, dh);
        uint8_t *stage_k = smem + 2 * SLOT + wave * 2 * ROWS32_BYTES<D>, *stage_v = stage_k + ROWS32_BYTES<D>;
        cp_kv.issue(rs_q, stage_k, k0 + wave * 32, ld, nq + g * dh);
        cp_kv.issue(rs_q, stage_v, k0 + wave * 32, ld, nq + nk + g * dh);
        if (part < n_steps) copy_tile(smem, h_first + part / tiles_per_head, qbeg + (part % tiles_per_head) * BT2);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            kf[ks] = frag_k<D>(stage_k, l32, ks, half);
            vf[ks] = frag_k<D>(stage_v, l32, ks, half);
        }
    }
    int slot = 0;
    for (int step = part; step - part < n_steps; step += PARTS, slot ^= 1) {
        const int qt = qbeg + (step % tiles_per_head) * BT2;
        const uint8_t *sQ = smem + slot * SLOT, *sdO = sQ + TILE;
        const float *sLse = reinterpret_cast<const float *>(sQ + 2 * TILE), *sD = sLse + BT2;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this step's tiles have landed
        lds_barrier();                                               // ... and everyone is done with the other slot
        if (step + PARTS < n_steps) {
            const int nh2 = (step + PARTS) / tiles_per_head, nqt = qbeg + ((step + PARTS) % tiles_per_head) * BT2;
            copy_tile(smem + (slot ^ 1) * SLOT, h_first + nh2, nqt);
        }
        if (PARTS == 2 && step >= n_steps) break;                    // the second group's last step of an odd number
        auto block = [&](auto B_) {
            constexpr int b = decltype(B_)::value;
            const int qb = qt + 32 * b;
            if (!((qb < w_hi_max) && (qb + 32 > w_lo_min))) return;
            // S[q, key] and dP[q, key]: rows = queries (registers), columns = keys (lanes); as assembly, so that the
            // results land in vector registers (see mfma_v), with the wait the vector ALU needs before it reads them
            f32x16 s, dp;
            static_for<0, KS>([&](auto K_) {
                constexpr int ks = decltype(K_)::value;
                const bf16x8 fq = frag_k<D>(sQ, 32 * b + l32, ks, half), fo = frag_k<D>(sdO, 32 * b + l32, ks, half);
                if constexpr (ks == 0) { mfma_v_first(s, fq, kf[0]); mfma_v_first(dp, fo, vf[0]); }
                else { mfma_v(s, fq, kf[ks]); mfma_v(dp, fo, vf[ks]); }
            });
            mfma_results_settle();
            const uint32_t tq = slot * SLOT, tdo = tq + TILE;
            // dO^T and Q^T fragments of MFMA 0 of the block
            shortx4 o0[4], o1[4], q0f[4], q1f[4];
            auto read_m = [&](auto M_) {
                constexpr int m = decltype(M_)::value;
                o0[0] = tr.template read<b, m, 0, 0>(tdo); o1[0] = tr.template read<b, m, 0, 1>(tdo);
                q0f[0] = tr.template read<b, m, 0, 0>(tq); q1f[0] = tr.template read<b, m, 0, 1>(tq);
                o0[1] = tr.template read<b, m, 1, 0>(tdo); o1[1] = tr.template read<b, m, 1, 1>(tdo);
                q0f[1] = tr.template read<b, m, 1, 0>(tq); q1f[1] = tr.template read<b, m, 1, 1>(tq);
                if constexpr (CB > 2) {
                    o0[2] = tr.template read<b, m, 2, 0>(tdo); o1[2] = tr.template read<b, m, 2, 1>(tdo);
                    q0f[2] = tr.template read<b, m, 2, 0>(tq); q1f[2] = tr.template read<b, m, 2, 1>(tq);
                    o0[3] = tr.template read<b, m, 3, 0>(tdo); o1[3] = tr.template read<b, m, 3, 1>(tdo);
                    q0f[3] = tr.template read<b, m, 3, 0>(tq); q1f[3] = tr.template read<b, m, 3, 1>(tq);
                } else {
                    o0[2] = o0[3] = o1[2] = o1[3] = q0f[2] = q0f[3] = q1f[2] = q1f[3] = shortx4{0, 0, 0, 0};
                }
            };
            read_m(std::integral_constant<int, 0>{});
            const bool inside = qb >= w_lo_max && qb + 32 <= w_hi_min;
            const unsigned span = (unsigned)(me.hi - me.lo);
            float p[16], ds[16];
            // two copies of the loop, so that a block no key of which is masked pays nothing for the mask
            auto softmax = [&](auto MASK_) {
                constexpr bool MASK = decltype(MASK_)::value;
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const int r0 = 32 * b + 8 * gq + 4 * half;        // 4 consecutive queries
                    const float4 l4 = *reinterpret_cast<const float4 *>(sLse + r0);
                    const float4 d4 = *reinterpret_cast<const float4 *>(sD + r0);
                    const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dvv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int i = 4 * gq + e;
                        float pv = __builtin_amdgcn_exp2f(fmaf(s[i], sl2, -lv[e] * LOG2E));
                        if (MASK) pv = (unsigned)(qt + r0 + e - me.lo) < span ? pv : 0.f;
                        p[i] = pv;
                        ds[i] = pv * (dp[i] + dvv[e]);                 // the D array holds -D
                    }
                }
            };
            if (inside) softmax(std::false_type{});
            else softmax(std::true_type{});
            asm volatile("s_waitcnt lgkmcnt(0)" : TR_WAIT4(o0), TR_WAIT4(o1), TR_WAIT4(q0f), TR_WAIT4(q1f));
            bf16x8 fo[4], fq[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) { fo[c] = join(o0[c], o1[c]); fq[c] = join(q0f[c], q1f[c]); }
            read_m(std::integral_constant<int, 1>{});                 // in flight during the next 2 CB MFMAs
            {
                const bf16x8 pf = pack8(p), dsf = pack8(ds);
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    dv[c] = MFMA(fo[c], pf, dv[c]);
                    dk[c] = MFMA(fq[c], dsf, dk[c]);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" : TR_WAIT4(o0), TR_WAIT4(o1), TR_WAIT4(q0f), TR_WAIT4(q1f));
            {
                const bf16x8 pf = pack8(p + 8), dsf = pack8(ds + 8);
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    dv[c] = MFMA(join(o0[c], o1[c]), pf, dv[c]);
                    dk[c] = MFMA(join(q0f[c], q1f[c]), dsf, dk[c]);
                }
            }
        };
        block(std::integral_constant<int, 0>{});
        block(std::integral_constant<int, 1>{});
    }
    }
done:
    lds_barrier();                                     // the tiles are done with: LDS now stages the output rows
    uint8_t *stage = smem_all;
    if constexpr (PARTS == 2) {
        uint8_t *box = smem_all + wave * 2 * XCHG_BYTES<16 * CB>;
        stage += 8 * XCHG_BYTES<16 * CB>;
        if (part == 1) {
            put_acc(box, dk);
            put_acc(box + XCHG_BYTES<16 * CB>, dv);
        }
        lds_barrier();
        if (part == 1) return;
        merge_acc(box, dk, 1.f, 1.f);
        merge_acc(box + XCHG_BYTES<16 * CB>, dv, 1.f, 1.f);
    }
    store_dkv<D, CB>(a, stage, wave, half, g, k0 + wave * 32, key, valid, dk, dv);
    add_busy(a.cu_busy ? a.cu_busy + 2048 : nullptr, true);
}

template <typename K>
hipError_t set_smem(K kern, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// Wavefronts per workgroup of the forward and dQ kernels: four (128 queries, two workgroups per compute unit) or eight (256, one).
// Four split the pack more finely: more compute units at work on short packs, less masked work on short segments, a smaller
// last round.  Eight fetch every K / V tile half as often, which tells where query tiles walk many keys and there are tiles
// enough for both.  64-wide heads always take four (encoder packs: forward 0.068 -> 0.054 ms; dQ + dK/dV 144 -> 131 us on 3000
// bidirectional tokens, 136 -> 136 us on 8192).  Wider ones, forward / backward us with eight -> four: 1031 causal tokens of 32
// heads in 4 segments 29 / 65 -> 25 / 63, 3000 in one long document 88 / 270 -> 79 / 263, 8192 in segments of 700
// 114 / 396 -> 111 / 398; but 8192 in one long document (60 steps of 64 keys per tile on average) 478 / 1593 -> 497 / 1621, and
// 4111 (30 steps, 544 workgroups) 137 / 449 -> 143 / 456.
template <int D>
bool four_waves(const AttnArgs &a) {
    const long tiles = ceil_div(a.T, FQ);
    return D <= 64 || tiles * a.nh < 512 || (a.q_steps > 0 && a.q_steps <= 14 * tiles);
}

// Two groups of four wavefronts per workgroup, each with every other 64-row step of the same 128 queries (keys) and their partial
// results merged at the end: where 128 rows per workgroup do not even give every compute unit two workgroups, a workgroup's chain
// of steps is what a launch takes, one wavefront per SIMD has nothing to hide its waits, and the halved chain pays for the merge.
// With two workgroups per compute unit and more it is the other way round.  Forward / dQ + dK/dV in us, one -> two groups:
// 16 heads of 64, 576 tokens 14 / 34 -> 12 / 29, 2304 in a long document (288 workgroups) 36 / 103 -> 28 / 76, 3500 (448) 52 / 152
// -> 40 / 113; 16 of 80, 3500 42 / 113 -> 40 / 111; 32 of 128 (whose dK/dV kernel has no such form), 1031 (288) 25 / 62 -> 21 / 55,
// 1500 (384) 31 / 78 -> 25 / 70; but 2304 (576) 33 / 98 -> 38 / 103 and 64 heads of 128, 1031 (576) 28 / 94 -> 30 / 94.
bool two_parts(long workgroups) { return workgroups <= 512; }

template <int D, int KS, int CB, int W, int PARTS>
hipError_t launch_fwd(const AttnArgs &a, hipStream_t st) {
    static std::atomic<bool> configured{false};     // set once; concurrent first calls repeat the same idempotent set-up
    constexpr int XCHG = PARTS == 1 ? 0 : W * XCHG_BYTES<16 * CB + 2>;
    const int smem = std::max(PARTS * FWD_LDS_BYTES<D, W>, XCHG + W * STAGE_BYTES<D>);
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = set_smem(attn_fwd_kernel<D, KS, CB, W, PARTS>, smem);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    attn_fwd_kernel<D, KS, CB, W, PARTS><<<dim3(a.nh, ceil_div(a.T, FQ) * (FQ / (W * 32))), W * PARTS * 64, smem, st>>>(a);
    return hipGetLastError();
}
template <int D, int KS, int CB, int W, int PARTS>
hipError_t launch_dq(const AttnArgs &a, hipStream_t st) {
    static std::atomic<bool> configured{false};
    constexpr int XCHG = PARTS == 1 ? 0 : W * XCHG_BYTES<16 * CB>;
    const int smem = std::max(PARTS * DQ_LDS_BYTES<D, W>, XCHG + W * STAGE_BYTES<D>);
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = set_smem(attn_dq_kernel<D, KS, CB, W, PARTS>, smem);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    attn_dq_kernel<D, KS, CB, W, PARTS><<<dim3(a.nh, ceil_div(a.T, FQ) * (FQ / (W * 32))), W * PARTS * 64, smem, st>>>(a);
    return hipGetLastError();
}
template <int D, int PARTS>
hipError_t launch_dkv_plain(const AttnArgs &a, const dim3 &grid, hipStream_t st) {
    static std::atomic<bool> configured{false};
    static_assert(8 * XCHG_BYTES<D / 2> + 4 * STAGE32_BYTES<D> <= 2 * DKV_PLAIN_LDS<D> && 4 * STAGE32_BYTES<D> <= DKV_PLAIN_LDS<D>,
                  "room for the exchange and the staged rows");
    if (!configured.load(std::memory_order_acquire)) {
        hipError_t e = set_smem(attn_dkv_plain_kernel<D, PARTS>, PARTS * DKV_PLAIN_LDS<D>);
        if (e != hipSuccess) return e;
        configured.store(true, std::memory_order_release);
    }
    attn_dkv_plain_kernel<D, PARTS><<<grid, PARTS * 256, PARTS * DKV_PLAIN_LDS<D>, st>>>(a);
    return hipGetLastError();
}

template <int D, int KS, int CB>
hipError_t launch_fwd(const AttnArgs &a, hipStream_t st) {
    if (two_parts((long)a.nh * ceil_div(a.T, 128))) return launch_fwd<D, KS, CB, 4, 2>(a, st);
    if constexpr (D > 64)
        if (!four_waves<D>(a)) return launch_fwd<D, KS, CB, 8, 1>(a, st);
    return launch_fwd<D, KS, CB, 4, 1>(a, st);
}

template <int D, int KS, int CB>
hipError_t launch_bwd(const AttnArgs &a, hipStream_t st) {
    hipError_t e;
    if (two_parts((long)a.nh * ceil_div(a.T, 128))) e = launch_dq<D, KS, CB, 4, 2>(a, st);
    else if (four_waves<D>(a)) e = launch_dq<D, KS, CB, 4, 1>(a, st);
    else if constexpr (D > 64) e = launch_dq<D, KS, CB, 8, 1>(a, st);
    if (e != hipSuccess) return e;
    const dim3 grid(a.nkv, ceil_div(a.T, BQ), a.dkv_parts);
    if constexpr (D <= 64) {                            // the plain form (see attn_dkv_plain_kernel)
        if (two_parts((long)grid.x * grid.y * grid.z)) e = launch_dkv_plain<D, 2>(a, grid, st);
        else e = launch_dkv_plain<D, 1>(a, grid, st);
    } else {
        static std::atomic<bool> configured{false};
        static_assert(4 * STAGE32_BYTES<D> <= DKV_PAIR_LDS<D>, "room for the staged fp32 rows");
        if (!configured.load(std::memory_order_acquire)) {
            if ((e = set_smem(attn_dkv_kernel<D, KS, CB>, DKV_PAIR_LDS<D>)) != hipSuccess) return e;
            configured.store(true, std::memory_order_release);
        }
        attn_dkv_kernel<D, KS, CB><<<grid, 512, DKV_PAIR_LDS<D>, st>>>(a);
    }
    if (a.dkv_parts > 1) dkv_reduce_kernel<<<ceil_div((long)a.T * 2 * a.nkv * (a.d / 8), 256), 256, 0, st>>>(a);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace

hipError_t attn_mfma_fwd(const AttnArgs &a, hipStream_t st) {
    if (a.T == 0) return hipSuccess;
    if ((size_t)a.T * a.ld_qkv * 2 >= MAX_TENSOR_BYTES) return hipErrorInvalidValue;
    return a.d <= 64 ? launch_fwd<64, 4, 2>(a, st) : a.d <= 80 ? launch_fwd<128, 5, 3>(a, st) : a.d <= 96 ? launch_fwd<128, 6, 3>(a, st)
                                                                                             : launch_fwd<128, 8, 4>(a, st);
}

// Workgroups that share a group's query heads in the dK/dV kernels.  One workgroup per 128 keys and key/value head walks all
// heads of the group one after the other: 64 query on 8 key/value heads over 2047 tokens are 128 workgroups for 256 compute
// units, each with a chain of up to 96 steps.  Shared out, each writes fp32 partial sums (dkv_reduce_kernel adds them in order),
// which costs 16 bytes per key, head and feature pair.  Only divisors of the group, so that the shares are equal (8 heads over 3
// workgroups: 8 % slower than over 2), and as many as give two workgroups per compute unit, one at a time (128-wide heads), or
// six, two at a time.  dQ + dK/dV in us, 64 / 8 heads of 128, one causal segment, without -> with: 500 tokens 116 -> 53 (8 workgroups per
// group), 1031 232 -> 109 (4), 2047 460 -> 301 (4), 4096 1127 -> 906 (2), 6000 2053 -> 1952 (2), where one and a half rounds become three; at 8192
// tokens (512 workgroups as they are) two would gain 4 to 8 % for 134 MB of scratch, at 12000 nothing (these two with one wavefront per 32
// keys).  32 / 8 heads, 2047 tokens: 247 -> 175.  16 / 2 heads of 64, 2047 tokens: 294 -> 80 (8).
static long longest_shared(long parts, int nkv, int d) {              // the longest pack whose groups are shared out over `parts` workgroups
    const long tiles = d <= 64 ? 1536 / (parts * nkv) : (parts == 2 ? 384 : std::min(384l, 512 / parts)) / nkv;
    return std::min(tiles * BQ, (long)(DKV_PART_BYTES_MAX / (parts * attn_dkv_part_bytes(1, nkv, d))));
}
int attn_dkv_parts(int T, int nh, int nkv, int d) {
    int parts = 1;
    for (int p = 2; p <= nh / nkv; ++p)
        if (nh / nkv % p == 0 && T <= longest_shared(p, nkv, d)) parts = p;
    return parts;
}
size_t attn_dkv_room(int T, int nh, int nkv, int d) {
    size_t most = 0;
    for (int p = 2; p <= nh / nkv; ++p)
        if (nh / nkv % p == 0) most = std::max(most, p * attn_dkv_part_bytes((int)std::min((long)T, longest_shared(p, nkv, d)), nkv, d));
    return most;
}

hipError_t attn_mfma_bwd(const AttnArgs &args, hipStream_t st) {
    if (args.T == 0) return hipSuccess;
    if ((size_t)args.T * args.ld_qkv * 2 >= MAX_TENSOR_BYTES) return hipErrorInvalidValue;
    AttnArgs a = args;
    a.dkv_parts = attn_dkv_parts(a.T, a.nh, a.nkv, a.d);
    if (a.dkv_parts > 1 && a.dkv_part_bytes < a.dkv_parts * attn_dkv_part_bytes(a.T, a.nkv, a.d)) a.dkv_parts = 1;
    return a.d <= 64 ? launch_bwd<64, 4, 2>(a, st) : a.d <= 80 ? launch_bwd<128, 5, 3>(a, st) : a.d <= 96 ? launch_bwd<128, 6, 3>(a, st)
                                                                                             : launch_bwd<128, 8, 4>(a, st);
}

}  // namespace mmt
