// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulation.
//
//   C[M,N] (+)= opA(A) . opB(B) (+ bias[N]) (+ residual[M,N])
//
// Tiling.  One 256-thread workgroup (4 wavefronts, one per SIMD, 2 x 2) owns a tile of C, 256 x 256 in
// the largest shape: each wavefront then owns a 128x128 quadrant as 8x8 MFMA tiles of 16x16 (256
// accumulator registers per lane).  K advances in steps of 64; the operand tiles (256 rows x 64 k = 32 KiB) of
// successive steps go round two rings of LDS slots, three for A and two for B, which is all of the CU's
// 160 KiB.  Smaller tile shapes (TileShape) trade operand traffic for more workgroups and look further ahead.
//
// Global -> LDS.  Every operand tile is copied 16 bytes per lane directly into LDS (buffer_load ... lds:
// no register staging, no LDS write instructions), in the operand's own memory order, so weight- and
// input-gradient GEMMs need no transposed copies in HBM and no transposes in registers:
//   * operands whose contraction index is contiguous in memory (A of NT/NN, B of NT) are kept as
//     tile[row][64 k] (128 bytes = eight 16-byte units per row).  Unit u of row r is stored at unit
//     position u ^ (r & 7).  A fragment read (lane l: row l & 15, unit 4 s + (l >> 4), 16 bytes) is served 16
//     lanes at a time, lanes 0-7 together with 24-31 and 8-15 with 16-23 (measured), at full rate if those fall
//     into 16 distinct 16-byte slots modulo 256 bytes: rows 0-7 of one unit and rows 8-15 of its neighbour do
//     with this swizzle (with (r ^ (r >> 3)) & 7, which suits 32-row fragments, they ran at half rate);
//   * operands whose contraction index is the row index in memory (B of NN, A and B of TN) are kept as
//     tile[64 k][rows] (512 bytes per k for 256 rows) and the fragments are formed by the transposing LDS read
//     ds_read_b64_tr_b16; 32-byte chunks are XOR-swizzled with k & 3 against bank conflicts.
// k out of range is zero-filled by the buffer descriptor's bounds check; rows out of range meet only outputs that are not stored.
//
// Epilogue.  Accumulators go through a per-wavefront fp32 LDS staging area so that C,
// residual and bias are accessed as full 16-byte row-major vectors; bias / residual / previous
// C (accumulate) are added in fp32 before the single rounding to bf16.
//
// Workgroup -> tile map.  The kernel is persistent: one workgroup per compute unit walks over
// several tiles, so the output stores of one tile drain while the next tile is already being
// multiplied.  Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2; each
// XCD works on a contiguous run of the tile order, which goes in column-major groups of 8
// tile-rows so that concurrently resident tiles share A and B panels.
#pragma once
#include "kernels.h"
#include "reduce.h"
#include <atomic>
#include <utility>
#include <type_traits>

namespace mmt {
namespace gemm_detail {

constexpr int BK = 64;
constexpr int GROUP_M = 8;

// Tile of a workgroup: 2 x 2 wavefronts, each RA x RB blocks of 16 x 16; AHEAD = how many K steps ahead the operand
// tiles are requested.  LDS holds AHEAD + 1 A tiles and AHEAD B tiles.
template <int RA_, int RB_, int AHEAD_>
struct TileShape {
    static constexpr int RA = RA_, RB = RB_, AHEAD = AHEAD_;
    static constexpr int BM = 32 * RA, BN = 32 * RB;
    static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    static constexpr int EPI_PITCH = 16 * RB + 4;                     // floats per staged row
    static constexpr int RING_BYTES = (AHEAD + 1) * A_BYTES + AHEAD * B_BYTES;
    static constexpr int EPI_BYTES = 4 * 32 * EPI_PITCH * 4;
    static constexpr int SMEM = RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES;
    static constexpr int PER_CU = 160 * 1024 / SMEM < 4 ? 160 * 1024 / SMEM : 4;     // workgroups a compute unit holds
};
typedef TileShape<8, 8, 2> Tile256;           // 160 KiB: all of the compute unit's LDS

struct GemmP {
    int M, N, K;
    const bf16_t *A; int lda;
    const bf16_t *B; int ldb;
    bf16_t *C; int ldc;
    const bf16_t *bias;
    const bf16_t *residual;
    int accumulate;
    int c_f32;                 // C holds fp32 (weight gradients into fp32 main-gradient buffers)
    int tiles_m, tiles_n;
    // split K (fp32 output only): the K range is cut into `splits` chunks of k_chunk (a multiple of 64); chunk s of
    // every tile is a work item of its own, its partial product goes to the s-th M x ldc matrix from C on
    int splits, k_chunk;
    // A launch covers tiles [tile_begin, tile_begin + tile_count) of the tile order.  With `compact` (fp32 output, 256 x 256
    // tiles) the partial product of chunk s of the launch's tile j is a dense block at C + (s * tile_count + j) * 65536
    // instead of a window of an M x N matrix.
    int tile_begin, tile_count, compact;
    int late_start;            // units of 512 clocks that every second workgroup waits at its start
    unsigned long long *clock_probe;       // see GemmArgs
};

// Several products of one layout and epilogue in one launch (the weight gradients of a narrow layer, each with too few
// tiles to fill the chip): the work items of problem i are [first[i], first[i + 1]); first[i] for i >= n is the total.
constexpr int MAX_GROUP = 4;
// workgroups that add up sums riding along, a unit of 32 columns at a time (8 arrays of a 1024-wide encoder layer: 416 units)
constexpr int GROUP_SUM_WORKGROUPS = 64;
struct GemmGroup {
    GemmP p[MAX_GROUP];
    int first[MAX_GROUP + 1];
    int n;
    // Sums that ride along: the workgroups behind the first `workgroups` add these up, on compute units that have no tile (any more)
    int workgroups;
    ReduceJobSet reduce;
};
// what the kernel needs from its argument, for one product or a group
__device__ __forceinline__ const GemmP &first_problem(const GemmP &a) { return a; }
__device__ __forceinline__ const GemmP &first_problem(const GemmGroup &a) { return a.p[0]; }
__device__ __forceinline__ int gemm_workgroups(const GemmP &) { return gridDim.x; }
__device__ __forceinline__ int gemm_workgroups(const GemmGroup &a) { return a.workgroups; }
__device__ __forceinline__ int work_items(const GemmP &a, bool split) { return a.tile_count * (split ? a.splits : 1); }
__device__ __forceinline__ int work_items(const GemmGroup &a, bool) { return a.first[MAX_GROUP]; }
// work item `logical` of the launch -> its problem and its index among that problem's items
__device__ __forceinline__ GemmP pick(const GemmP &a, int logical, int &local) { local = logical; return a; }
__device__ __forceinline__ GemmP pick(const GemmGroup &a, int logical, int &local) {
    GemmP p = a.p[0];
    local = logical;
    if (logical >= a.first[1]) { p = a.p[1]; local = logical - a.first[1]; }
    if (logical >= a.first[2]) { p = a.p[2]; local = logical - a.first[2]; }
    if (logical >= a.first[3]) { p = a.p[3]; local = logical - a.first[3]; }
    return p;
}

// position t of the tile order -> tile coordinates: column-major inside groups of GROUP_M tile-rows
__device__ __forceinline__ void tile_coords(int t, int tiles_m, int tiles_n, int &tm, int &tn) {
    const int width = GROUP_M * tiles_n;
    const int group = t / width, first_m = group * GROUP_M;
    const int gsize = min(tiles_m - first_m, GROUP_M);
    tm = first_m + (t % width) % gsize;
    tn = (t % width) / gsize;
}

__device__ __forceinline__ int swz(int row) { return row & 7; }

// Global memory is read through raw buffer descriptors: an access whose byte offset lies at or beyond
// the descriptor's size returns zero, which is how out-of-range rows and the K tail are zero-filled
// without branches.
constexpr uint32_t OOB = 0xfffffff0u;
constexpr int STREAMING = 2;                      // cache policy of a buffer store: nt
typedef __attribute__((ext_vector_type(4))) uint32_t rawx4;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)bytes, 0x00020000);
}
// the descriptor make_rsrc builds, as four scalar words
__device__ __forceinline__ rawx4 raw_rsrc(const void *p, size_t bytes) {
    const uint64_t a = (uint64_t)p;
    rawx4 r;
    r[0] = __builtin_amdgcn_readfirstlane((uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu);
    r[2] = __builtin_amdgcn_readfirstlane((uint32_t)bytes);
    r[3] = 0x00020000u;
    return r;
}
__device__ __forceinline__ uint4 buf_load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
    const rawx4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// K-contiguous operand: X[rows, K] row-major, copied global -> LDS without passing through registers
// (buffer_load ... lds).  One such instruction writes lane l's 16 bytes to LDS base + 16 l, i.e. one
// instruction fills 8 consecutive tile rows (1 KiB); the swizzled layout is obtained by choosing which
// 16-byte unit of the row each lane fetches: lane l of the slab starting at row r0 (a multiple of 8) fetches unit
// (l & 7) ^ swz(r0 + (l >> 3)) = (l & 7) ^ (l >> 3).  Wavefront w copies rows 32 i + 8 w .. + 7 for every item i.
typedef __attribute__((address_space(3))) void lds_void;
template <int NB>                                  // 32 NB rows
struct LoaderKC {
    static constexpr int ITEM_LDS = 32 * 128;      // LDS bytes between consecutive items
    __amdgpu_buffer_rsrc_t rs;
    rawx4 rsv;                    // the same descriptor as four words, for the copies written as assembly
    uint32_t vo[NB];              // this lane's byte offset for item i, without k0
    __device__ __forceinline__ uint32_t step_soff(int k0) const { return (uint32_t)k0 * 2u; }
    int kc0, K, slab0;            // unit column (elements) this lane fetches; first slab's LDS offset
    // Rows beyond the matrix read as zero on the fast path too: their offset lies at or beyond the descriptor's size
    // whatever k is added.
    __device__ __forceinline__ void init(const bf16_t *X, int ld, int row0, int nrows, int K_) {
        rs = make_rsrc(X, ((size_t)(nrows - 1) * ld + K_) * 2);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        K = K_;
        kc0 = (((lane & 7) ^ (lane >> 3)) & 7) * 8;
        const uint32_t off0 = (uint32_t)((size_t)(row0 + w * 8 + (lane >> 3)) * ld * 2) + (uint32_t)kc0 * 2u;
        const uint32_t row_step = (uint32_t)ld * 64u;
        slab0 = __builtin_amdgcn_readfirstlane(w * 8 * 128);
        // one register per item, kept there (recomputed inside the K loop they would cost a vector add per copy)
#pragma unroll
        for (int i = 0; i < NB; ++i) { vo[i] = off0 + (uint32_t)i * row_step; asm volatile("" : "+v"(vo[i])); }
        rsv = raw_rsrc(X, ((size_t)(nrows - 1) * ld + K_) * 2);
    }
    // item i of the tile at k0: rows 32 i + 8 w .. + 7 -> LDS.  FAST: the caller guarantees k0 + 64 <= K; then the per-lane
    // offset is a constant and the rest of the address is a scalar, so no vector instruction precedes the copy (a copy that
    // has to wait for the vector ALU to deliver its address holds up the MFMAs queued behind it).
    template <bool FAST>
    __device__ __forceinline__ void copy_one(uint8_t *tile, int k0, int i) const {
        lds_void *dst = (lds_void *)(tile + slab0 + i * ITEM_LDS);
        if (FAST) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, (int)vo[i], __builtin_amdgcn_readfirstlane(k0 * 2), 0, 0);
        } else {
            const uint32_t off = k0 + kc0 < K ? vo[i] + (uint32_t)k0 * 2u : OOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, (int)off, 0, 0, 0);
        }
    }
    template <bool FAST>
    __device__ __forceinline__ void copy_all(uint8_t *tile, int k0) const {
#pragma unroll
        for (int i = 0; i < NB; ++i) copy_one<FAST>(tile, k0, i);
    }
};

// K-strided operand: X[K, rows] row-major.  It is copied global -> LDS in its memory order, tile[k][row]
// with 64 NB bytes per k, by the same direct copies (one instruction = 16 / NB k-rows), and the MFMA fragments
// are formed by the transposing LDS read (ds_read_b64_tr_b16): 16 lanes read a 4(k) x 16(row) block, 8
// bytes per lane, and lane j of the 16 receives the 4 k-values of row j.  Two such reads give a lane its
// 8 consecutive k.  The 32-byte chunk c of k-row k is stored at chunk position c ^ (k & 3), so that the 4
// k-rows of one block fall into different banks; the copy chooses which chunk each lane fetches.
// Wavefront w copies k-rows 16 w .. + 15, 16 / NB of them per item.
typedef __attribute__((ext_vector_type(4))) short shortx4;
typedef __attribute__((ext_vector_type(8))) short shortx8;
typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
// Columns beyond the matrix need no mask: what the copy finds there (the next k-row, or zero beyond the end) meets only
// outputs that are not stored.
template <int NB>                                  // 32 NB rows; NB = 2, 4 or 8
struct LoaderKS {
    static_assert(NB == 2 || NB == 4 || NB == 8, "a copy covers whole k-rows");
    static constexpr int ITEM_LDS = 1024, KPI = 16 / NB;      // LDS bytes and k-rows per item
    __amdgpu_buffer_rsrc_t rs;
    rawx4 rsv;
    uint32_t vo[NB], k_step;         // this lane's byte offset for item i, without k0; bytes per k
    int slab0;
    __device__ __forceinline__ uint32_t step_soff(int k0) const { return (uint32_t)k0 * k_step; }
    __device__ __forceinline__ void init(const bf16_t *X, int ld, int row0, int nrows, int K_) {
        rs = make_rsrc(X, ((size_t)(K_ - 1) * ld + nrows) * 2);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const int pos = lane & (4 * NB - 1), kh = lane / (4 * NB);          // 16-byte position in the k-row; which of the item's k-rows
        k_step = (uint32_t)ld * 2u;
        slab0 = __builtin_amdgcn_readfirstlane(w * NB * 1024);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int k = KPI * i + kh, n = (((pos >> 1) ^ (k & 3)) << 4) + (pos & 1) * 8;
            vo[i] = (uint32_t)(((size_t)(w * 16 + k) * ld + row0 + n) * 2);
            asm volatile("" : "+v"(vo[i]));
        }
        rsv = raw_rsrc(X, ((size_t)(K_ - 1) * ld + nrows) * 2);
    }
    // k beyond the matrix reads as zero either way; FAST: as for the K-contiguous loader
    template <bool FAST>
    __device__ __forceinline__ void copy_one(uint8_t *tile, int k0, int i) const {
        lds_void *dst = (lds_void *)(tile + slab0 + i * ITEM_LDS);
        if (FAST) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, (int)vo[i], __builtin_amdgcn_readfirstlane(k0 * (int)k_step), 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, (int)(vo[i] + (uint32_t)k0 * k_step), 0, 0, 0);
    }
    template <bool FAST>
    __device__ __forceinline__ void copy_all(uint8_t *tile, int k0) const {
#pragma unroll
        for (int i = 0; i < NB; ++i) copy_one<FAST>(tile, k0, i);
    }
};

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding
// global store to be acknowledged (its release fence), which would expose the latency of the output
// stores at each barrier; here only LDS operations (lgkmcnt) are waited for.  Direct-to-LDS copies are
// tracked by vmcnt and waited for separately where a stage is handed over.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// Orders this wavefront's own LDS writes before its later LDS reads (other lanes' data, same wavefront).
__device__ __forceinline__ void lds_wave_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Fragment reads issued as assembly.  The compiler makes every LDS read that it cannot prove independent
// of an older direct-to-LDS copy wait for that copy (vmcnt), which it does for the transposing read; written
// as assembly the read carries no such wait.  The price is that the compiler does not know when the data
// arrive: every use is preceded by an explicit s_waitcnt lgkmcnt (wait_frags below), which names the fragment
// registers as operands so that the MFMAs that consume them cannot be moved in front of it.
template <int OFF, int PITCH>                     // PITCH: bytes per k-row
__device__ __forceinline__ bf16x8 lds_read_tr(uint32_t addr) {
    shortx4 lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(OFF));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(OFF + 4 * PITCH));
    const shortx8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return *reinterpret_cast<const bf16x8 *>(&v);
}
template <int OFF>
__device__ __forceinline__ bf16x8 lds_read_b128(uint32_t addr) {
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
// A 32-deep k-slice is worked off in groups of up to four MFMAs: group g multiplies row block g / GPR of A with the
// (g % GPR)-th four (two for a 64-wide tile) blocks of B.  Its RA + RB fragments (16 rows each) are read one slice ahead in
// the order A0 B0 .. A1 .., spread evenly over the groups, and so are the copies of one operand tile.  LDS reads return in
// order, so a group may proceed once at most lgkm_allowed LDS instructions are outstanding: the previous slice's reads
// behind the last fragment the group needs plus this slice's reads issued so far (a group's own reads follow its first
// MFMA).  The counter holds 15 at most.
template <class TS>
struct SliceSched {
    static constexpr int RA = TS::RA, RB = TS::RB;
    static constexpr int GJ = RB < 4 ? RB : 4;                 // MFMAs per group
    static constexpr int GPR = RB / GJ, NG = RA * GPR, NF = RA + RB;
    static constexpr bool is_a(int f) { return f == 0 || f > RB; }
    static constexpr int index(int f) { return f == 0 ? 0 : f <= RB ? f - 1 : f - RB; }
    // items begin(g, n) .. begin(g + 1, n) - 1 of n things to do belong to group g
    static constexpr int begin(int g, int n) { return (g * n + NG - 1) / NG; }
    static constexpr int need(int g) { return g < GPR ? GJ * (g + 1) : RB + g / GPR; }
    template <bool A_KC, bool B_KC>
    static constexpr int lgkm_allowed(int g) {
        const int ca = A_KC ? 1 : 2, cb = B_KC ? 1 : 2;
        int n = 0;
        for (int f = need(g) + 1; f < NF; ++f) n += is_a(f) ? ca : cb;
        for (int f = 0; f < begin(g, NF); ++f) n += is_a(f) ? ca : cb;
        return n < 15 ? n : 15;
    }
};
template <int N>
__device__ __forceinline__ void wait_frags(bf16x8 &a, bf16x8 &b, bf16x8 &c, bf16x8 &d, bf16x8 &e) {
    asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(e) : "n"(N));
}
template <int N>
__device__ __forceinline__ void wait_frags(bf16x8 &a, bf16x8 &b, bf16x8 &c, bf16x8 &d) {
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N));
}
template <int N>
__device__ __forceinline__ void wait_frags(bf16x8 &a, bf16x8 &b, bf16x8 &c) {
    asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(a), "+v"(b), "+v"(c) : "n"(N));
}
template <int N>
__device__ __forceinline__ void wait_frags(bf16x8 &a) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(a) : "n"(N));
}
template <int... I, class F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}

// One MFMA with the copy of one item of an operand tile behind it, as one statement: M0 (the LDS destination) is written in
// front of the MFMA, which also is the wait state the copy needs after that write, and the copy's scalar offset is the same for
// all items of a step (the builtin form costs a scalar add for the offset, one for M0 and a no-op per copy).
template <int MOFF>
__device__ __forceinline__ void mfma_copy(f32x4 &acc, const bf16x8 &b, const bf16x8 &a, uint32_t mbase, uint32_t vo, const rawx4 &rsv,
                                          uint32_t so) {
    asm volatile("s_add_u32 m0, %[mb], %[moff]\n\tv_mfma_f32_16x16x32_bf16 %[acc], %[b], %[a], %[acc]\n\t"
                 "buffer_load_dwordx4 %[vo], %[rs], %[so] offen lds"
                 : [acc] "+a"(acc) : [b] "v"(b), [a] "v"(a), [mb] "s"(mbase), [moff] "n"(MOFF), [vo] "v"(vo), [rs] "s"(rsv), [so] "s"(so)
                 : "memory", "m0", "scc");
}

// fp32 epilogue: unit u (16 bytes) of staged row r, 64 RB bytes long, is kept at unit u ^ staged_turn(r).  A write covers 16 rows at one unit.  Rows 0-7
// fall into distinct slots modulo 256 bytes, and so do rows 8-15; of a 64-wide tile (RB = 2, rows of 128 bytes) rows r and r + 8 share one.  The form that
// separates all 16 there, (r >> 1) & 7, gains nothing: 1024 x 1024, 2880 tokens 13.5 -> 13.6 us, added to contents 14.1 -> 14.2.
template <int RB>
constexpr int staged_turn(int r) { return RB == 2 ? ((r >> 2) & 1) | ((r & 3) << 1) : r & 15; }
template <int RB>
constexpr bool staged_rows_distinct(int first, int rows) {
    uint32_t seen = 0;
    for (int r = first; r < first + rows; ++r) seen |= 1u << ((r * 4 * RB + staged_turn<RB>(r)) & 15);
    return __builtin_popcount(seen) == rows;
}
static_assert(staged_rows_distinct<2>(0, 8) && staged_rows_distinct<2>(8, 8) && staged_rows_distinct<4>(0, 16) && staged_rows_distinct<8>(0, 16),
              "what a staging write covers");

template <bool KC, int NB> struct LoaderSel { typedef LoaderKC<NB> type; };
template <int NB> struct LoaderSel<false, NB> { typedef LoaderKS<NB> type; };

template <bool A_KC, bool B_KC, bool HAS_ADD, bool OUT_F32, class TS = Tile256, typename ARG = GemmP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TS::PER_CU, TS::PER_CU)))
void gemm_mfma_kernel(const ARG arg) {
    constexpr int RA = TS::RA, RB = TS::RB, AHEAD = TS::AHEAD, BM = TS::BM, BN = TS::BN;
    constexpr int A_PITCH = 2 * BM, B_PITCH = 2 * BN;             // bytes per k-row of a K-strided tile
    typedef SliceSched<TS> Sched;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const unsigned long long *const probe_ = first_problem(arg).clock_probe;
    unsigned long long *const clock_probe = const_cast<unsigned long long *>(probe_);

    if constexpr (std::is_same<ARG, GemmGroup>::value) {
        const int workgroups = arg.workgroups;
        if ((int)blockIdx.x >= workgroups) {
            typedef typename std::conditional<OUT_F32, float, bf16_t>::type T;
            for (int unit = blockIdx.x - workgroups; unit < arg.reduce.units[8]; unit += gridDim.x - workgroups) {
                reduce_unit<T>(arg.reduce, unit, reinterpret_cast<float (*)[36]>(smem), threadIdx.x);
                __syncthreads();
            }
            return;
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    if (clock_probe && blockIdx.x == 0 && threadIdx.x == 0) {
        clock_probe[0] = (unsigned long long)clock64();
        clock_probe[1] = (unsigned long long)wall_clock64();
    }

    // ---- persistent workgroup -> tiles.  Workgroup b runs on XCD b % 8 (round-robin dispatch); XCD x
    // owns a contiguous run of the tile order, and its workgroups stride through that run together.
    const int ntiles = work_items(arg, OUT_F32);                  // work items: (K chunk, tile), chunk-major
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int per = ntiles >> 3, rem = ntiles & 7;
    const int run_begin = xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per;
    const int run_end = run_begin + per + (xcd < rem ? 1 : 0);
    const int wg_per_xcd = (gemm_workgroups(arg) - xcd + 7) >> 3;

    // fragment addressing (v_mfma_f32_16x16x32_bf16: lane l holds row l & 15, k = 8 (l >> 4) .. + 7 of a
    // 16-row, 32-deep fragment).  K-contiguous tile: row block i, slice s -> row 16 i + (l & 15), unit
    // 4 s + (l >> 4); the swizzle of that row is that of row l & 15, so two offsets per operand (one per slice)
    // cover all blocks, the block itself being an immediate offset of the read.  K-strided tile: the 16 lanes with
    // the same l >> 4 form rows 0..15 of the block at k = 8 (l >> 4) ..; lane j of them supplies the address
    // of k-row (j >> 2), rows 4 (j & 3) .. + 3, for each of the two transposing reads.
    const int frow = lane & 15, fq = lane >> 4;
    constexpr int AC = RA < 4 ? RA : 4, BC = RB < 4 ? RB : 4;
    int a_rd[AC][2], b_rd[BC][2];
#pragma unroll
    for (int c = 0; c < AC; ++c)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            if (A_KC) a_rd[c][sl] = (wm * 16 * RA + frow) * 128 + (((sl * 4 + fq) ^ swz(frow)) << 4);
            else a_rd[c][sl] = (sl * 32 + 8 * fq + (frow >> 2)) * A_PITCH + (frow & 3) * 8 + ((wm * RA + c) ^ (frow >> 2)) * 32;
        }
#pragma unroll
    for (int c = 0; c < BC; ++c)
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            if (B_KC) b_rd[c][sl] = (wn * 16 * RB + frow) * 128 + (((sl * 4 + fq) ^ swz(frow)) << 4);
            else b_rd[c][sl] = (sl * 32 + 8 * fq + (frow >> 2)) * B_PITCH + (frow & 3) * 8 + ((wn * RB + c) ^ (frow >> 2)) * 32;
        }

    if constexpr (OUT_F32)                                        // (see late_start)
        if (q & 1)
            for (int i = 0; i < first_problem(arg).late_start; ++i) __builtin_amdgcn_s_sleep(8);

    for (int logical = run_begin + q; logical < run_end; logical += wg_per_xcd) {
    int tm, tn, item;
    const GemmP p = pick(arg, logical, item);                  // (a group: the problem this work item belongs to)
    const int chunk = OUT_F32 ? item / p.tile_count : 0;
    const int tl = item - chunk * p.tile_count;                // tile within this launch
    tile_coords(p.tile_begin + tl, p.tiles_m, p.tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    // this work item's K range (only the fp32-output kernels are ever split)
    const int k_begin = OUT_F32 ? chunk * p.k_chunk : 0;
    const int Kc = OUT_F32 ? min(p.k_chunk, p.K - k_begin) : p.K;

    typename LoaderSel<A_KC, RA>::type la;
    typename LoaderSel<B_KC, RB>::type lb;
    la.init(p.A + (size_t)k_begin * (A_KC ? 1 : p.lda), p.lda, m0, p.M, Kc);
    lb.init(p.B + (size_t)k_begin * (B_KC ? 1 : p.ldb), p.ldb, n0, p.N, Kc);

    f32x4 acc[RA][RB];
    // cleared (4 cycles a register, 1 k for a 256 x 256 tile) while the tile's first copies are on their way
    auto clear = [&]() {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                asm volatile("" : "+a"(acc[i][j]));
            }
        __builtin_amdgcn_sched_barrier(0);
    };

    bf16x8 fa[2][RA], fb[2][RB];
    // Kernels with a K-strided operand read all their fragments as assembly (see lds_read_tr) and wait for
    // them explicitly; the all-K-contiguous kernel leaves reads and waits to the compiler.
    constexpr bool ASM_READS = !(A_KC && B_KC);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void *)smem;
    // fragment f of slice SL (0, 1) of the tiles at LDS offsets ta, tb, into fragment buffer buf
    auto read_frag = [&](auto SL, auto F, int ta, int tb, int buf) {
        constexpr int sl = decltype(SL)::value, f = decltype(F)::value;
        constexpr bool is_a = Sched::is_a(f);
        constexpr int i = Sched::index(f);
        // K-contiguous: all blocks share the swizzle term; K-strided: one offset per block modulo 4, the rest an immediate
        constexpr int kc_imm = i * 16 * 128, ks_imm = (i >> 2) * 4 * 32, c = i & 3;
        if constexpr (is_a) {
            if (A_KC) {
                if (!ASM_READS) fa[buf][i] = *reinterpret_cast<const bf16x8 *>(smem + ta + a_rd[c][sl] + kc_imm);
                else fa[buf][i] = lds_read_b128<kc_imm>(lds0 + ta + a_rd[c][sl]);
            } else fa[buf][i] = lds_read_tr<ks_imm, A_PITCH>(lds0 + ta + a_rd[c][sl]);
        } else {
            if (B_KC) {
                if (!ASM_READS) fb[buf][i] = *reinterpret_cast<const bf16x8 *>(smem + tb + b_rd[c][sl] + kc_imm);
                else fb[buf][i] = lds_read_b128<kc_imm>(lds0 + tb + b_rd[c][sl]);
            } else fb[buf][i] = lds_read_tr<ks_imm, B_PITCH>(lds0 + tb + b_rd[c][sl]);
        }
    };
    // before MFMA group g of a slice held in fragment buffer `buf`
    auto wait_group = [&](auto G, int buf) {
        constexpr int g = decltype(G)::value;
        constexpr int n = Sched::template lgkm_allowed<A_KC, B_KC>(g);
        if constexpr (!ASM_READS) return;
        else if constexpr (g == 0 && Sched::GJ == 4) wait_frags<n>(fa[buf][0], fb[buf][0], fb[buf][1], fb[buf][2], fb[buf][3]);
        else if constexpr (g == 0) wait_frags<n>(fa[buf][0], fb[buf][0], fb[buf][1]);
        else if constexpr (g < Sched::GPR) wait_frags<n>(fb[buf][4 * g], fb[buf][4 * g + 1], fb[buf][4 * g + 2], fb[buf][4 * g + 3]);
        else if constexpr (g % Sched::GPR == 0) wait_frags<n>(fa[buf][g / Sched::GPR]);
    };
    // MFMA t of group g of a k-slice: row block g / GPR of A against block GJ (g % GPR) + t of B.
    // Operands are swapped: the accumulator tile is held transposed (lane = m, registers run over n),
    // so that each lane owns 4 consecutive n of one row for the epilogue.  The instruction is written out
    // with the accumulator tied to itself in the accumulation registers: left to the register allocator,
    // the accumulators are shuffled between registers in every iteration.  An accumulator is touched
    // again only RA * RB MFMAs (4 at least) later, and the code after the K loop starts with waits
    // and a barrier, so none of the software-managed MFMA hazards can occur.
    auto mfma = [&](int buf, int g, int t) {
        const int i = g / Sched::GPR, j = Sched::GJ * (g % Sched::GPR);
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[i][j + t]) : "v"(fb[buf][j + t]), "v"(fa[buf][i]));
    };

    // Software pipeline, one barrier per 64-deep K step.  A tiles go round a ring of AHEAD + 1 LDS slots, B tiles round one of
    // AHEAD.  Step kt multiplies K tile kt in two 32-deep k-slices; every group of a slice also reads its share of the
    // fragments of the following slice, so after the first slice every wavefront has read all of A(kt) and B(kt): past the
    // barrier in the middle of the step B(kt)'s slot is handed to B(kt + AHEAD) and A(kt)'s to A(kt + 1 + AHEAD), and the
    // second slice's groups read the first slice of tile kt + 1.  A wavefront issues its copies of A(kt + AHEAD) in the first
    // slice and those of B(kt + AHEAD) in the second, spread over the groups: the compute unit's address path takes about 20
    // cycles per 1 KiB copy, and four wavefronts issuing one in every group of four MFMAs would back it up and stall the MFMAs
    // behind it.  At the barrier of step kt the tiles A(kt+1) and B(kt+1) must have landed; the copies younger than B(kt+1)
    // may still be in flight (memory operations retire in issue order).
    const int nk = (Kc + BK - 1) / BK, nk_whole = Kc / BK;       // K tiles; those without a remainder
    // Where every workgroup has one tile, the XCDs walk over the whole K tiles in a circle, each from an eighth further on.  They share
    // operand panels but no L2: in step, up to eight of them ask for a line that is still on its way from HBM, and each waits for it; out
    // of step one fetches it and the others find it in the memory-side cache.  (The workgroups of one XCD stay in step: apart, they lose
    // what L2 shares, 125 us and 199 us for the copies of 8192 x 4096 x 4096.)  From HBM, us: 1031 x 4096 x 11008 122 -> 98, 1031 x 4096 x
    // 4096 45 -> 39, 2304 x 1024 x 4096 NN 38.8 -> 35.8, 4111 x 1280 x 5120 61.7 -> 59.9; 120 products of random sizes: 2 % less in 64 x 64
    // tiles, 6 % in 64 x 128 and 128 x 128.  Operands in that cache: the same, but 1 % more (0.2 us) in 64 x 64 tiles (46 x 2048 x 5120 NN 17.5 ->
    // 17.8); whole layers' weights come from HBM.  An element's sum then depends in its order on the tile that it lies in.  Launches of
    // several rounds are out of step as they are (8192 x 4096 x 22016 lost 1 %), and below 32 K tiles everything is requested almost at
    // once in any order: 4111 x 3840 x 1280 35.2 -> 36.3, 1031 x 4096 x 1024 the same, x 2048 25.4 -> 21.7.  Nor do weight gradients, which read
    // longer pieces of their operands' rows: 4096 x 1024 x 2048 20.6 -> 20.9 from the cache, 24.1 -> 23.9 from HBM.
    const int k_start = A_KC && nk_whole >= 32 && run_end - run_begin <= wg_per_xcd ? xcd * nk_whole / 8 : 0;     // the first K tile
    typedef std::integral_constant<int, 0> S0;
    typedef std::integral_constant<int, 1> S1;
    typedef std::make_integer_sequence<int, Sched::NG> Groups;
    typedef std::make_integer_sequence<int, Sched::NF> Frags;
    constexpr int B0 = (AHEAD + 1) * TS::A_BYTES;                  // LDS offset of the first B slot
    if (nk_whole >= AHEAD) {
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            const int k = (k_start + j >= nk_whole ? k_start + j - nk_whole : k_start + j) * BK;
            la.template copy_all<true>(smem + j * TS::A_BYTES, k);
            lb.template copy_all<true>(smem + B0 + j * TS::B_BYTES, k);
        }
        clear();
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * (RA + RB)) : "memory");     // A0 and B0 have landed
    } else {                                                   // a short K: only the tiles it has, all of them waited for
        const int n = min(nk, AHEAD);
#pragma unroll 1
        for (int j = 0; j < n; ++j) {
            la.template copy_all<false>(smem + j * TS::A_BYTES, j * BK);
            lb.template copy_all<false>(smem + B0 + j * TS::B_BYTES, j * BK);
        }
        clear();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    lds_barrier();
    static_for(Frags{}, [&](auto F) { read_frag(S0{}, F, 0, B0, 0); });

    // LDS offsets of the slots of A(kt), A(kt+1), A(kt+AHEAD) and of B(kt), which is B(kt+AHEAD)'s as well, and B(kt+1)
    int oa = 0, oa1 = TS::A_BYTES, oad = AHEAD * TS::A_BYTES, ob = B0, ob1 = B0 + (AHEAD > 1 ? TS::B_BYTES : 0);
    // scalar offsets of what the next step requests (of whole tiles)
    uint32_t so_a = la.step_soff((k_start + AHEAD) * BK), so_b = lb.step_soff((k_start + AHEAD) * BK);
    // COPY: 2 = tile kt + AHEAD is whole (fast copies), 1 = it reaches beyond K, 0 = there is no such tile
    auto step = [&](auto COPY_, int kt) {
        constexpr int COPY = decltype(COPY_)::value;
        const int k2 = (kt + AHEAD) * BK;                      // (where the tile reaches beyond K)
        typedef std::remove_reference_t<decltype(la)> LA;
        typedef std::remove_reference_t<decltype(lb)> LB;
        // fast path: LDS destinations of this step's copies
        const uint32_t mb_a = __builtin_amdgcn_readfirstlane(lds0 + oad + la.slab0), mb_b = __builtin_amdgcn_readfirstlane(lds0 + ob + lb.slab0);
        // first slice: fragments of the second slice; A(kt+AHEAD) into the slot A(kt-1) had
        static_for(Groups{}, [&](auto G) {
            constexpr int g = decltype(G)::value, i = g / Sched::GPR, j = Sched::GJ * (g % Sched::GPR);
            constexpr int f0 = Sched::begin(g, Sched::NF), f1 = Sched::begin(g + 1, Sched::NF);
            constexpr int c0 = Sched::begin(g, RA), c1 = Sched::begin(g + 1, RA);
            wait_group(G, 0);
            mfma(0, g, 0);
            __builtin_amdgcn_sched_barrier(0);
            static_for(std::make_integer_sequence<int, f1 - f0>{}, [&](auto F) { read_frag(S1{}, std::integral_constant<int, f0 + decltype(F)::value>{}, oa, ob, 1); });
            __builtin_amdgcn_sched_barrier(0);
            static_for(std::make_integer_sequence<int, Sched::GJ - 1>{}, [&](auto U) {
                constexpr int t = decltype(U)::value + 1, c = c0 + t - 1;
                if constexpr (COPY == 2 && c < c1) mfma_copy<c * LA::ITEM_LDS>(acc[i][j + t], fb[0][j + t], fa[0][i], mb_a, la.vo[c], la.rsv, so_a);
                else mfma(0, g, t);
                if constexpr (t <= 2) __builtin_amdgcn_sched_barrier(0);
                if constexpr (COPY == 1 && c < c1) { la.template copy_one<false>(smem + oad, k2, c); __builtin_amdgcn_sched_barrier(0); }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        // A(kt+1) and B(kt+1) have landed
        if constexpr (COPY != 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 2) * (RA + RB) + RA) : "memory");
        else if (AHEAD > 3 && nk - kt > 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD > 3 ? 2 * (RA + RB) : 0) : "memory");
        else if (AHEAD > 2 && nk - kt > 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD > 2 ? RA + RB : 0) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();                                         // and nobody reads A(kt), B(kt) any more
        // second slice: fragments of the first slice of tile kt+1; B(kt+AHEAD) into the slot B(kt) had.
        // The barrier has waited for every LDS read, so this slice's MFMAs need no wait of their own.
        if constexpr (ASM_READS) {         // ties the MFMAs below to this side of the barrier
#pragma unroll
            for (int i = 0; i < RA; ++i) asm volatile("" : "+v"(fa[1][i]));
#pragma unroll
            for (int j = 0; j < RB; ++j) asm volatile("" : "+v"(fb[1][j]));
        }
        static_for(Groups{}, [&](auto G) {
            constexpr int g = decltype(G)::value, i = g / Sched::GPR, j = Sched::GJ * (g % Sched::GPR);
            constexpr int f0 = Sched::begin(g, Sched::NF), f1 = Sched::begin(g + 1, Sched::NF);
            constexpr int c0 = Sched::begin(g, RB), c1 = Sched::begin(g + 1, RB);
            mfma(1, g, 0);
            __builtin_amdgcn_sched_barrier(0);
            static_for(std::make_integer_sequence<int, f1 - f0>{}, [&](auto F) { read_frag(S0{}, std::integral_constant<int, f0 + decltype(F)::value>{}, oa1, ob1, 0); });
            __builtin_amdgcn_sched_barrier(0);
            static_for(std::make_integer_sequence<int, Sched::GJ - 1>{}, [&](auto U) {
                constexpr int t = decltype(U)::value + 1, c = c0 + t - 1;
                if constexpr (COPY == 2 && c < c1) mfma_copy<c * LB::ITEM_LDS>(acc[i][j + t], fb[1][j + t], fa[1][i], mb_b, lb.vo[c], lb.rsv, so_b);
                else mfma(1, g, t);
                if constexpr (t <= 2) __builtin_amdgcn_sched_barrier(0);
                if constexpr (COPY == 1 && c < c1) { lb.template copy_one<false>(smem + ob, k2, c); __builtin_amdgcn_sched_barrier(0); }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        const int last = oa;
        oa = oa1;
        oa1 = AHEAD == 2 ? oad : oa1 + TS::A_BYTES == B0 ? 0 : oa1 + TS::A_BYTES;
        oad = last;
        const int lastb = ob;
        ob = ob1;
        ob1 = AHEAD == 2 ? lastb : ob1 + TS::B_BYTES == TS::RING_BYTES ? B0 : ob1 + TS::B_BYTES;
    };
    const int nk_fast = max(nk_whole - AHEAD, 0), nk_copy = max(nk - AHEAD, 0);
    int kt = 0;
    for (int lap = nk_fast - k_start;;) {                        // the requests pass the end of K at step `lap` and go on from its start
        if (kt >= lap) { lap = nk_fast; so_a -= la.step_soff(nk_whole * BK); so_b -= lb.step_soff(nk_whole * BK); }
#pragma unroll 1
        for (; kt < lap; ++kt) {
            step(std::integral_constant<int, 2>{}, kt);
            so_a += la.step_soff(BK);
            so_b += lb.step_soff(BK);
        }
        if (kt >= nk_fast) break;
    }
    for (; kt < nk_copy; ++kt) step(std::integral_constant<int, 1>{}, kt);
    for (; kt < nk; ++kt) step(std::integral_constant<int, 0>{}, kt);
    asm volatile("s_nop 15\n\ts_waitcnt vmcnt(0)" ::: "memory");   // the last MFMAs have written their accumulators, and no copy is
                                                                  // outstanding
    if constexpr (ASM_READS) {
        // the last slice's reads (never used) still target these registers: keep them reserved until they land
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < RA; ++i) asm volatile("" : "+v"(fa[0][i]));
#pragma unroll
        for (int j = 0; j < RB; ++j) asm volatile("" : "+v"(fb[0][j]));
    }
    lds_barrier();

    if constexpr (OUT_F32) {
        // ---- fp32 epilogue (never together with bias or residual): one row block of 16 rows at a time through this wavefront's own
        // staging area, so that loads and stores cover whole rows of 64 RB bytes and whole cache lines (64-byte pieces straight from the
        // accumulators leave the L2 half filled: 29 % more bytes written).  A wavefront's LDS instructions execute in order, so neither the
        // read-back of a block nor the writes of the next one into the same place wait for what stands in front of them; the compiler is
        // only kept from reordering them.  The previous contents are fetched a row block ahead of their use, in front of the stores in
        // between: memory operations retire in order, and a load behind a store returns only when that store has been acknowledged.  Every
        // row block has a descriptor of its own, so that 32-bit offsets reach rows of up to 2^26 elements; lanes outside the matrix carry
        // an offset that the descriptor's bounds check turns into nothing, without a branch.  22016 x 4096, 1031 tokens added to fp32
        // gradients: 308 -> 257 us, 300 tokens 223 -> 172 (in 32-row chunks whose loads stood behind stores).
        const uint32_t pitch = p.compact ? 256u : (uint32_t)p.ldc;
        const int wm0 = __builtin_amdgcn_readfirstlane(wm) * 16 * RA;         // first row of this wavefront
        float *const out = reinterpret_cast<float *>(p.C) + (size_t)wm0 * pitch +
                           (p.compact ? (size_t)(chunk * p.tile_count + tl) << 16 : (size_t)chunk * p.M * p.ldc + (size_t)m0 * p.ldc + n0);
        constexpr int UNITS = 4 * RB, RPP = 64 / UNITS, PASSES = 16 / RPP, DEPTH = 2;       // 16-byte units per row, rows per pass
        const int er = lane / UNITS, eu = lane % UNITS;
        const int col0 = wn * 16 * RB + eu * 4, rows = p.M - m0 - wm0;
        const uint32_t col_bytes = n0 + col0 < p.N ? (uint32_t)col0 * 4u : OOB;
        uint8_t *stg = smem + wave * (16 * 16 * RB * 4);
        constexpr auto turn = staged_turn<RB>;
        rawx4 prev[DEPTH][PASSES];
        auto block = [&](int i) { return make_rsrc(out + (size_t)(16 * i) * pitch, OOB); };
        auto offset = [&](int i, int pass) {
            const int r = RPP * pass + er;
            return (int)(16 * i + r < rows && col_bytes != OOB ? (uint32_t)r * pitch * 4u + col_bytes : OOB);
        };
        auto fetch = [&](auto I_) {
            constexpr int i = decltype(I_)::value;
#pragma unroll
            for (int pass = 0; pass < PASSES; ++pass) prev[i % DEPTH][pass] = __builtin_amdgcn_raw_buffer_load_b128(block(i), offset(i, pass), 0, 0);
        };
        auto finish = [&](auto ADD_) {
            constexpr bool ADD = decltype(ADD_)::value;
            if constexpr (ADD) fetch(std::integral_constant<int, 0>{});
            static_for(std::make_integer_sequence<int, RA>{}, [&](auto I_) {
                constexpr int i = decltype(I_)::value;
                asm volatile("" ::: "memory");
#pragma unroll
                for (int j = 0; j < RB; ++j)
                    *reinterpret_cast<f32x4 *>(stg + frow * (RB * 64) + (((j * 4 + fq) ^ turn(frow)) << 4)) = acc[i][j];
                if constexpr (ADD && i + 1 < RA) fetch(std::integral_constant<int, i + 1>{});
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                f32x4 v[PASSES];
#pragma unroll
                for (int pass = 0; pass < PASSES; ++pass) {
                    const int r = RPP * pass + er;
                    v[pass] = *reinterpret_cast<const f32x4 *>(stg + r * (RB * 64) + ((eu ^ turn(r)) << 4));
                }
#pragma unroll
                for (int pass = 0; pass < PASSES; ++pass) {
                    if constexpr (ADD) v[pass] += *reinterpret_cast<const f32x4 *>(&prev[i % DEPTH][pass]);
                    __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const rawx4 *>(&v[pass]), block(i), offset(i, pass), 0, STREAMING);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        if (p.accumulate) finish(std::true_type{});
        else finish(std::false_type{});
        lds_barrier();
        continue;
    }
    // ---- epilogue: 32 rows x 16 RB columns at a time through this wavefront's own staging area; the output
    // stores are left in flight (nothing below waits for them) and drain under the next tile's K loop
    constexpr int EPI_PITCH = TS::EPI_PITCH, LPR = 2 * RB, RPP = 64 / LPR;      // lanes per row, rows per pass of the read-back
    constexpr int CHUNKS = (RA + 1) / 2, PASSES = 32 / RPP;
    float *stg = reinterpret_cast<float *>(smem) + wave * (32 * EPI_PITCH);
    const int er = lane / LPR, ec = (lane % LPR) * 8;      // read-back: row er + RPP*pass, columns ec..ec+7
    const int gn = n0 + wn * 16 * RB + ec;
    const bool nok = gn < p.N;
    float bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (p.bias && nok) {
        const uint4 raw = *reinterpret_cast<const uint4 *>(p.bias + gn);
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) { bv[2 * e] = __uint_as_float(w[e] << 16); bv[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u); }
    }
    // Everything that is added to the product (residual, previous C) is fetched before the first output
    // store is issued: memory operations retire in order, so a load issued after a store would have to
    // wait for that store to be acknowledged.
    const bf16_t *addend = p.residual ? p.residual : p.C;      // HAS_ADD: residual and / or accumulate
    uint4 add[HAS_ADD ? CHUNKS : 1][PASSES];
    if (HAS_ADD) {
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i)
#pragma unroll
            for (int pass = 0; pass < PASSES; ++pass) {
                if (i * 32 + pass * RPP >= 16 * RA) continue;
                const int gm = m0 + wm * 16 * RA + i * 32 + pass * RPP + er;
                add[i][pass] = make_uint4(0, 0, 0, 0);
                if (gm < p.M && nok) add[i][pass] = *reinterpret_cast<const uint4 *>(addend + (size_t)gm * p.ldc + gn);
            }
    }
    const bool both = HAS_ADD && p.residual && p.accumulate;   // rare: the second addend is read in the store loop
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        // accumulator tile (2 i + ii, j), register e  <->  m = 16 (2 i + ii) + (lane & 15),  n = 16 j + 4 (lane >> 4) + e
#pragma unroll
        for (int ii = 0; ii < 2 && 2 * i + ii < RA; ++ii)
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                const f32x4 t = acc[2 * i + ii][j];
                *reinterpret_cast<float4 *>(stg + (ii * 16 + frow) * EPI_PITCH + j * 16 + fq * 4) = make_float4(t[0], t[1], t[2], t[3]);
            }
        lds_wave_sync();
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            if (i * 32 + pass * RPP >= 16 * RA) continue;          // (an odd number of row blocks: the last chunk is half)
            const int r = pass * RPP + er;
            const int gm = m0 + wm * 16 * RA + i * 32 + r;
            if (gm < p.M && nok) {
                const float4 v0 = *reinterpret_cast<const float4 *>(stg + r * EPI_PITCH + ec);
                const float4 v1 = *reinterpret_cast<const float4 *>(stg + r * EPI_PITCH + ec + 4);
                float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
                if (p.bias) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] += bv[e];
                }
                const size_t off = (size_t)gm * p.ldc + gn;
                if (HAS_ADD) {
                    const uint32_t w[4] = {add[i][pass].x, add[i][pass].y, add[i][pass].z, add[i][pass].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) { v[2 * e] += __uint_as_float(w[e] << 16); v[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u); }
                }
                if (both) {
                    const uint4 raw = *reinterpret_cast<const uint4 *>(p.C + off);
                    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) { v[2 * e] += __uint_as_float(w[e] << 16); v[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u); }
                }
                uint4 o;
                o.x = pack_bf16x2(v[0], v[1]); o.y = pack_bf16x2(v[2], v[3]);
                o.z = pack_bf16x2(v[4], v[5]); o.w = pack_bf16x2(v[6], v[7]);
                // streaming store: the output is not read again by this kernel, so it should not displace
                // operand panels from the L2
                __builtin_nontemporal_store(*reinterpret_cast<const rawx4 *>(&o), reinterpret_cast<rawx4 *>(p.C + off));
            }
        }
        lds_wave_sync();
    }
    lds_barrier();      // staging area is free again: the next tile's first stage may overwrite it
    }   // tiles of this workgroup
    if (clock_probe && blockIdx.x == 0 && threadIdx.x == 0) {
        clock_probe[2] = (unsigned long long)clock64();
        clock_probe[3] = (unsigned long long)wall_clock64();
    }
}

// Sums added to fp32 contents move 8 bytes per element: all compute units multiplying at once and then all at memory at once leave each
// idle half of the time.  Where every workgroup has two tiles and more, every second one starts later, by half a tile's time but no more
// than its memory phase takes.  The longer the K loop beside that phase, the less there is to hide and the more the workgroups drift out of
// step by themselves.  Without -> with it, us, mean of two boxes: K = 1031: 8192 x 4096 (two rounds of 256 x 256 tiles) 125 -> 107, 12288 x 4096
// (three) 147 -> 133, 28672 x 4096 (seven) 316 -> 294; K = 2048 160 -> 143, 203 -> 191, 451 -> 441; K = 4096 234 -> 223, 336 -> 330, 766 -> 763 and
// 8192 x 12288 (six) 649 -> 648; but K = 6144 315 -> 312, 467 -> 472, 1104 -> 1100, 916 -> 922 and K = 8192 401 -> 404, 612 -> 616, 1432 -> 1433, 1179 -> 1196.
// In 256 x 128 tiles, 6144 x 4096 (three): K = 1031 85 -> 81, 2048 119.7 -> 120.6, 4096 199 -> 200.  Every second workgroup, whichever have a tile more
// than the others: to spare those gains where they are two of 32 (8448 x 4096 127 -> 116) and loses where they are 28 (11776 x 4096 132 -> 140).
template <class TS>
int late_start(int accumulate, int K, int items, int workgroups) {
    constexpr int BLOCKS = TS::RA * TS::RB;
    if (!accumulate || items / workgroups < 2 || K > (BLOCKS == 64 ? 4096 : 1536)) return 0;
    const int clocks = (K + BK - 1) / BK * 1200 + 10000;
    return (clocks < 30000 ? clocks : 30000) * BLOCKS / 64 / 512;
}

// compute units of the current device, rounded down to whole XCD octets (one persistent workgroup each)
inline hipError_t compute_units(int &n) {
    static std::atomic<int> cached{0};
    int n_cu = cached.load(std::memory_order_relaxed);
    if (n_cu == 0) {
        int dev = 0, v = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        if (v <= 0) v = 256;
        v &= ~7;
        n_cu = v ? v : 8;
        cached.store(n_cu, std::memory_order_relaxed);
    }
    n = n_cu;
    return hipSuccess;
}

// Dynamic LDS of `kern` raised to `bytes` (beyond 64 KiB a kernel has to ask for it), once per kernel.
inline hipError_t allow_lds(std::atomic<bool> &configured, const void *kern, int bytes) {
    if (configured.load(std::memory_order_acquire)) return hipSuccess;    // concurrent first calls repeat the same idempotent set-up
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) configured.store(true, std::memory_order_release);
    return e;
}

template <bool A_KC, bool B_KC, bool HAS_ADD, bool OUT_F32, class TS>
hipError_t launch(GemmP p, hipStream_t st) {
    static std::atomic<bool> configured{false};
    auto kern = gemm_mfma_kernel<A_KC, B_KC, HAS_ADD, OUT_F32, TS>;
    hipError_t e = allow_lds(configured, reinterpret_cast<const void *>(kern), TS::SMEM);
    if (e != hipSuccess) return e;
    // persistent workgroups, as many as the device holds at once
    int n_cu = 0;
    e = compute_units(n_cu);
    if (e != hipSuccess) return e;
    const int items = p.tile_count * (OUT_F32 ? p.splits : 1), room = n_cu * TS::PER_CU;
    if (items <= 0) return hipSuccess;
    const int workgroups = items < room ? items : room;
    p.late_start = OUT_F32 ? late_start<TS>(p.accumulate, p.K, items, workgroups) : 0;
    kern<<<workgroups, 256, TS::SMEM, st>>>(p);
    return hipGetLastError();
}

// Tile shapes smaller than 256 x 256 (choose_tile in gemm_mfma.hip).  AHEAD is as deep as LDS allows with the number of
// workgroups per compute unit that hides a small tile's barrier waits: a 64 x 64 step is 128 cycles of MFMA against several
// hundred of memory latency.  Those of 224, 192, 160 and 96 rows need a K-contiguous A.
typedef TileShape<7, 8, 2> Tile224;
typedef TileShape<6, 8, 2> Tile192;
typedef TileShape<5, 8, 2> Tile160;
typedef TileShape<8, 4, 2> Tile256x128;
typedef TileShape<6, 4, 3> Tile192x128;
typedef TileShape<5, 4, 3> Tile160x128;
typedef TileShape<4, 4, 4> Tile128;
typedef TileShape<3, 4, 4> Tile96x128;
typedef TileShape<2, 4, 3> Tile64x128;
typedef TileShape<2, 2, 4> Tile64;
enum { TILE_256, TILE_224, TILE_192, TILE_160, TILE_256x128, TILE_192x128, TILE_160x128, TILE_128, TILE_96x128, TILE_64x128, TILE_64, N_TILE_SHAPES };

// the launch of a forward or input-gradient product in tiles of shape TS
template <bool A_KC, bool B_KC, class TS>
hipError_t launch_tile(GemmP p, hipStream_t st) {
    p.tiles_m = ceil_div(p.M, TS::BM); p.tiles_n = ceil_div(p.N, TS::BN);
    p.tile_count = p.tiles_m * p.tiles_n;
    return p.residual || p.accumulate ? launch<A_KC, B_KC, true, false, TS>(p, st) : launch<A_KC, B_KC, false, false, TS>(p, st);
}
template <bool A_KC, bool B_KC>
hipError_t launch_tile_shape(int shape, const GemmP &p, hipStream_t st) {
    switch (shape) {
        case TILE_224: return launch_tile<A_KC, B_KC, Tile224>(p, st);
        case TILE_192: return launch_tile<A_KC, B_KC, Tile192>(p, st);
        case TILE_160: return launch_tile<A_KC, B_KC, Tile160>(p, st);
        case TILE_256x128: return launch_tile<A_KC, B_KC, Tile256x128>(p, st);
        case TILE_192x128: return launch_tile<A_KC, B_KC, Tile192x128>(p, st);
        case TILE_160x128: return launch_tile<A_KC, B_KC, Tile160x128>(p, st);
        case TILE_128: return launch_tile<A_KC, B_KC, Tile128>(p, st);
        case TILE_96x128: return launch_tile<A_KC, B_KC, Tile96x128>(p, st);
        case TILE_64x128: return launch_tile<A_KC, B_KC, Tile64x128>(p, st);
        case TILE_64: return launch_tile<A_KC, B_KC, Tile64>(p, st);
        default: return hipErrorInvalidValue;
    }
}
// gemm_mfma_nt.hip / gemm_mfma_nn.hip: one product in one of the smaller shapes
hipError_t launch_nt(int shape, const GemmP &p, hipStream_t st);
hipError_t launch_nn(int shape, const GemmP &p, hipStream_t st);
// gemm_mfma_tn.hip: up to MAX_GROUP weight gradients in one launch, all in the same tile shape (a single one: n = 1)
// reduce: when not null, sums to be added up by the same launch
hipError_t launch_tn(int shape, const GemmP *p, int n, const ReduceJobSet *reduce, hipStream_t st);

}  // namespace gemm_detail
}  // namespace mmt
