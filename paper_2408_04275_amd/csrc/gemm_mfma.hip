// Host side of the bf16 GEMM (kernel: gemm_mfma.h): which tile shape, the K-cut of a gradient's partly filled last round, and
// the 256 x 256 kernels.
#include "gemm_mfma.h"
#include <algorithm>
#include <cmath>

namespace mmt {

using namespace gemm_detail;

namespace {

constexpr int TILE = 256;              // the largest tile, and the one the K-cut works with

// C (+)= sum over the K chunks of the fp32 partial products; C is bf16 or fp32.  4 elements per thread.  The partial products
// are dense 256 x 256 blocks of the tiles [tile_begin, tile_begin + tile_count) of the tile order: block
// (s * tile_count + j) belongs to chunk s of tile tile_begin + j.  64 workgroups per tile.
template <typename TC>
__global__ __launch_bounds__(256) void tail_reduce_kernel(const float *__restrict__ part, int splits, int tile_begin, int tile_count,
                                                          int tiles_m, int tiles_n, int M, int N, TC *__restrict__ C, int ldc,
                                                          int accumulate) {
    const int j = blockIdx.x >> 6;
    const int e0 = ((blockIdx.x & 63) * 256 + threadIdx.x) * 4;         // element of the block: row e0 / 256, column e0 % 256
    int tm, tn;
    tile_coords(tile_begin + j, tiles_m, tiles_n, tm, tn);
    const int m = tm * TILE + (e0 >> 8), n = tn * TILE + (e0 & 255);
    if (m >= M || n >= N) return;                                       // N is a multiple of 8: the 4 columns are in or out together
    f32x4 v = *reinterpret_cast<const f32x4 *>(part + ((size_t)j << 16) + e0);
    for (int sp = 1; sp < splits; ++sp) v += *reinterpret_cast<const f32x4 *>(part + ((size_t)(sp * tile_count + j) << 16) + e0);
    TC *c = C + (size_t)m * ldc + n;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float r = v[e];
        if (accumulate) r += Elem<TC>::load(c + e);
        Elem<TC>::store(c + e, r);
    }
}

// C (+)= sum over the K chunks of the M x N fp32 partial products, dense and one after the other (N a multiple of 8).
// Streams (splits * 4 + 2) bytes per element; 8 elements per thread, rows on the grid's y.
__global__ __launch_bounds__(256) void sum_chunks_kernel(const float *__restrict__ part, int splits, int M, int N, bf16_t *__restrict__ C,
                                                         int ldc, int accumulate) {
    const int n = (blockIdx.x * 256 + threadIdx.x) * 8;
    if (n >= N) return;
    const size_t plane = (size_t)M * N;
    for (int m = blockIdx.y; m < M; m += gridDim.y) {
        const float *src = part + (size_t)m * N + n;
        f32x4 a = *reinterpret_cast<const f32x4 *>(src), b = *reinterpret_cast<const f32x4 *>(src + 4);
        for (int s = 1; s < splits; ++s) {
            a += *reinterpret_cast<const f32x4 *>(src + s * plane);
            b += *reinterpret_cast<const f32x4 *>(src + s * plane + 4);
        }
        bf16_t *c = C + (size_t)m * ldc + n;
        if (accumulate)
#pragma unroll
            for (int e = 0; e < 4; ++e) { a[e] += bf16_to_f32(c[e]); b[e] += bf16_to_f32(c[4 + e]); }
#pragma unroll
        for (int e = 0; e < 4; ++e) { Elem<bf16_t>::store(c + e, a[e]); Elem<bf16_t>::store(c + 4 + e, b[e]); }
    }
}

GemmP params(const GemmArgs &g) {
    GemmP p;
    p.M = g.M; p.N = g.N; p.K = g.K;
    p.A = (const bf16_t *)g.A; p.lda = g.lda;
    p.B = (const bf16_t *)g.B; p.ldb = g.ldb;
    p.C = (bf16_t *)g.C; p.ldc = g.ldc;
    p.bias = (const bf16_t *)g.bias;
    p.residual = (const bf16_t *)g.residual;
    p.accumulate = g.accumulate ? 1 : 0;
    p.c_f32 = g.c_f32 ? 1 : 0;
    p.tiles_m = ceil_div(g.M, TILE);
    p.tiles_n = ceil_div(g.N, TILE);
    p.splits = 1; p.k_chunk = g.K;
    p.tile_begin = 0; p.tile_count = p.tiles_m * p.tiles_n; p.compact = 0; p.late_start = 0;
    p.clock_probe = g.clock_probe;
    return p;
}

// all K chunks of the tiles p covers as fp32 partial products (p.C: scratch)
hipError_t launch_partials(int layout, const GemmP &p, hipStream_t st) {
    return layout == GEMM_TN ? launch<false, false, false, true, Tile256>(p, st)
                             : launch<true, false, false, true, Tile256>(p, st);
}

}  // namespace

bool gemm_mfma_supported(const GemmArgs &g) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
    if (g.c_f32 && (g.layout != GEMM_TN || g.bias || g.residual)) return false;   // fp32 output: weight gradients only
    if (g.c_f32 && g.ldc > 1 << 26) return false;                                 // 16 rows of it are addressed with 32-bit byte offsets
    if ((g.lda | g.ldb | g.ldc | g.N) & 7) return false;
    const bool a_kc = g.layout != GEMM_TN, b_kc = g.layout == GEMM_NT;
    if ((a_kc || b_kc) && (g.K & 7)) return false;
    if (!a_kc && (g.M & 7)) return false;
    // operands are addressed with 32-bit byte offsets, tile overhang included
    const size_t rows_a = a_kc ? g.M : g.K, rows_b = b_kc ? g.N : g.K;
    if ((rows_a + 256) * (size_t)g.lda * 2 >= 0xfff00000ull || (rows_b + 256) * (size_t)g.ldb * 2 >= 0xfff00000ull)
        return false;
    const uintptr_t bits = (uintptr_t)g.A | (uintptr_t)g.B | (uintptr_t)g.C | (uintptr_t)g.bias | (uintptr_t)g.residual;
    return (bits & 15) == 0;
}

// The last, partly filled round of a large GEMM.  With one workgroup per compute unit the tiles are worked off in
// rounds of n_cu; when the last round holds at most half that many tiles, each of them is cut along K into
// n_cu / tiles chunks so that the round takes a fraction of a full one.  Returns the number of chunks (1: do not
// split) and the number of tiles in that round.  Only for input- and weight-gradient GEMMs without bias or
// residual, with scratch for the partial products, and only for long K: a partly filled round is faster than a full
// one to begin with (fewer active compute units run at a higher clock), and the cut costs two extra launches.
// Measured on the 22016 x 4096 x 8192 weight gradient (96 tiles in the last round, 2 chunks): 1.137 -> 1.100 ms; the
// 8192 x 11008 x 4096 input gradient gains nothing, hence the bound on K.
static int tail_chunks(long tiles, long K, int n_cu) {
    const long rem = tiles % n_cu;
    if (tiles < n_cu || rem == 0 || rem > n_cu / 2) return 1;
    const long s = std::min({n_cu / rem, K / 512, 16l});
    return s >= 2 && K * (s - 1) / s >= 4096 ? (int)s : 1;
}
int gemm_mfma_tail_splits(const GemmArgs &g, int n_cu, int &tail_tiles) {
    tail_tiles = 0;
    if (g.layout == GEMM_NT || !g.split_ws || g.bias || g.residual) return 1;
    const long tiles = (long)ceil_div(g.M, TILE) * ceil_div(g.N, TILE);
    long s = tail_chunks(tiles, g.K, n_cu);
    if (s < 2) return 1;
    const long rem = tiles % n_cu, fit = (long)(g.split_ws_bytes / ((size_t)rem * TILE * TILE * 4));
    s = s < fit ? s : fit;
    if (s < 2 || (long)g.K * (s - 1) / s < 4096) return 1;
    tail_tiles = (int)rem;
    return (int)s;
}

// chunks that few_tile_splits may cut an input gradient into: no more tiles than compute units, 512 of K each
constexpr int MAX_CHUNKS = 8;
static int few_tile_chunks(long tiles, long K, int n_cu) { return (int)std::min({(long)MAX_CHUNKS, n_cu / tiles, K / 512}); }

// Scratch with which neither cut is ever restricted, for an input gradient of at most M rows: the most that any row count up to M
// uses, so that a caller's buffer for its longest pack serves every shorter one (the number of chunks falls as the rows grow).
constexpr int WHOLE_CHIP = 256;                                       // compute units
size_t gemm_mfma_nn_scratch(long M, long N, long K) {
    const long tn = (N + TILE - 1) / TILE, tm = (M + TILE - 1) / TILE;
    size_t most = 0;
    for (long s = few_tile_chunks(tn, K, WHOLE_CHIP); s >= 2; --s)    // the most rows that s chunks are possible for
        most = std::max(most, (size_t)s * std::min(M, WHOLE_CHIP / (s * tn) * TILE) * N * 4);
    const long first = (WHOLE_CHIP + tn - 1) / tn;                    // the tile count modulo 256 repeats after 256 tile rows at most
    for (long t = first; t <= tm && t < first + WHOLE_CHIP; ++t) {
        const int s = tail_chunks(t * tn, K, WHOLE_CHIP);
        if (s >= 2) most = std::max(most, (size_t)s * (t * tn % WHOLE_CHIP) * TILE * TILE * 4);
    }
    return most;
}
// The same for a weight gradient over at most K tokens (chunks grow with K)
size_t gemm_mfma_tn_scratch(long M, long N, long K) {
    const long tiles = (M + TILE - 1) / TILE * ((N + TILE - 1) / TILE);
    const int s = tail_chunks(tiles, K, WHOLE_CHIP);
    return s >= 2 ? (size_t)s * (tiles % WHOLE_CHIP) * TILE * TILE * 4 : 0;
}

// Weight-gradient products whose outputs have few tiles (at most 128: a narrow layer), run together: every tile of every
// product is one work item with the whole contraction, so nothing goes through scratch and one launch fills the chip that
// each product alone would leave mostly idle.
bool gemm_mfma_few_tiles(const GemmArgs &g) {
    return g.layout == GEMM_TN && !g.bias && !g.residual && gemm_mfma_supported(g) &&
           (long)ceil_div(g.M, TILE) * ceil_div(g.N, TILE) <= 128;
}

// Tile shape of a product, or of a group of products of one layout and contraction.  The 256 x 256 tile does the most arithmetic per byte
// fetched, but a product with few of them leaves most compute units idle (one image of 576 patches through a 1024 x 1024 linear: 12 tiles)
// and one with a few more than a whole number of rounds runs a nearly empty last one.  The rule is the time each shape needs: every compute
// unit works off ceil(tiles / compute units) tiles one after the other, a tile costs a start and epilogue plus so much per 64-deep K step,
// and a step gets slower as the chip fills (clock, L2).  The constants (us) are least-squares fits to 150 random shapes each for the
// forward and input-gradient products (250 - 12000 rows, widths 1024 - 22016; nine tile shapes) and for the weight gradients (512 - 5120
// square to oblong, K = 250 - 12000; five shapes, A and B both strided): the shape the rule picked was 0.03 % / 0.07 % slower than the best
// of them on average, 2 % / 7 % at worst (the two shapes between, 160 x 128 and 96 x 128, came later: see MIN_K_BETWEEN).  The K loop of
// one round and the fp32 epilogue have become faster since; another 140 and 60 random shapes, half of them from HBM: 0.4 % / 0.5 % on
// average, 18 % (345 x 2752 x 9592 from HBM, 78 us in 64 x 64) / 9 % (3944 x 1208 x 379, 11.4 us in 256 x 128) at worst.  Against 256 x 256
// throughout it measured 65.9 -> 13.5 us on the 576 x 1024 x 4096 forward product (64 x 64 tiles), 22.6 -> 14.8 us on 2304 x 3072 x 1024
// (256 x 128), 72.2 -> 65.6 us on 9536 x 1024 x 4096 (160 x 256), and 58.3 -> 25.8 us on the 4096 x 1024 x 2880 weight gradient, which was
// cut along K before (128 x 128); products of whole rounds of large tiles stay where they were.
constexpr size_t FROM_HBM_BYTES = size_t(96) << 20;     // operands beyond this mostly come from HBM and not from the memory-side cache
struct TileCost { int shape, bm, bn; double tile, step; };
constexpr TileCost COST_ROWS[] = {                     // K-contiguous A
    {TILE_256, 256, 256, 4.13, 0.958}, {TILE_224, 224, 256, 2.92, 0.866}, {TILE_192, 192, 256, 2.19, 0.778},
    {TILE_160, 160, 256, 1.37, 0.694}, {TILE_256x128, 256, 128, 1.15, 0.575}, {TILE_192x128, 192, 128, 1.01, 0.462},
    {TILE_160x128, 160, 128, 0.89, 0.405}, {TILE_128, 128, 128, 0.77, 0.348}, {TILE_96x128, 96, 128, 0.60, 0.295},
    {TILE_64x128, 64, 128, 0.0, 0.223}, {TILE_64, 64, 64, 0.0, 0.142}};
constexpr TileCost COST_WGRAD[] = {
    {TILE_256, 256, 256, 4.05, 1.044}, {TILE_256x128, 256, 128, 2.10, 0.618}, {TILE_128, 128, 128, 1.49, 0.389},
    {TILE_64x128, 64, 128, 0.10, 0.254}, {TILE_64, 64, 64, 0.0, 0.176}};

// 160 x 128 and 96 x 128 stand between the older shapes, where 128 x 128 or 192 x 128 leave a quarter to a half of the compute units idle:
// such products are bound by what a unit copies into LDS per K step, which falls with the tile (96 x 128: 28 KiB instead of 32, 160 x 128:
// 36 instead of 40).  From the cache / from HBM, us: 2304 x 1024 x 4096 in 128 x 128 (144 tiles) -> 96 x 128 (192) 27.9 -> 24.9 / 38.4 ->
// 31.8, 2880 x 1024 x 4096 NN 30.7 -> 27.8 / 36.0 -> 32.8, 1031 x 4096 x 11008 in 192 x 128 (192) -> 160 x 128 (224) 90.1 -> 81.1 / 100.6
// -> 94.9; of 67 random products of 40 and more K steps the rule took one of them for 18, which became 2 to 15 % faster, and none slower
// than two runs of one build differ.  Another 330 of 40 steps and more: from the cache 7 % faster on average, seven of them 2 % and more
// slower; from HBM 6 %, but with as many tiles as before, of fewer rows, 7 % slower (284 x 7368 x 10048 in 174 tiles of 128 x 128 -> 96 x
// 128 74 -> 88 us, 442 x 8248 x 7616 in 195 of 192 x 128 -> 160 x 128 16 %), with up to 15 % more 2 % slower, 15 to 30 % more 5 % faster,
// beyond 12 %; six and seven row tiles instead of five and six, below 700 rows, 1 % slower (520 x 4096 x 14336 92 -> 98 us) where those of
// longer ones gain.  So operands that come from HBM need 15 % more tiles, 22 % up to 1024 rows, or a full round of them (600 x 8192 x 8192
// 82 -> 79 us).  Below 40 steps, 60 products of 6 to 39: 7 % faster from the cache and 6 % from HBM on average, between 2 % slower (384
// deep) and 13 % faster, with few rows from HBM up to 13 % slower.  Those keep the older shapes, which the tests of short contractions
// name.
constexpr int MIN_K_BETWEEN = 2560;
constexpr double MIN_MORE_BETWEEN = 1.15, MIN_MORE_FEW_ROWS = 1.22;
struct LaunchCost { double launch, rounds_power, load; };
constexpr LaunchCost LAUNCH_ROWS = {3.4, 1.042, 0.276}, LAUNCH_WGRAD = {3.7, 1.079, 0.105};
long tiles_of(const TileCost &t, const GemmArgs *gs, int n) {
    long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (long)ceil_div(gs[i].M, t.bm) * ceil_div(gs[i].N, t.bn);
    return tiles;
}
double tiles_us(const TileCost &t, const LaunchCost &c, long tiles, int K, int n_cu) {
    const double share = (double)tiles / n_cu, fill = share < 1. ? share * share : 1.;
    return c.launch + pow(ceil(share), c.rounds_power) * (t.tile + ceil_div(K, BK) * t.step * (1. + c.load * fill));
}
// older_us: the estimate without the two shapes between
template <int N>
int choose_tile(const TileCost (&table)[N], const LaunchCost &cost, const GemmArgs *gs, int n, int n_cu, double &best_us, double &older_us) {
    int best = TILE_256;
    long older_tiles = 0;
    size_t bytes = 0;
    for (int i = 0; i < n; ++i) bytes += (size_t)(gs[i].M + gs[i].N) * gs[i].K * 2;
    const bool from_hbm = bytes > FROM_HBM_BYTES;
    for (const bool between : {false, true}) {
        if (between && gs[0].K < MIN_K_BETWEEN) break;
        for (const TileCost &t : table) {
            if ((t.shape == TILE_160x128 || t.shape == TILE_96x128) != between) continue;
            const long tiles = tiles_of(t, gs, n);
            if (between && from_hbm && tiles % n_cu && tiles < (gs[0].M < 1024 ? MIN_MORE_FEW_ROWS : MIN_MORE_BETWEEN) * older_tiles) continue;
            const double us = tiles_us(t, cost, tiles, gs[0].K, n_cu);
            // a smaller tile moves more bytes per product: only for a gain beyond the fit's error, and beyond what they cost more from HBM
            // (operands of more than 96 MB: 1397 x 28672 x 5120 takes 336 us in 256 x 256 and 379 in 160 x 256, which the model puts 4 % ahead)
            if (t.shape == TILE_256 || us < best_us * (best != TILE_256 ? 1. : from_hbm ? 0.95 : 0.98)) {
                best = t.shape;
                best_us = us;
                if (!between) older_tiles = tiles;
            }
        }
        if (!between) older_us = best_us;
    }
    return best;
}
// A K of at most four steps lies below what the constants were fitted to, and there a tile's time is mostly that of its stores, which
// the model lacks: 256 x 256 wherever its rounds are well filled.  Measured with the model's choice -> 256 x 256, us: forward and
// input gradients 28360 x 7384 x 16 228 -> 175, 9504 x 4344 x 16 41 -> 33, 1000 x 28672 x 192 25.2 -> 22.1 (rounds 98, 95 and 88 % full),
// but 6000 x 4096 x 128 18.8 -> 19.8 (75 %); weight gradients 4096 x 4096 x 64 12.6 -> 10.6, 28672 x 4096 x 64 64 -> 55, 4096 x 11008 x
// 128 36.5 -> 30.6, 6144 x 2048 x 160 14.3 -> 13.3 (75 %).
bool short_k_full_rounds(const GemmArgs *gs, int n, int n_cu) {
    if (gs[0].K > 4 * BK) return false;
    long tiles = 0;
    for (int i = 0; i < n; ++i) tiles += (long)ceil_div(gs[i].M, TILE) * ceil_div(gs[i].N, TILE);
    const double filled = (double)tiles / ((double)ceil_div(tiles, n_cu) * n_cu);
    return filled >= (gs[0].layout == GEMM_TN ? 0.75 : 0.8);
}
int choose_tile(const GemmArgs *gs, int n, int n_cu, double &us, double &older_us) {
    us = older_us = 0.;
    if (short_k_full_rounds(gs, n, n_cu)) return TILE_256;
    return gs[0].layout == GEMM_TN ? choose_tile(COST_WGRAD, LAUNCH_WGRAD, gs, n, n_cu, us, older_us) : choose_tile(COST_ROWS, LAUNCH_ROWS, gs, n, n_cu, us, older_us);
}
int choose_tile(const GemmArgs *gs, int n, int n_cu) {
    double us, older_us;
    return choose_tile(gs, n, n_cu, us, older_us);
}

// An input gradient (NN) with few tiles and a very long K, cut along K as a whole: `splits` chunks of 256 x 256 tiles through scratch, and
// a kernel that adds them up.  The smaller tile shapes fill the chip too, but at half or a quarter of the arithmetic per byte on every K
// step; the cut pays for its scratch traffic and second launch once, so it wins where K is long. The rule compares choose_tile's estimate
// with the same model for K / splits, plus the reduction (its launch and 0.345 us per MB), and asks for 5 % as both are fits.  The tile
// shapes' constants hold for operands that the memory-side cache keeps (256 MB); from HBM they take 1.1 to 1.6 times as long (the 256 x 256
// chunks, each of which one XCD's L2 reads once, do not), so operands of more than 96 MB, most of which are a large layer's weights, count
// against them: their estimate then stands at 1.15 times itself instead of 0.95.  Measured with operands from HBM, tile shape -> cut: 1031
// x 4096 x 22016 (the gate / up input gradient of a short pack) 209 -> 169 us in three chunks, 1031 x 4096 x 12288 (QKV) 116 -> 100, 1031 x
// 4096 x 11008 104 -> 92, 366 x 4096 x 12288 87 -> 50 in eight, 1031 x 1280 x 22016 129 -> 67 in eight, 2304 x 1024 x 11008 93 -> 62 in
// six; from the cache the first three 185 -> 164, 98 -> 98, 88 -> 91.  With two chunks it is about even: 1500 x 4096 x 22016 248 -> 238
// (from the cache 210 -> 222), 2047 x 4096 x 22016 304 -> 266, 700 x 8192 x 13824 145 -> 157.  Up to K = 8192 the tile shapes are ahead.
// The estimate compared with leaves 160 x 128 and 96 x 128 out (gemm_mfma_plan): these fall furthest behind it from HBM.  Cut -> tile, from
// the cache / from HBM: 1031 x 2048 x 11008 in six 57 -> 59 / 59 -> 82, 1984 x 1280 x 14336 72 -> 83 / 77 -> 108, 576 x 5120 x 11264 in
// four 74 -> 68 / 77 -> 101, 1088 x 4096 x 9728 in three 85 -> 80 / 88 -> 98.  A cut in two is weighed against them: 640 x 8192 x 13824 154
// -> 124 / 154 -> 139, 576 x 8192 x 27648 286 -> 259 / 288 -> 263.
int few_tile_splits(const GemmArgs &g, int n_cu, double best_us) {
    if (g.layout != GEMM_NN || g.bias || g.residual || !g.split_ws) return 1;
    const long tiles = (long)ceil_div(g.M, TILE) * ceil_div(g.N, TILE);
    const size_t plane = (size_t)g.M * g.N * 4;
    best_us *= (size_t)(g.M + g.N) * g.K * 2 > FROM_HBM_BYTES ? 1.15 : 0.95;
    int best = 1;
    for (int s = 2; s <= few_tile_chunks(tiles, g.K, n_cu) && s * plane <= g.split_ws_bytes; ++s) {
        const double fill = (double)(s * tiles) / n_cu;
        const double us = 3.4 + 4.13 + ceil_div(ceil_div(g.K, BK), s) * 0.958 * (1. + 0.276 * fill * fill) + 3.4 + 0.345e-6 * plane * (s + 0.5);
        if (us < best_us) { best = s; best_us = us; }
    }
    return best;
}

// Sums ride along where the launch leaves compute units without a tile, no full round or a last one that is at most three quarters full,
// and where they are done about when that round is.  The few workgroups that add them up take longer than a launch of their own would: a
// unit of 32 columns about 2 us of latency and 5 ns per row.  What they spare is that launch and its run, 8 us together (measured: 2 to
// 20). Backward pass of an encoder layer, alone -> along, us: 512 wide, 300 and 3000 tokens 76.4 -> 74.2, 153.7 -> 146.0; 1024 wide, 900
// and 9536 139.6 -> 134.1, 627 -> 619; 1280 wide (600 tiles in 2.34 rounds), 900, 2304 and 6000 202 -> 221, 314 -> 317, 664 -> 651; 1408
// and 1536 wide, whose feed-forward gradients do not take part, 300, 900, 1500 and 2304 tokens 144 -> 155, 238.5 -> 252, 306 -> 308, 410 ->
// 399.  In those, and in 512, 1536 and 2048 wide decoder layers, 64 to 9536 tokens, nothing that rides along by this rule was slower than
// alone by more than two runs of one build differ.
constexpr double SUM_UNIT_US = 2., SUM_ROW_US = 0.005, SUMS_LAUNCH_US = 8.;
bool gemm_mfma_group_has_room(const GemmArgs *gs, int n, const ReduceJobSet &sums, int n_cu) {
    if (n <= 0) return false;
    double sum_us = 0.;
    const int shape = choose_tile(gs, n, n_cu);
    for (int j = 0; j < 8; ++j) sum_us += (sums.units[j + 1] - sums.units[j]) * (SUM_UNIT_US + SUM_ROW_US * sums.rows[j]);
    sum_us /= std::max(1, std::min(sums.units[8], GROUP_SUM_WORKGROUPS));
    for (const TileCost &t : COST_WGRAD)
        if (t.shape == shape) {
            const long tiles = tiles_of(t, gs, n), last = tiles % n_cu;
            return last > 0 && 4 * last <= 3 * n_cu &&
                   sum_us <= tiles_us(t, LAUNCH_WGRAD, tiles, gs[0].K, n_cu) / ceil_div(tiles, n_cu) + SUMS_LAUNCH_US;
        }
    return false;
}
bool gemm_mfma_group_has_room(const GemmArgs *gs, int n, const ReduceJobSet &sums) {
    int n_cu = 0;
    return compute_units(n_cu) == hipSuccess && gemm_mfma_group_has_room(gs, n, sums, n_cu);
}
hipError_t gemm_mfma_group(const GemmArgs *gs, int n, const ReduceJobSet *reduce, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    if (n > MAX_GROUP) return hipErrorInvalidValue;
    GemmP p[MAX_GROUP];
    for (int i = 0; i < n; ++i) {
        if (!gemm_mfma_few_tiles(gs[i]) || gs[i].K != gs[0].K || gs[i].accumulate != gs[0].accumulate || gs[i].c_f32 != gs[0].c_f32)
            return hipErrorInvalidValue;
        p[i] = params(gs[i]);
    }
    int n_cu = 0;
    hipError_t e = compute_units(n_cu);
    if (e != hipSuccess) return e;
    return launch_tn(choose_tile(gs, n, n_cu), p, n, reduce, st);
}

GemmPlan gemm_mfma_plan(const GemmArgs &g, int n_cu) {
    GemmPlan plan = {TILE_256, TILE, TILE, 0, 1, g.K};
    int chunks = gemm_mfma_tail_splits(g, n_cu, plan.tail_tiles);
    if (plan.tail_tiles == 0) {
        double us, older_us;
        const int shape = choose_tile(&g, 1, n_cu, us, older_us);
        chunks = few_tile_splits(g, n_cu, older_us);
        if (chunks == 2) chunks = few_tile_splits(g, n_cu, us);
        if (chunks == 1) plan.shape = shape;
    }
    for (const TileCost &t : COST_ROWS)
        if (t.shape == plan.shape) { plan.tile_m = t.bm; plan.tile_n = t.bn; }
    if (chunks > 1) {
        plan.k_chunk = ceil_div(ceil_div(g.K, chunks), BK) * BK;
        plan.chunks = ceil_div(g.K, plan.k_chunk);
    }
    return plan;
}

int gemm_mfma_late_start(const GemmArgs &g, int n_cu) {
    const GemmPlan plan = gemm_mfma_plan(g, n_cu);
    const int items = ceil_div(g.M, plan.tile_m) * ceil_div(g.N, plan.tile_n) - plan.tail_tiles;
    auto units = [&](auto TS_) {
        typedef decltype(TS_) TS;
        return late_start<TS>(g.accumulate, g.K, items, std::min(items, n_cu * TS::PER_CU));
    };
    if (!g.c_f32) return 0;
    switch (plan.shape) {
        case TILE_256x128: return units(Tile256x128{});
        case TILE_128: return units(Tile128{});
        case TILE_64x128: return units(Tile64x128{});
        case TILE_64: return units(Tile64{});
        default: return units(Tile256{});
    }
}

hipError_t gemm_mfma(const GemmArgs &g, hipStream_t st) {
    GemmP p = params(g);
    int n_cu = 0;
    hipError_t e = compute_units(n_cu);
    if (e != hipSuccess) return e;
    const GemmPlan plan = gemm_mfma_plan(g, n_cu);
    const int tail_tiles = plan.tail_tiles;
    if (plan.chunks > 1 && tail_tiles == 0) {
        p.k_chunk = plan.k_chunk; p.splits = plan.chunks;
        p.C = (bf16_t *)g.split_ws; p.ldc = g.N; p.accumulate = 0; p.c_f32 = 1;
        if ((e = launch_partials(g.layout, p, st)) != hipSuccess) return e;
        if (g.chunks) { *g.chunks = p.splits; return hipSuccess; }
        sum_chunks_kernel<<<dim3(ceil_div(g.N, 2048), g.M < 4096 ? g.M : 4096), 256, 0, st>>>((const float *)g.split_ws, p.splits, g.M, g.N,
                                                                                               (bf16_t *)g.C, g.ldc, g.accumulate ? 1 : 0);
        return hipGetLastError();
    }
    if (plan.shape != TILE_256)
        return g.layout == GEMM_NT ? launch_nt(plan.shape, p, st) : g.layout == GEMM_NN ? launch_nn(plan.shape, p, st) : launch_tn(plan.shape, &p, 1, nullptr, st);
    p.tile_count -= tail_tiles;                                       // the full rounds
    const bool add = p.residual || p.accumulate;
    if (g.c_f32) e = launch<false, false, false, true, Tile256>(p, st);
    else if (g.layout == GEMM_NT) e = add ? launch<true, true, true, false, Tile256>(p, st) : launch<true, true, false, false, Tile256>(p, st);
    else if (g.layout == GEMM_NN) e = add ? launch<true, false, true, false, Tile256>(p, st) : launch<true, false, false, false, Tile256>(p, st);
    else e = add ? launch<false, false, true, false, Tile256>(p, st) : launch<false, false, false, false, Tile256>(p, st);
    if (e != hipSuccess || tail_tiles == 0) return e;
    GemmP t = params(g);
    t.C = (bf16_t *)g.split_ws; t.accumulate = 0; t.c_f32 = 1;
    t.tile_begin = p.tile_count; t.tile_count = tail_tiles; t.compact = 1;
    t.k_chunk = plan.k_chunk; t.splits = plan.chunks;
    e = launch_partials(g.layout, t, st);
    if (e != hipSuccess) return e;
    if (g.c_f32)
        tail_reduce_kernel<float><<<tail_tiles * 64, 256, 0, st>>>((const float *)g.split_ws, t.splits, t.tile_begin, tail_tiles, t.tiles_m,
                                                                  t.tiles_n, g.M, g.N, (float *)g.C, g.ldc, g.accumulate ? 1 : 0);
    else
        tail_reduce_kernel<bf16_t><<<tail_tiles * 64, 256, 0, st>>>((const float *)g.split_ws, t.splits, t.tile_begin, tail_tiles, t.tiles_m,
                                                                   t.tiles_n, g.M, g.N, (bf16_t *)g.C, g.ldc, g.accumulate ? 1 : 0);
    return hipGetLastError();
}

}  // namespace mmt
