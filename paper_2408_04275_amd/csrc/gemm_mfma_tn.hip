// Weight-gradient products of the bf16 GEMM, one or several per launch, in the tile shapes smaller than 256 x 256.
#include "gemm_mfma.h"

namespace mmt {
namespace gemm_detail {
namespace {

template <bool HAS_ADD, bool OUT_F32, class TS>
hipError_t launch_group(GemmGroup &g, hipStream_t st) {
    static std::atomic<bool> configured{false};
    auto kern = gemm_mfma_kernel<false, false, HAS_ADD, OUT_F32, TS, GemmGroup>;
    hipError_t e = allow_lds(configured, reinterpret_cast<const void *>(kern), TS::SMEM);
    if (e != hipSuccess) return e;
    int n_cu = 0;
    e = compute_units(n_cu);
    if (e != hipSuccess) return e;
    const int items = g.first[MAX_GROUP], room = n_cu * TS::PER_CU;
    if (items <= 0) return hipSuccess;
    const int workgroups = items < room ? items : room;
    g.workgroups = workgroups;
    const int sums = g.reduce.units[8] < GROUP_SUM_WORKGROUPS ? g.reduce.units[8] : GROUP_SUM_WORKGROUPS;
    static_assert(TS::SMEM >= REDUCE_LDS, "room for a reduction");
    g.p[0].late_start = OUT_F32 ? late_start<TS>(g.p[0].accumulate, g.p[0].K, items, workgroups) : 0;
    kern<<<workgroups + sums, 256, TS::SMEM, st>>>(g);
    return hipGetLastError();
}

template <class TS>
hipError_t launch_shape(const GemmP *p, int n, const ReduceJobSet *reduce, hipStream_t st) {
    GemmGroup g = {};
    if (reduce) g.reduce = *reduce;
    int total = 0;
    for (int i = 0; i < MAX_GROUP; ++i) {
        g.first[i] = total;
        g.p[i] = p[i < n ? i : 0];
        g.p[i].tiles_m = ceil_div(g.p[i].M, TS::BM); g.p[i].tiles_n = ceil_div(g.p[i].N, TS::BN);
        g.p[i].tile_count = g.p[i].tiles_m * g.p[i].tiles_n;
        if (i < n) total += g.p[i].tile_count;
    }
    g.first[MAX_GROUP] = total;
    g.n = n;
    if (p[0].c_f32) return launch_group<false, true, TS>(g, st);
    return p[0].accumulate || p[0].residual ? launch_group<true, false, TS>(g, st) : launch_group<false, false, TS>(g, st);
}

}  // namespace

hipError_t launch_tn(int shape, const GemmP *p, int n, const ReduceJobSet *reduce, hipStream_t st) {
    switch (shape) {
        case TILE_256: return launch_shape<Tile256>(p, n, reduce, st);
        case TILE_256x128: return launch_shape<Tile256x128>(p, n, reduce, st);
        case TILE_128: return launch_shape<Tile128>(p, n, reduce, st);
        case TILE_64x128: return launch_shape<Tile64x128>(p, n, reduce, st);
        case TILE_64: return launch_shape<Tile64>(p, n, reduce, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace gemm_detail
}  // namespace mmt
