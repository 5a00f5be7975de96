// Forward products of the bf16 GEMM in the tile shapes smaller than 256 x 256.
#include "gemm_mfma.h"

namespace mmt {
namespace gemm_detail {
hipError_t launch_nt(int shape, const GemmP &p, hipStream_t st) { return launch_tile_shape<true, true>(shape, p, st); }
}  // namespace gemm_detail
}  // namespace mmt
