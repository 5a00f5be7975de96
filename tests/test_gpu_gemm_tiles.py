"""Forward and input-gradient products in every tile shape the host can choose: sizes just past a tile edge, K with a remainder,
K shorter than the look-ahead of the K loop and longer, with and without addends."""
import pytest

from paper_2408_04275_amd import binding as mm
from test_gpu_ops import gemm_case

pytestmark = pytest.mark.gpu

# (M, N, K) and the tile the rule in csrc/gemm_mfma.hip picks for it
SHAPES = [(9, 40, 24, "64x64"), (65, 136, 712, "64x64"), (129, 72, 256, "64x64"), (323, 2848, 8, "64x128"), (577, 2184, 1096, "64x128"),
          (593, 3328, 200, "128x128"), (705, 3208, 584, "128x128"), (1095, 3592, 136, "192x128"), (2703, 2184, 136, "256x128"),
          (2312, 3480, 72, "160x256"), (3880, 2576, 136, "192x256"), (3485, 3464, 328, "224x256")]


@pytest.mark.parametrize("layout", [mm.GEMM_NT, mm.GEMM_NN])
@pytest.mark.parametrize("M,N,K,tile", SHAPES)
def test_gemm_tile_shape(layout, M, N, K, tile):
    gemm_case(mm.BF16, layout, M, N, K, seed=21)
    gemm_case(mm.BF16, layout, M, N, K, bias=True, residual=True, accumulate=K > 500, seed=22)
