"""Forward and input-gradient products in the two tile shapes that stand between 192 x 128, 128 x 128 and 64 x 128 (long contractions only): one row
past a tile edge and one short of it, K with a remainder and without, with and without addends; and sums of small whole numbers, exact in any order."""
import pytest

from paper_2408_04275_amd import binding as mm
from test_gpu_gemm_tiles import test_contraction_that_starts_anywhere as exact_sums
from test_gpu_ops import gemm_case
from util import gemm_route

BETWEEN = [(2305, 1032, 2568, "96x128"), (2303, 1024, 2560, "96x128"), (481, 4104, 2632, "96x128"), (3361, 1288, 2584, "160x128"),
           (1119, 4096, 4096, "160x128")]
LAYOUTS = [mm.GEMM_NT, mm.GEMM_NN]


@pytest.mark.parametrize("layout", LAYOUTS)
def test_routes(layout):
    for M, N, K, tile in BETWEEN:
        assert "%dx%d" % gemm_route(layout, M, N, K)[:2] == tile
        assert "%dx%d" % gemm_route(layout, M, N, 2552)[:2] not in ("96x128", "160x128")       # below 40 K steps


@pytest.mark.gpu
@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("M,N,K,tile", BETWEEN)
def test_tile_shape(layout, M, N, K, tile):
    gemm_case(mm.BF16, layout, M, N, K, seed=31)
    gemm_case(mm.BF16, layout, M, N, K, bias=True, residual=True, accumulate=K % 16 == 0, seed=32)
    exact_sums(layout, M, N, K, tile)
