"""Products in every tile shape the host can choose and cut along K, each at sizes that do take that form (test_routes.py asks the
library, also without a GPU): sizes just past a tile edge, K with a remainder, K shorter than the look-ahead of the K loop and longer, with and
without addends."""
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from test_gpu_ops import gemm_case
from util import gemm_route

pytestmark = pytest.mark.gpu

# (M, N, K) and the tile that the rule in csrc/gemm_mfma.hip picks for it
SHAPES = [(9, 40, 24, "64x64"), (65, 136, 712, "64x64"), (129, 72, 256, "64x64"), (323, 2848, 8, "64x128"), (577, 2184, 1096, "64x128"),
          (593, 3328, 200, "128x128"), (705, 3208, 584, "128x128"), (1095, 3592, 136, "192x128"), (2703, 2184, 136, "256x128"),
          (2312, 3480, 72, "160x256"), (3880, 2576, 136, "192x256"), (3485, 3464, 328, "224x256")]


@pytest.mark.parametrize("layout", [mm.GEMM_NT, mm.GEMM_NN])
@pytest.mark.parametrize("M,N,K,tile", SHAPES)
def test_gemm_tile_shape(layout, M, N, K, tile):
    assert "%dx%d" % gemm_route(layout, M, N, K)[:2] == tile
    gemm_case(mm.BF16, layout, M, N, K, seed=21)
    gemm_case(mm.BF16, layout, M, N, K, bias=True, residual=True, accumulate=K > 500, seed=22)


# a K of one to four steps: 256 x 256 tiles whose look-ahead is longer than K, several to a workgroup, ragged at every edge
@pytest.mark.parametrize("layout,M,N,K", [(mm.GEMM_NT, 4200, 3464, 8), (mm.GEMM_NN, 4200, 3464, 64), (mm.GEMM_NT, 4200, 3464, 136),
                                          (mm.GEMM_TN, 4104, 3464, 1), (mm.GEMM_TN, 4104, 3464, 65), (mm.GEMM_TN, 6152, 4040, 250)])
def test_short_contractions(layout, M, N, K):
    assert gemm_route(layout, M, N, K)[:2] == (256, 256)
    gemm_case(mm.BF16, layout, M, N, K, seed=26)
    gemm_case(mm.BF16, layout, M, N, K, residual=layout != mm.GEMM_TN, accumulate=True, seed=27)


# weight gradients: one row or column of 8 past a tile edge, K (the tokens) with every kind of remainder
WGRAD_SHAPES = [(8, 8, 1, "64x64"), (72, 136, 67, "64x64"), (520, 1032, 583, "64x64"), (1032, 2312, 321, "64x128"), (1544, 1288, 1411, "128x128"),
                (2056, 1928, 1411, "256x128")]


@pytest.mark.parametrize("M,N,K,tile", WGRAD_SHAPES)
def test_weight_gradient_tile_shape(M, N, K, tile):
    assert "%dx%d" % gemm_route(mm.GEMM_TN, M, N, K)[:2] == tile
    gemm_case(mm.BF16, mm.GEMM_TN, M, N, K, seed=23)
    gemm_case(mm.BF16, mm.GEMM_TN, M, N, K, accumulate=True, seed=24)


# few tiles and a long K: with the scratch of its size query an input gradient is cut along K (8, 7 and 5 chunks; K with a remainder, the last chunk shorter,
# rows and columns past a tile edge); scratch for fewer chunks allows no more than those, scratch for one leaves it whole
CUTS = [(366, 4096, 12288, None, 8), (257, 2056, 25608, None, 8), (257, 4104, 25608, None, 7), (520, 4096, 22016, None, 5),
        (2304, 1032, 22024, None, 5), (257, 4104, 25608, 5, 5), (257, 4104, 25608, 1, 1)]


@pytest.mark.parametrize("M,N,K,room,chunks", CUTS)
def test_input_gradient_cut_along_k(M, N, K, room, chunks, monkeypatch):
    size = room * M * N * 4 if room else mm.mmtrain_gemm_workspace_bytes(mm.GEMM_NN, M, N)
    assert gemm_route(mm.GEMM_NN, M, N, K, size)[2:] == (0, chunks)
    monkeypatch.setattr(mm, "mmtrain_gemm_workspace_bytes", lambda layout, m, n: size)
    gemm_case(mm.BF16, mm.GEMM_NN, M, N, K, accumulate=chunks == 5, seed=25, workspace=True)


# one tile per workgroup and 32 whole K tiles or more: every XCD starts at another eighth of K and goes round (31, and weight gradients: all at its start).  Small whole numbers
# have exact sums in any order, so each K tile has to come in exactly once; a start next to the end of K, a remainder, each tile shape
CIRCLES = [(mm.GEMM_NT, 9, 40, 2040, "64x64"), (mm.GEMM_NN, 129, 200, 2048, "64x64"), (mm.GEMM_TN, 72, 264, 2111, "64x64"), (mm.GEMM_NT, 577, 2184, 2568, "64x128"),
           (mm.GEMM_TN, 1032, 2312, 2183, "128x128"), (mm.GEMM_NN, 2304, 1032, 2184, "128x128"), (mm.GEMM_NT, 1031, 4096, 2112, "192x128"), (mm.GEMM_NT, 2703, 2184, 2624, "256x128"),
           (mm.GEMM_TN, 2056, 1928, 3000, "256x128"), (mm.GEMM_NN, 2312, 3480, 2056, "160x256"), (mm.GEMM_NT, 3880, 2576, 2696, "192x256"),
           (mm.GEMM_NT, 3485, 3464, 2120, "224x256"), (mm.GEMM_NN, 4096, 4000, 2072, "256x256"), (mm.GEMM_TN, 4096, 4096, 2113, "256x256")]


@pytest.mark.parametrize("layout,M,N,K,tile", CIRCLES)
def test_contraction_that_starts_anywhere(layout, M, N, K, tile):
    assert "%dx%d" % gemm_route(layout, M, N, K)[:2] == tile
    gen = torch.Generator().manual_seed(28)
    a, b = (torch.randint(-1, 2, (rows, K), generator=gen).float() for rows in (M, N))
    A = (a.t() if layout == mm.GEMM_TN else a).contiguous().bfloat16().cuda()
    B = (b if layout == mm.GEMM_NT else b.t()).contiguous().bfloat16().cuda()
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    assert mm.mmtrain_gemm(mm.BF16, layout, M, N, K, A, A.shape[1], B, B.shape[1], out, N) == 0
    torch.cuda.synchronize()
    assert torch.equal(out.cpu(), (a @ b.t()).bfloat16())
