"""fp32 storage on the fp32 matrix instruction: products at tile edges and remainders in both tile sizes, attention over ragged
packs and grouped heads, and an infinity or NaN in one segment staying in that segment."""
import numpy as np
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import workloads as wl
from paper_2408_04275_amd.harness import check
from test_gpu_ops import attn_case, gemm_case

pytestmark = pytest.mark.gpu


# one row past a 32 x 32 tile, K shorter than one wavefront's block, K with a remainder of 4 and of 12, 64 x 64 tiles with ragged
# edges; widths that are no multiple of 4, and a short K over many tiles (20; 92 too in a weight gradient), take the vector-ALU kernel
@pytest.mark.parametrize("layout", [mm.GEMM_NT, mm.GEMM_NN, mm.GEMM_TN])
@pytest.mark.parametrize("M,N,K", [(4, 4, 4), (36, 68, 20), (64, 32, 140), (100, 36, 1028), (1300, 1228, 92), (1300, 1228, 108), (1300, 1228, 20), (33, 30, 18)])
def test_gemm_f32_tiles(layout, M, N, K):
    M = M if layout != mm.GEMM_TN else (M + 3) // 4 * 4
    gemm_case(mm.F32, layout, M, N, K, seed=31)
    gemm_case(mm.F32, layout, M, N, K, bias=True, residual=True, accumulate=True, seed=32)


@pytest.mark.parametrize("nh,nkv,d", [(2, 2, 64), (6, 2, 64), (4, 1, 128), (3, 3, 128)])
def test_attention_f32(nh, nkv, d):
    rng = np.random.default_rng(nh * 1000 + d)
    lens = [1, 15, 16, 17, 130, 2, 301, 64, 33]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    attn_case(mm.F32, nh, nkv, d, cu, rng.integers(0, 2, len(lens)).astype(np.uint8), seed=33)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_attention_f32_non_finite_rows_stay_in_their_segment(d, value):
    # segment boundaries inside the 16-row blocks; the k, v and dO rows of one token of the middle segment are not finite
    cu, modes = np.array([0, 21, 50, 77], dtype=np.int32), np.array([0, 1, 0], dtype=np.uint8)
    nh, nkv, T, bad = 2, 1, 77, 30
    rng = np.random.default_rng(5)
    qkv = rng.standard_normal((T, (nh + 2 * nkv) * d)).astype(np.float32)
    d_o = rng.standard_normal((T, nh * d)).astype(np.float32)

    def run(qkv, d_o):
        desc = mm.make_desc(mm.DECODER, mm.F32, 64, nh, nkv, d, 64)
        batch = mm.PackedBatch.on_device(cu, modes)
        wsb = mm.mmtrain_attn_workspace_bytes(T, 3, nh)
        ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
        x, g = torch.from_numpy(qkv).cuda(), torch.from_numpy(d_o).cuda()
        o, lse, dx = torch.empty_like(g), torch.empty((nh, T), device="cuda"), torch.empty_like(x)
        check(mm.mmtrain_attn_fwd(desc, batch, x, o, lse, ws, wsb), "mmtrain_attn_fwd")
        check(mm.mmtrain_attn_bwd(desc, batch, x, o, lse, g, dx, ws, wsb), "mmtrain_attn_bwd")
        torch.cuda.synchronize()
        return o.cpu().numpy(), dx.cpu().numpy()

    clean = run(qkv, d_o)
    qkv[bad, nh * d:] = value
    d_o[bad] = value
    dirty = run(qkv, d_o)
    outside = np.r_[0:21, 50:77]
    for a, b in zip(clean, dirty):
        assert np.isfinite(b[outside]).all()
        # the same sums in another order (blocks with such a row take them element by element): a few roundings of at most 33 terms
        assert np.abs(a[outside] - b[outside]).max() <= 33 * 2.0 ** -23 * np.abs(a).max()
    assert not np.isfinite(dirty[0][21:50]).all()
