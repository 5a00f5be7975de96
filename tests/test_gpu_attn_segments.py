"""A call of attention alone finds segments by itself up to 64 of them, one per lane of a wavefront, and through a table of tokens beyond: either side
of that line, with empty segments at both ends, next to each other and on tile edges, and one mask mode for all."""
import numpy as np
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd.harness import check
from test_gpu_ops import attn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nh,nkv,d", [(3, 3, 64), (4, 1, 128), (2, 2, 80)])
@pytest.mark.parametrize("segments", [2, 63, 64, 65, 130])
def test_either_side_of_the_line(nh, nkv, d, segments):
    rng = np.random.default_rng(segments)
    cuts = np.sort(rng.integers(0, 700, segments - 1))
    cuts[: segments // 8] = 0
    cuts[segments // 2: segments // 2 + segments // 8] = 256
    cuts[segments - 1 - segments // 8:] = 700
    cu = np.concatenate([[0], np.sort(cuts), [700]]).astype(np.int32)
    attn_case(mm.BF16, nh, nkv, d, cu, rng.integers(0, 2, segments).astype(np.uint8), seed=58)


# no array of modes but one mode for all segments: what the same modes spelled out give, bit for bit
@pytest.mark.parametrize("nh,nkv,d", [(3, 3, 64), (4, 1, 128), (2, 2, 80)])
@pytest.mark.parametrize("mode", [mm.MASK_CAUSAL, mm.MASK_BIDIR])
@pytest.mark.parametrize("segments", [1, 64, 65])
def test_one_mode_for_all(nh, nkv, d, mode, segments):
    T = 700
    cuts = np.random.default_rng(segments).integers(0, T, segments - 1)
    cu = np.concatenate([[0], np.sort(cuts), [T]]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(59)
    qkv = torch.randn((T, (nh + 2 * nkv) * d), device="cuda", generator=g).to(torch.bfloat16)
    d_o = torch.randn((T, nh * d), device="cuda", generator=g).to(torch.bfloat16)
    desc = mm.make_desc(mm.DECODER, mm.BF16, 64, nh, nkv, d, 64)
    n = mm.mmtrain_attn_workspace_bytes(T, segments, nh)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")

    def run(batch):
        o, d_qkv, lse = torch.zeros_like(d_o), torch.zeros_like(qkv), torch.zeros((nh, T), device="cuda")
        check(mm.mmtrain_attn_fwd(desc, batch, qkv, o, lse, ws, n), "mmtrain_attn_fwd")
        check(mm.mmtrain_attn_bwd(desc, batch, qkv, o, lse, d_o, d_qkv, ws, n), "mmtrain_attn_bwd")
        torch.cuda.synchronize()
        return o, lse, d_qkv

    other = mm.MASK_BIDIR if mode == mm.MASK_CAUSAL else mm.MASK_CAUSAL                  # ignored where there is an array
    spelled_out = run(mm.PackedBatch.on_device(cu, np.full(segments, mode, dtype=np.uint8), other))
    for a, b in zip(run(mm.PackedBatch.on_device(cu, None, mode)), spelled_out):
        assert torch.equal(a, b)
