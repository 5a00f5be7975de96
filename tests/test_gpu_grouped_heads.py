"""Attention backward with a group's query heads shared out over several workgroups: every share count the rule can give, head
widths that are not native, and the same call with a workspace that has no room for partial sums."""
import numpy as np
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import workloads as wl
from paper_2408_04275_amd.harness import check, to_device
from test_gpu_ops import attn_case

pytestmark = pytest.mark.gpu

LENS = [1, 70, 129, 64, 7, 200, 31]
CU = np.concatenate([[0], np.cumsum(LENS)]).astype(np.int32)
MODES = np.array([0, 1, 0, 1, 1, 0, 0], dtype=np.uint8)


@pytest.mark.parametrize("nh,nkv,d", [(8, 1, 128), (6, 2, 128), (7, 1, 64), (6, 1, 80), (4, 2, 48), (16, 16, 64), (32, 16, 128)])
def test_shared_query_heads(nh, nkv, d):
    attn_case(mm.BF16, nh, nkv, d, CU, MODES, seed=41)


def test_without_room_for_partial_sums():
    nh, nkv, d, T, S = 8, 2, 128, int(CU[-1]), len(LENS)
    rng = np.random.default_rng(42)
    qkv = to_device(wl.round_to(rng.standard_normal((T, (nh + 2 * nkv) * d)), mm.BF16), mm.BF16)
    d_o = to_device(wl.round_to(rng.standard_normal((T, nh * d)), mm.BF16), mm.BF16)
    desc, batch = mm.make_desc(mm.DECODER, mm.BF16, 64, nh, nkv, d, 64), mm.PackedBatch.on_device(CU, MODES)
    full = mm.mmtrain_attn_workspace_bytes(T, S, nh)
    tables = T * 4 + T * 8 + T * nh * 4 + 4 * 256                     # token tables and row sums, rounded up
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    o, lse = torch.empty_like(d_o), torch.empty((nh, T), dtype=torch.float32, device="cuda")
    check(mm.mmtrain_attn_fwd(desc, batch, qkv, o, lse, ws, tables), "mmtrain_attn_fwd")
    got = []
    for nbytes in (full, tables):
        d_qkv = torch.full_like(qkv, float("nan"))
        check(mm.mmtrain_attn_bwd(desc, batch, qkv, o, lse, d_o, d_qkv, ws, nbytes), "mmtrain_attn_bwd")
        got.append(d_qkv.float())
    nq = nh * d
    assert torch.equal(got[0][:, :nq], got[1][:, :nq])
    # dK, dV: fp32 sums in another order, one bf16 rounding each: a value may move by one unit in the last place (2^-8 of its size)
    diff, scale = (got[0] - got[1]).abs(), got[1].abs().clamp_min(1e-3 * got[1].abs().max())
    assert (diff / scale).max().item() <= 2.0 ** -7 and not torch.isnan(diff).any()
    assert mm.mmtrain_attn_bwd(desc, batch, qkv, o, lse, d_o, d_qkv, ws, T * nh * 4) == mm.ERR_WORKSPACE
