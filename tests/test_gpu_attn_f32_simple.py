"""fp32 attention on the vector ALUs: what packs beyond the matrix-instruction kernels' limits take.  Those limits are 4 GB of q, k, v
or more than 65535 heads; the second is the one a small test can reach."""
import numpy as np
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd.harness import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nh,nkv,d,cu,modes", [(65536, 16384, 64, [0, 1, 6, 12], [0, 1, 0]), (65540, 65540, 64, [0, 5, 5, 9], [1, 0, 0]),
                                               (65536, 32768, 128, [0, 2, 7], [0, 1])])
def test_more_heads_than_a_grid_row(nh, nkv, d, cu, modes):
    T, S, scale = cu[-1], len(cu) - 1, d ** -0.5
    gen = torch.Generator(device="cuda").manual_seed(T)
    qkv = torch.randn((T, (nh + 2 * nkv) * d), generator=gen, device="cuda")
    d_o = torch.randn((T, nh * d), generator=gen, device="cuda")
    desc = mm.make_desc(mm.DECODER, mm.F32, 64, nh, nkv, d, 64)
    batch = mm.PackedBatch.on_device(np.array(cu, dtype=np.int32), np.array(modes, dtype=np.uint8))
    wsb = mm.mmtrain_attn_workspace_bytes(T, S, nh)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    o, lse, d_qkv = torch.full_like(d_o, float("nan")), torch.empty((nh, T), device="cuda"), torch.full_like(qkv, float("nan"))
    check(mm.mmtrain_attn_fwd(desc, batch, qkv, o, lse, ws, wsb), "mmtrain_attn_fwd")
    check(mm.mmtrain_attn_bwd(desc, batch, qkv, o, lse, d_o, d_qkv, ws, wsb), "mmtrain_attn_bwd")
    group = nh // nkv
    # a dozen key/value heads from all over the range, in float64: [head, token, feature]
    heads = [0, 1, 2, nkv // 3, nkv // 2, nkv - 2, nkv - 1]

    def cols(t, n, at):                             # columns `at` heads onwards of a [T, heads x d] tensor
        return torch.stack([t[:, (at + h) * d:(at + h + 1) * d] for h in n]).double().cpu()

    qh = [g * group + j for g in heads for j in range(group)]
    q, k, v, go = cols(qkv, qh, 0), cols(qkv, heads, nh), cols(qkv, heads, nh + nkv), cols(d_o, qh, 0)
    k, v = k.repeat_interleave(group, 0), v.repeat_interleave(group, 0)
    seg = np.repeat(np.arange(S), np.diff(cu))
    i, j = np.arange(T)[:, None], np.arange(T)[None, :]
    seen = torch.from_numpy((seg[:, None] == seg[None, :]) & ((np.array(modes)[seg][:, None] == 1) | (j <= i)))
    s = (q @ k.transpose(1, 2) * scale).masked_fill(~seen, -torch.inf)
    ref_lse = torch.logsumexp(s, 2)
    p = torch.exp(s - ref_lse[:, :, None])
    ref_o = p @ v
    ds = p * (go @ v.transpose(1, 2) - (go * ref_o).sum(2, keepdim=True)) * scale
    ref = {"o": ref_o, "lse": ref_lse, "dq": ds @ k, "dk": (ds.transpose(1, 2) @ q).reshape(len(heads), group, T, d).sum(1),
           "dv": (p.transpose(1, 2) @ go).reshape(len(heads), group, T, d).sum(1)}
    got = {"o": cols(o, qh, 0), "lse": lse[qh].double().cpu(), "dq": cols(d_qkv, qh, 0), "dk": cols(d_qkv, heads, nh), "dv": cols(d_qkv, heads, nh + nkv)}
    for name in ref:
        # fp32 sums of at most 128 features and 12 x group rows, an exponential and a division: a few hundred roundings of 6e-8
        assert (got[name] - ref[name]).abs().max() <= 2e-5 * ref[name].abs().max(), name
    assert not torch.isnan(o).any() and not torch.isnan(d_qkv).any()           # every head was written
