"""With 256 queries per workgroup the forward kernel computes scores one block of 32 keys ahead: packs whose wavefronts begin at the first, at an odd and
at a later even block of their workgroup's keys and end in either half of a step, and scores that leave the first blocks' maxima far behind; the
other two workgroup forms beside it."""
import numpy as np
import pytest
import torch

from oracle import bf16_storage, layer_oracle as orc
from paper_2408_04275_amd import binding as mm, parity, workloads as wl
from test_gpu_ops import assert_parity, check, to_device, to_host

pytestmark = pytest.mark.gpu

# starts of segments at 37, 75 and 613: within the first step of a workgroup's keys, in its second block, and 18 and 19 blocks behind the first key
PACKS = [([0, 37, 75, 613, 1100], [0, 1, 0, 1]), ([0, 545, 1100], [1, 0])]
LONG = [([0, 37, 1100], [0, 1]), ([0, 1090, 1155, 2200], [1, 0, 1]), ([0, 1191, 2200], [1, 1])]
# 128-query workgroups: 3 heads of 1100 tokens take two groups of wavefronts, 57 one; 104 heads, or 57 of 2200 tokens, and at least 15 steps per
# tile of 256 queries: 256
FORMS = [(3, 1, 128, *p) for p in PACKS] + [(57, 19, 64, *p) for p in PACKS] + [(104, 8, 128, *LONG[0])] + \
        [(57, 3, d, *p) for d in (80, 96, 128) for p in LONG[1:]]


# standard deviation of q, k, v: the scores' is its square, 25 in units of e moves the reference several times per row.  The bar is the
# operator tests': what rounding probabilities and output to bf16 costs this very case, in the oracle
@pytest.mark.parametrize("std", [1.0, 5.0])
@pytest.mark.parametrize("nh,nkv,d,cu,modes", FORMS)
def test_first_and_last_blocks(nh, nkv, d, cu, modes, std):
    cu, modes, T = np.array(cu, dtype=np.int32), np.array(modes, dtype=np.uint8), cu[-1]
    qkv = wl.round_to(np.random.default_rng(56).standard_normal((T, (nh + 2 * nkv) * d)) * std, mm.BF16)
    q, k, v = (a.reshape(T, -1, d).astype(np.float64) for a in np.split(qkv, [nh * d, (nh + nkv) * d], axis=1))
    ref, lse_ref = orc.attention_fwd(q, k, v, cu, modes, 1 / np.sqrt(d))
    floor = parity.errors(bf16_storage.bf16_round(bf16_storage.attention_fwd_rounded(q, k, v, cu, modes, 1 / np.sqrt(d))), ref)
    n = mm.mmtrain_attn_workspace_bytes(T, len(modes), nh)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    o = torch.zeros((T, nh * d), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((nh, T), dtype=torch.float32, device="cuda")
    check(mm.mmtrain_attn_fwd(mm.make_desc(mm.DECODER, mm.BF16, 64, nh, nkv, d, 64), mm.PackedBatch.on_device(cu, modes),
                              to_device(qkv, mm.BF16), o, lse, ws, n), "mmtrain_attn_fwd")
    torch.cuda.synchronize()
    assert_parity("o", to_host(o), ref.reshape(T, nh * d), mm.BF16, floor=floor)
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref)) < 2e-2
