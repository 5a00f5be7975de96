"""Weight gradients written and added as fp32 (bf16 operands), at the edges of their tiles: widths 16 past a tile,
few and many tiles, and enough of them that workgroups take several in turn and every second one starts later.  The sums are the
same whatever they are written as, so nothing here needs a tolerance: rounding the fp32 result gives the bf16 run's bits, and adding
it to previous contents is one fp32 addition per element."""
import numpy as np
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import workloads as wl
from paper_2408_04275_amd.harness import LayerRunner, check

pytestmark = pytest.mark.gpu

# hidden, heads, head width, feed-forward width, tokens
SHAPES = [(80, 1, 64, 144, 67), (272, 4, 64, 528, 300), (1296, 10, 128, 2576, 131), (2064, 16, 128, 8208, 70)]
# the same with more tokens than the K loop looks ahead, and the tiles that the gradients of the two feed-forward weights take
LONGER = [(2064, 4, 128, 5520, 777, "256x128", "256x256"), (2064, 16, 128, 8208, 450, "256x256", "256x128")]


@pytest.mark.parametrize("H,nh,d,F,T", SHAPES + [s[:5] for s in LONGER])
def test_added_to_previous_contents(H, nh, d, F, T):
    shape = wl.LayerShape("f32g", wl.DECODER, wl.BF16, H, nh, nh, d, F, T)
    cu, modes = np.array([0, 9, T], dtype=np.int32), np.zeros(2, dtype=np.uint8)
    W = wl.make_weights(shape, 3, std=0.05)
    x, dy = wl.make_activations(shape, T, 3)
    runs = []
    for f32 in (False, True):
        r = LayerRunner(shape, W, cu, modes, grads_f32=f32)
        r.set_inputs(x, dy)
        check(r.forward(), "fwd")
        check(r.backward(mm.BWD_WGRAD_F32 if f32 else 0), "bwd")
        runs.append(r)
    torch.cuda.synchronize()
    once = {k: g.clone() for k, g in runs[1].g.items()}
    for k, g in once.items():
        assert torch.equal(g.bfloat16(), runs[0].g[k]), k
    gen = torch.Generator(device="cuda").manual_seed(5)
    before = {k: torch.randn(g.shape, generator=gen, device="cuda") for k, g in once.items()}
    for k, g in runs[1].g.items():
        g.copy_(before[k])
    check(runs[1].backward(mm.BWD_WGRAD_F32 | mm.BWD_ACCUMULATE_WGRAD), "bwd, added")
    torch.cuda.synchronize()
    for k, g in runs[1].g.items():
        assert torch.equal(g, before[k] + once[k]), k


def test_rows_of_more_than_2_21_elements():
    # the gradient of the second feed-forward weight: rows of 8 MiB, two tiles of them, ragged in both directions
    H, nh, d, F, T = 272, 4, 64, (1 << 21) + 16, 8
    desc = mm.make_desc(mm.DECODER, mm.BF16, H, nh, nh, d, F)
    batch = mm.PackedBatch.on_device(np.array([0, T], dtype=np.int32), np.zeros(1, dtype=np.uint8))
    gen = torch.Generator(device="cuda").manual_seed(6)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    w = {"norm1_w": rand(H), "w_qkv": rand(3 * nh * d, H) * 0.05, "w_o": rand(H, nh * d) * 0.05, "norm2_w": rand(H),
         "w_fc1": rand(2 * F, H) * 0.05, "w_fc2": rand(H, F) * 0.001}
    x, dy = rand(T, H), rand(T, H)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    nbytes = max(mm.mmtrain_layer_workspace_bytes(desc, T, 1, b) for b in (0, 1))
    ws, ctx = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (nbytes, mm.mmtrain_layer_ctx_bytes(desc, T)))
    weights = mm.make_weights(w)
    check(mm.mmtrain_layer_fwd(desc, batch, weights, x, y, ctx, ws, nbytes), "fwd")
    before = torch.randn((H, F), generator=gen, device="cuda")
    g = [torch.empty((H, F), dtype=torch.bfloat16, device="cuda"), torch.empty_like(before), before.clone()]
    for out, flags in zip(g, (0, mm.BWD_WGRAD_F32, mm.BWD_WGRAD_F32 | mm.BWD_ACCUMULATE_WGRAD)):
        check(mm.mmtrain_layer_bwd(desc, batch, weights, x, dy, ctx, dx, mm.make_grads({"w_fc2": out}), flags, ws, nbytes), "bwd")
    torch.cuda.synchronize()
    assert g[1].abs().max() > 0 and torch.equal(g[1].bfloat16(), g[0])
    assert torch.equal(g[2], before + g[1])
