"""fp32 layers whose products do the elementwise work behind them (rotary embedding, SwiGLU and its gradient) and whose weight gradients take the
gain and bias sums along: edges of the 32 x 32 and 64 x 64 tiles, half a tile of columns from either side of a pair.  Against the fp64 oracle."""
import numpy as np
import pytest

from oracle import layer_oracle as orc
from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import parity
from paper_2408_04275_amd import workloads as wl
from paper_2408_04275_amd.harness import LayerRunner
from test_gpu_ops import attn_case

pytestmark = pytest.mark.gpu


# one token; grouped heads of 64 and 128; one and several half tiles of the gate; 64 x 64 tiles (612 of QKV, 833 of the gate and up, 425 of their gradient)
# with a remainder of 16 columns and of 16 rows; the encoder, whose products have no such work but take the sums along
@pytest.mark.parametrize("kind,H,nh,nkv,d,F,lens", [
    (wl.DECODER, 64, 1, 1, 64, 16, [1]), (wl.DECODER, 80, 2, 1, 64, 48, [1, 32]), (wl.DECODER, 128, 4, 2, 128, 272, [5, 60, 1, 31]),
    (wl.DECODER, 512, 12, 12, 64, 1552, [300, 1, 739]), (wl.ENCODER, 96, 2, 2, 64, 48, [33, 2])])
def test_f32_layers_with_fused_launches(kind, H, nh, nkv, d, F, lens):
    T = sum(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    modes = np.array([(i % 2 if kind == wl.DECODER else 1) for i in range(len(lens))], dtype=np.uint8)
    shape = wl.LayerShape("fused", kind, wl.F32, H, nh, nkv, d, F, T)
    W = wl.make_weights(shape, 3, std=0.05)
    x, dy = wl.make_activations(shape, T, 3)
    y, cache = orc.layer_fwd(kind, nh, nkv, d, cu, modes, W, x)
    dx, G = orc.layer_bwd(W, cache, dy)
    r = LayerRunner(shape, W, cu, modes)
    r.set_inputs(x, dy)
    for _ in range(2):                                                  # the second pass overwrites the first one's outputs
        r.step()
    gy, gdx, gG = r.results()
    parity.check("y", gy, y, wl.F32)
    parity.check("dx", gdx, dx, wl.F32)
    for k in G:
        parity.check("d" + k, gG[k], G[k], wl.F32)


# many workgroups of 64-wide heads: a dQ and a dK/dV launch
def test_f32_attention_with_many_heads():
    attn_case(mm.F32, 40000, 40000, 64, np.array([0, 5, 9], dtype=np.int32), np.array([0, 1], dtype=np.uint8), seed=34)


# dQ and dK/dV rows of workgroups together beyond what one grid holds
def test_f32_attention_backward_beyond_one_grid():
    attn_case(mm.F32, 40000, 40000, 128, np.array([0, 1, 2], dtype=np.int32), np.array([0, 1], dtype=np.uint8), seed=36)


# one launch for both and one each, at the line between them (448 workgroups of dK/dV) and past it, grouped heads too
@pytest.mark.parametrize("nh,nkv,T", [(32, 32, 224), (32, 32, 225), (28, 14, 512), (28, 14, 513), (4, 1, 97)])
def test_f32_attention_backward_together_and_apart(nh, nkv, T):
    attn_case(mm.F32, nh, nkv, 64, np.array([0, T // 3, T // 3 + 1, T], dtype=np.int32), np.array([0, 1, 0], dtype=np.uint8), seed=35)
