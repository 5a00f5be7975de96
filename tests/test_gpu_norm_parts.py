"""Decoder layers of short packs: the input gradient in front of the second normalisation is cut along K as a whole, and the normalisation's backward
kernel adds up its parts, in rows of up to 4096; wider ones (4112) keep a kernel that sums them.  One and several rows per workgroup, both widths
the kernel is built for, whole and partly filled batches of parts."""
import numpy as np
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import workloads as wl
from paper_2408_04275_amd.harness import LayerRunner, check
from util import compare_layer, gemm_route, gpu_run, oracle_run, say, storage_floors, summary

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,F,chunks", [(520, 4112, 6144, 5), (1031, 2048, 11008, 6), (40, 4096, 11008, 8)])
def test_parts_of_an_input_gradient(T, H, F, chunks):
    assert gemm_route(mm.GEMM_NN, T, H, 2 * F, 1 << 40)[3] == chunks
    cu, modes = np.array([0, T // 3, T], dtype=np.int32), np.array([0, 1], dtype=np.uint8)
    shape = wl.LayerShape("parts", wl.DECODER, wl.BF16, H, 2, 1, 64, F, T)
    W = wl.make_weights(shape, 5, std=0.02)
    x, dy = wl.make_activations(shape, T, 5)
    ref = oracle_run(shape, cu, modes, W, x, dy)
    floors = storage_floors(shape, cu, modes, W, x, dy, ref)
    what = f"parts T={T} H={H} F={F}: "
    errs = compare_layer(shape, gpu_run(shape, cu, modes, W, x, dy), ref, what, floors=floors)
    say(what + summary(errs, floors))


# parts in front of both normalisations; and a pack so long that the weight gradient behind the parts is cut along K too, in its last round, through the
# same scratch.  fp32 gradients added up twice, none at all, and dx over dy: the same sums, bit for bit.
@pytest.mark.parametrize("T,H,nh,nkv,d,F,qkv,fc1,tail", [(97, 2048, 64, 64, 128, 12288, 8, 8, 0), (4700, 1536, 2, 1, 64, 5632, 1, 2, 8)])
def test_parts_and_the_scratch_they_lie_in(T, H, nh, nkv, d, F, qkv, fc1, tail):
    room = 1 << 40
    assert gemm_route(mm.GEMM_NN, T, H, (nh + 2 * nkv) * d, room)[2:] == (0, qkv)
    assert gemm_route(mm.GEMM_NN, T, H, 2 * F, room)[2:] == (0, fc1)
    assert gemm_route(mm.GEMM_TN, 2 * F, H, T, room)[2] == tail
    cu, modes = np.array([0, T // 3, T // 3 + 1, T], dtype=np.int32), np.array([0, 1, 0], dtype=np.uint8)
    shape = wl.LayerShape("scratch", wl.DECODER, wl.BF16, H, nh, nkv, d, F, T)
    W = wl.make_weights(shape, 6, std=0.02)
    x, dy = wl.make_activations(shape, T, 6)
    ref = oracle_run(shape, cu, modes, W, x, dy)
    floors = storage_floors(shape, cu, modes, W, x, dy, ref, round_param_grads=False)
    what = f"scratch T={T} H={H}: "
    r = LayerRunner(shape, W, cu, modes, grads_f32=True)
    r.set_inputs(x, dy)
    r.step(mm.BWD_WGRAD_F32)
    say(what + summary(compare_layer(shape, r.results(), ref, what, floors=floors), floors))
    dx, grads = r.dx.clone(), {k: g.clone() for k, g in r.g.items()}
    check(r.backward(mm.BWD_WGRAD_F32 | mm.BWD_ACCUMULATE_WGRAD), "accumulate")
    torch.cuda.synchronize()
    assert torch.equal(r.dx, dx)
    for k, g in grads.items():
        assert torch.equal(r.g[k], 2 * g), k
    frozen = LayerRunner(shape, W, cu, modes, grad_names=[])
    frozen.set_inputs(x, dy)
    frozen.step()
    torch.cuda.synchronize()
    assert torch.equal(frozen.dx, dx)
    r.dx = r.dy
    check(r.backward(mm.BWD_WGRAD_F32), "dx over dy")
    torch.cuda.synchronize()
    assert torch.equal(r.dx, dx)
    for k, g in grads.items():
        assert torch.equal(r.g[k], g), k
