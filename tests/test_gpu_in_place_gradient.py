"""Backward with dx written over dy: every gradient, the fc2 weight gradient (which reads dy) among them, is what separate buffers
give, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import workloads as wl
from paper_2408_04275_amd.harness import LayerRunner, check

pytestmark = pytest.mark.gpu


# narrow layers, whose weight gradients run together at the end of the pass
@pytest.mark.parametrize("kind,dtype", [(wl.DECODER, wl.F32), (wl.ENCODER, wl.F32), (wl.DECODER, wl.BF16), (wl.ENCODER, wl.BF16)])
@pytest.mark.parametrize("stack", [False, True])
def test_dx_over_dy(kind, dtype, stack):
    shape = wl.LayerShape("in-place", kind, dtype, 128, 2, 2, 64, 208, 300)
    cu, modes = np.array([0, 7, 180, 300], dtype=np.int32), np.ones(3, dtype=np.uint8)
    r = LayerRunner(shape, wl.make_weights(shape, 3), cu, modes)
    r.set_inputs(*wl.make_activations(shape, 300, 3))

    def backward(dx):
        if stack:                                   # one layer: dy and dx of the stack are the layer's
            n = mm.mmtrain_stack_workspace_bytes(r.desc, 1, r.T, 3, 1, 0)
            ws = torch.empty(n, dtype=torch.uint8, device="cuda")
            check(mm.mmtrain_stack_bwd(r.desc, 1, r.batch, [r.weights], r.x, r.dy, r.ctx, dx, [r.grads], 0, ws, n), "mmtrain_stack_bwd")
        else:
            check(mm.mmtrain_layer_bwd(r.desc, r.batch, r.weights, r.x, r.dy, r.ctx, dx, r.grads, 0, r.ws, r.ws_bytes), "mmtrain_layer_bwd")
        torch.cuda.synchronize()
        return dx.clone(), {k: g.clone() for k, g in r.g.items()}

    check(r.forward(), "mmtrain_layer_fwd")
    dx, g = backward(r.dx)
    dx_over, g_over = backward(r.dy)
    assert torch.equal(dx, dx_over)
    for k in g:
        assert torch.equal(g[k], g_over[k]), k
