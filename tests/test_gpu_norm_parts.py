"""Decoder layers of short packs: the input gradient in front of the second normalisation is cut along K as a whole, and the normalisation's backward
kernel adds up its parts, in rows of up to 4096; wider ones (4112) keep a kernel that sums them.  One and several rows per workgroup, both widths
the kernel is built for, whole and partly filled batches of parts."""
import numpy as np
import pytest

from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import workloads as wl
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
