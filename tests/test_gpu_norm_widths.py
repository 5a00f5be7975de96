"""Normalisation, GELU and column-sum kernels at the widths and pack lengths where their forms change: rows up to 512, 1024, 1536 and
2048 wide take a wavefront each (forward; backward up to 1024), slabs of 4, 8 and 16 rows by pack length."""
import numpy as np
import pytest

from paper_2408_04275_amd import workloads as wl
from util import compare_layer, gpu_run, oracle_run, storage_floors

pytestmark = pytest.mark.gpu


def run(kind, dtype, H, T, seed):
    shape = wl.LayerShape("norm-widths", kind, dtype, H, 2, 2, 64, 48, T)
    cuts = np.arange(0, T, 97)[1:]
    cu = np.concatenate([[0], cuts, [T]]).astype(np.int32)
    modes = np.ones(len(cu) - 1, dtype=np.uint8)
    # the workloads' own weight scale: at 0.05 the rounding of stored tensors alone reaches max_err 2.7e-2 on dx at H = 1536,
    # above the fixed bar of 2e-2 that no test widens
    W = wl.make_weights(shape, seed, std=0.02)
    x, dy = wl.make_activations(shape, T, seed)
    ref = oracle_run(shape, cu, modes, W, x, dy)
    floors = storage_floors(shape, cu, modes, W, x, dy, ref)
    # floor_err is the largest of n errors: near-Gaussian ones of standard deviation l2_err (relative to the tensor's rms) reach 5 of
    # these with a probability of 6e-7 n, but one sample of the floor may be as low as 2.4 on a small tensor (the 128 elements of
    # dnorm2_b at 3073 tokens: 7.6e-3 at an l2_err of 3.1e-3, where ten seeds average 9.4e-3), so there it does not bound another
    # rounding by itself.  From 4096 elements on the largest lies between 3.2 and 4.5 deviations, and 1.5 times that does.
    for k, f in (floors or {}).items():
        n = T * H if k in ("y", "dx") else W[k].size
        if n < 4096:
            f["floor_err"] = max(f["floor_err"], 5. / 1.5 * f["l2_err"])
    compare_layer(shape, gpu_run(shape, cu, modes, W, x, dy), ref, floors=floors)


@pytest.mark.parametrize("kind", [wl.ENCODER, wl.DECODER])
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("H", [16, 512, 528, 1024, 1040, 1536, 1552, 2048, 2064])
def test_row_width(kind, dtype, H):
    run(kind, dtype, H, 67, seed=61)


@pytest.mark.parametrize("T", [1, 5, 2049, 3073, 6145])
def test_pack_length(T):
    run(wl.ENCODER, wl.BF16, 128, T, seed=62)
