"""The QKV bias gradient of an encoder, summed where the attention kernels store dQ, dK and dV (heads of up to 96 features; wider ones in a pass of
their own): ragged ends of 32 and 128 tokens, both workgroup forms, padded heads."""
import numpy as np
import pytest

from paper_2408_04275_amd import workloads as wl
from test_gpu_layer import run_case

pytestmark = pytest.mark.gpu


# 64 heads of 1100 tokens make 576 workgroups of 128 (one group of wavefronts each), the others two groups
@pytest.mark.parametrize("nh,d,T", [(4, 64, 31), (4, 64, 33), (64, 16, 1100), (4, 80, 129), (2, 96, 700), (2, 128, 300)])
def test_qkv_bias_gradient(nh, d, T):
    shape = wl.LayerShape("bias", wl.ENCODER, wl.BF16, 272, nh, nh, d, 528, T)
    cu = np.array([0, T // 3, T // 3 + 1, T], dtype=np.int32)
    run_case(shape, cu, np.ones(3, dtype=np.uint8), seed=61, std=0.05, what=f"bias {nh} x {d}, {T} tokens ")
