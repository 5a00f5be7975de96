"""The two forms of the forward and dQ kernels for heads wider than 64 features: 128 queries per workgroup on short packs, 256 where
many workgroups walk many keys, either side of the line and with ragged ends."""
import numpy as np
import pytest

from paper_2408_04275_amd import binding as mm
from test_gpu_ops import attn_case

pytestmark = pytest.mark.gpu


# 1100 bidirectional tokens: 5 query tiles of 18 steps of 64 keys; 104 heads make 520 workgroups of 256 queries, 100 make 500
@pytest.mark.parametrize("nh,nkv,d", [(104, 8, 128), (104, 4, 80), (100, 4, 96)])
def test_long_rows_many_heads(nh, nkv, d):
    attn_case(mm.BF16, nh, nkv, d, np.array([0, 1100], dtype=np.int32), np.array([1], dtype=np.uint8), seed=51)


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("T", [1, 127, 129, 257, 383])
def test_ends_of_128_query_workgroups(d, T):
    cut = T // 3
    attn_case(mm.BF16, 3, 3, d, np.array([0, cut, T], dtype=np.int32), np.array([0, 1], dtype=np.uint8), seed=52)
