"""The forms of the attention kernels: 256 queries per workgroup where many workgroups walk many keys (heads wider than 64 features), 128
on short packs, and there two groups of wavefronts that share the steps up to 512 workgroups; either side of the lines, ragged ends."""
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


# 1100 tokens: 9 tiles of 128; 57 heads make 513 workgroups, 56 make 504 (two groups of wavefronts, an even and an odd number of steps)
@pytest.mark.parametrize("nh,nkv,d", [(57, 57, 64), (56, 56, 64), (56, 7, 64), (57, 19, 48), (56, 28, 80), (56, 56, 96), (56, 8, 128)])
@pytest.mark.parametrize("cu,modes", [([0, 1, 66, 1100], [0, 1, 0]), ([0, 600, 728, 1100], [1, 0, 1])])
def test_workgroups_of_two_groups(nh, nkv, d, cu, modes):
    attn_case(mm.BF16, nh, nkv, d, np.array(cu, dtype=np.int32), np.array(modes, dtype=np.uint8), seed=53)


# dK/dV with two wavefronts per 32 keys: 1, 2, 3, 4 and 7 tiles of 64 queries per head (three slots, one block behind); a first segment of
# 33 tokens makes wavefronts skip single blocks of 32.  One head, or three and four of a group: one per workgroup, and all of them in one
# workgroup, which then changes head every 1 to 7 tiles while its copies are two tiles ahead
@pytest.mark.parametrize("nh,d,share_heads", [(1, 128, True), (3, 128, True), (3, 80, True), (1, 96, True), (3, 128, False), (4, 128, False), (3, 80, False), (4, 96, False)])
@pytest.mark.parametrize("T", [59, 123, 187, 251, 443])
def test_key_gradients_of_few_steps(nh, d, share_heads, T):
    attn_case(mm.BF16, nh, 1, d, np.array([0, T], dtype=np.int32), np.array([1], dtype=np.uint8), seed=54, share_heads=share_heads)
    attn_case(mm.BF16, nh, 1, d, np.array([0, 33, T], dtype=np.int32), np.array([0, 0], dtype=np.uint8), seed=55, share_heads=share_heads)
