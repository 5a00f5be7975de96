"""A call of attention alone finds segments by itself up to 64 of them, one per lane of a wavefront, and through a table of tokens beyond: either side
of that line, with empty segments at both ends, next to each other and on tile edges, and one mask mode for all."""
import numpy as np
import pytest

from paper_2408_04275_amd import binding as mm
from test_gpu_ops import attn_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nh,nkv,d", [(3, 3, 64), (4, 1, 128), (2, 2, 80)])
@pytest.mark.parametrize("segments", [2, 63, 64, 65, 130])
def test_either_side_of_the_line(nh, nkv, d, segments):
    rng = np.random.default_rng(segments)
    cuts = np.sort(rng.integers(0, 700, segments - 1))
    cuts[: segments // 8] = 0
    cuts[segments // 2: segments // 2 + segments // 8] = 256
    cuts[segments - 1 - segments // 8:] = 700
    cu = np.concatenate([[0], np.sort(cuts), [700]]).astype(np.int32)
    attn_case(mm.BF16, nh, nkv, d, cu, rng.integers(0, 2, segments).astype(np.uint8), seed=58)
