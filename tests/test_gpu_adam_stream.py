"""The optimizer step on shards on both sides of the line from which it streams (360 MiB in all), with remainders, against the fp64
oracle."""
import numpy as np
import pytest
import torch

from oracle import adam_oracle as ao
from paper_2408_04275_amd import binding as mm
from paper_2408_04275_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(12 << 20) + 1027, (12 << 20) + 2048, (20 << 20) + 1027, (20 << 20) + 2048])
@pytest.mark.parametrize("param_dtype", [mm.BF16, mm.F32])
def test_large_shard(n, param_dtype):
    rng = np.random.default_rng(n)
    w, g = (rng.standard_normal(n, dtype=np.float32) for _ in range(2))
    m, v = rng.standard_normal(n, dtype=np.float32) * np.float32(0.1), rng.random(n, dtype=np.float32) * np.float32(0.01)
    dw, dg, dm, dv = (torch.from_numpy(a.copy()).cuda() for a in (w, g, m, v))
    out = torch.full((n + 8,), 7.0, device="cuda", dtype=torch.bfloat16 if param_dtype == mm.BF16 else torch.float32)
    desc = mm.make_adam_desc(2e-3, 0.9, 0.999, 1e-8, 0.1, 0.5, 3, zero_grad=True)
    assert mm.mmtrain_adam_step(desc, n, dw, dg, dm, dv, out, param_dtype) == mm.OK
    lr, b1, b2, eps, wd, gs = (float(np.float32(x)) for x in (2e-3, 0.9, 0.999, 1e-8, 0.1, 0.5))
    rw, rm, rv = ao.adam_step(w.astype(np.float64), g, m.astype(np.float64), v.astype(np.float64), lr, b1, b2, eps, wd, gs, 3)
    got = dw.cpu().numpy()
    # fp32 arithmetic against fp64: a few ulp on w, m, v
    assert np.allclose(got, rw, rtol=4e-6, atol=2e-6)
    assert np.allclose(dm.cpu().numpy(), rm, rtol=2e-6, atol=1e-6 * np.abs(rm).max())
    assert np.allclose(dv.cpu().numpy(), rv, rtol=2e-6, atol=1e-6 * np.abs(rv).max())
    assert not dg.any().item()
    assert np.array_equal(out[:n].float().cpu().numpy(), wl.round_bf16(got) if param_dtype == mm.BF16 else got)
    assert bool((out[n:] == 7.0).all())                                # nothing beyond the shard is written
