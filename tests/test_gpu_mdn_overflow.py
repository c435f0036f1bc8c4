"""Draws of a network that gives NaN for some samples: finite parameters (which
set_params takes) that BF16 rounds to infinities, so that the layer-2 sum of a
last-degree unit is inf - inf where z~_0 > 0.  A sample's draw is a function of its seed and index alone, so
a call whose waves take several tiles in turn equals, bit for bit, calls whose
waves take one each; a NaN stays in its own sample."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth

pytestmark = pytest.mark.gpu


def _params():
    P = synth.mdn_params(21, gain=1.0).copy()
    W1, b1 = P[0:896].reshape(128, 7), P[896:1024]
    W2, b2 = P[1024:17408].reshape(128, 128), P[17408:17536]
    # units 0 .. 31 the sign of z~_0, units 32 .. 63 one; unit 5 (degree 5, which
    # only dimension 6 sees) adds the first and subtracts the second
    W1[:64] = 0.0
    W1[:32, 0] = 1e4
    b1[:32] = 0.0
    b1[32:64] = 1e4
    W2[5] = 0.0
    W2[5, :32] = np.finfo(np.float32).max
    W2[5, 32:64] = -np.finfo(np.float32).max
    b2[5] = 0.0
    return P


def test_a_nan_stays_in_its_sample():
    import torch
    n, part = 100_000, 4096   # 4096: 256 tiles, one a workgroup
    with ile.Proposal(seed=3) as p:
        p.set_params(_params())

        def draw(first, m):
            x = torch.zeros((7, m), dtype=torch.float64, device="cuda")
            lp, lq = (torch.zeros(m, dtype=torch.float64, device="cuda") for _ in range(2))
            torch.cuda.synchronize()
            p.sample_dev(11, first, m, x, m, lp, lq)
            p.sync()
            return torch.cat([x, lp[None], lq[None]]).cpu().numpy()
        whole = draw(0, n)
        parts = np.concatenate([draw(a, min(part, n - a)) for a in range(0, n, part)], axis=1)
    nan = np.isnan(parts[:7]).any(axis=0)
    assert 0.1 < nan.mean() < 0.9
    assert not np.isnan(parts[:6, ~nan]).any() and np.isfinite(parts[8, ~nan]).all()
    assert np.array_equal(whole, parts, equal_nan=True)
