"""The order of the samples: by pairs (small calls) and by counts, records read
through the order.  ln L of a sample does not depend on the samples around
it, so a call must return exactly the values of the same samples in calls of
other sizes, on both sides of the change of path and with every workgroup edge
(64 and 1024 samples), for draws spread over the prior, for a few distinct
samples repeated (one bucket holds a whole workgroup) and with invalid ones,
which become NaN and sort last."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth

pytestmark = pytest.mark.gpu

N = 20000


def _samples(kind, n_det):
    s, _ = synth.prior_samples(N, 17 + n_det)
    if kind == "few":
        s = np.ascontiguousarray(s[:, np.arange(N) % 3])
    if kind == "invalid":
        s[5, np.arange(N) % 7 == 2] = -1.0
    return s


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["spread", "few", "invalid"])
@pytest.mark.parametrize("n_det", [1, 2, 3])
def test_order_does_not_change_values(n_det, kind, precision):
    import torch
    inst = synth.make_instance(["D1", "D2", "D3"][:n_det], 3, 4096, 4096.0, 65, 5 + n_det)
    s = _samples(kind, n_det)
    bad = s[5] < 0
    with ile.Context(inst, precision=precision) as ctx:
        def run(n):
            d = torch.from_numpy(np.ascontiguousarray(s[:, :n])).cuda()
            out = torch.full((n,), 7.0, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            ctx.eval_dev(d, n, out)
            if bad[:n].any():
                with pytest.raises(ile.IleError):
                    ctx.sync()
            torch.cuda.synchronize()
            return out.cpu().numpy()
        want = run(N)
        assert np.array_equal(np.isnan(want), bad)
        for n in (1, 2, 63, 64, 65, 1000, 1024, 1025, 8191, 8192, 8193, 16384, 16385):
            assert np.array_equal(run(n), want[:n], equal_nan=True), n
