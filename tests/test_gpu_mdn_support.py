"""The learned proposal's density outside its support: a point that any
dimension's transform does not reach (u outside (0, 1)) has ln q = -inf and
carries no weight in the gradient, whatever the other dimensions hold: a
declination past the poles, an infinity, a NaN."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth

pytestmark = pytest.mark.gpu

# (dimension, value) outside; what another dimension holds beside it
OUTSIDE = [(5, 5.0), (5, 1000.0), (5, np.nan), (4, 1.0), (4, -1.5), (6, 0.02), (0, np.nan),
           (3, np.inf)]
BESIDE = [None, (1, 2.0), (1, -2.5), (1, 4.0)]


def _prop():
    p = ile.Proposal(seed=3)
    p.set_params(synth.mdn_params(21, gain=1.0))
    return p


@pytest.mark.parametrize("n", [1, 37])
@pytest.mark.parametrize("beside", BESIDE)
def test_outside_is_minus_infinity(beside, n):
    import torch
    x, _ = synth.prior_samples(n * len(OUTSIDE), 71)
    for j, (d, v) in enumerate(OUTSIDE):
        x[d, j * n:(j + 1) * n] = v
    if beside:
        x[beside[0]] = beside[1]
    m = x.shape[1]
    with _prop() as p:
        xd = torch.tensor(x).cuda()
        lq = torch.zeros(m, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        p.logpdf_dev(xd, m, m, lq)
        p.sync()
        assert np.all(lq.cpu().numpy() == -np.inf)


def test_outside_carries_no_weight():
    """Gradient and loss of a batch with such points against the batch without
    them: the same samples in the same workgroups, their weight zero there."""
    import torch
    n = 200
    x, _ = synth.prior_samples(n, 72)
    w = np.random.default_rng(4).uniform(0.1, 1.0, n)
    bad = np.arange(n) % 7 == 2
    xb = x.copy()
    xb[1, bad] = 2.0
    xb[5, bad] = 5.0
    with _prop() as p:
        def grad(a, wt):
            g = torch.zeros(ile.PROP_NPARAM, dtype=torch.float32, device="cuda")
            A, W = torch.tensor(a).cuda(), torch.tensor(wt).cuda()
            torch.cuda.synchronize()
            loss = p.grad_dev(A, n, n, W, g)
            return loss, g.cpu().numpy()
        l0, g0 = grad(xb, w)
        l1, g1 = grad(xb, np.where(bad, 0.0, w))
    assert np.isfinite(l1) and l0 == l1
    assert np.all(np.isfinite(g1)) and np.array_equal(g0, g1)
