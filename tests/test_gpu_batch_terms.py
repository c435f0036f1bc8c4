"""The phased engine's two forms of the per-sample terms in a batch, from a
kernel of their own and in the tiles (terms limit 0): each against the FP64
oracle with the parity tests' tolerances, over points of mixed shape, windows
before and after a chunk's last bin, a last tile with empty slots, and draws
outside the prior, whose values are NaN in both."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth
from test_gpu_parity import check_margT

pytestmark = pytest.mark.gpu

SITES = ["D1", "D2", "D3"]
SHAPES = [(1, 1, 33), (2, 3, 47), (3, 4, 301), (3, 9, 463), (3, 21, 465), (2, 21, 929), (3, 13, 1103)]


def _points():
    out = [synth.make_instance(SITES[:nd], nl, 16384, 16384.0, nt, 31 * nt + nl)
           for nd, nl, nt in SHAPES]
    four = synth.make_instance(SITES, 5, 16384, 16384.0, 161, 77)
    four.dets = four.dets + [(-32.0, 116.0, 20.0)]   # a fourth site with the first one's series
    four.Q, four.U, four.V = (np.concatenate([a, a[:1]]) for a in (four.Q, four.U, four.V))
    return out + [four]


@pytest.mark.parametrize("threads", [512, 256])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [1, 37, 203])
def test_both_forms_match_the_oracle(n, precision, threads):
    import torch
    from oracle import oracle as O
    pts = _points()
    S = np.stack([synth.prior_samples(n, 7 * n + p)[0] for p in range(len(pts))])
    d = torch.tensor(S).cuda()
    torch.cuda.synchronize()
    tol = dict(tol=1e-9) if precision == "fp64" else dict(tol=1e-4, rel=True)
    octx = [O.Ctx(p) for p in pts]
    want = [c.eval(s) for c, s in zip(octx, S)]
    with ile.Batch(precision) as b:
        for p in pts:
            b.add_point(p)
        b.set_tuning(threads=threads, wgs_per_cu=2, order=0, engine=1)
        for limit in (0, 1 << 30, 0):
            b.set_terms_limit(limit)
            print(f"n {n} {precision} threads {threads} limit {limit}", flush=True)
            res = b.run_dev(n, d)
            got = b.lnL(n)
            for p, inst in enumerate(pts):
                check_margT(got[p], want[p], S[p], octx[p], inst, **tol)
                ref = O.integrate(got[p], np.zeros(n), np.zeros(n))
                assert abs(res[p]["ln_L_marg"] - ref["ln_L_marg"]) <= 1e-9


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_invalid_draws_in_both_forms(precision):
    import torch
    pts, n = _points()[2:5], 100
    S = np.stack([synth.prior_samples(n, 5 + p)[0] for p in range(len(pts))])
    bad = np.arange(n) % 5 == 3
    bad[16:32] = True   # a tile of none but invalid samples is possible
    T = S.copy()
    T[:, 5, bad] = -1.0
    with ile.Batch(precision) as b:
        for p in pts:
            b.add_point(p)
        out = []
        for limit in (1 << 30, 0):
            b.set_terms_limit(limit)
            d, e = torch.tensor(S).cuda(), torch.tensor(T).cuda()
            torch.cuda.synchronize()
            b.run_dev(n, d)
            good = b.lnL(n)
            with pytest.raises(ile.IleError, match="outside the prior"):
                b.run_dev(n, e)
            got = b.lnL(n)
            assert np.all(np.isnan(got[:, bad])) and np.all(np.isfinite(got[:, ~bad]))
            out.append((good, got))
    scale = np.maximum(1.0, np.abs(out[0][0]))
    tol = 1e-9 if precision == "fp64" else 1e-4
    for a, c in zip(out[0], out[1]):
        assert np.nanmax(np.abs(a - c) / scale) <= tol


def test_limit_is_checked():
    with ile.Batch("fp64") as b:
        with pytest.raises(ile.IleError):
            b.set_terms_limit(-1)
