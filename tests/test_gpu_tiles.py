"""Phased tiles at their edges, against the FP64 oracle: one k-step and odd or
even numbers of them, one to four detectors, windows that end on, before and
after a chunk's last bin, chunks shorter than a tile, tiles whose window
starts spread wider than a chunk (few samples over the whole prior), and a
last tile with empty slots and invalid samples.  The tolerances are the
parity tests': 1e-9 absolute for FP64 and 1e-4 relative for FP32 (a bin's
2 n_lm n_det FP32 products lose at most a few 1e-6 of |ln L| here)."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth
from test_gpu_parity import check_margT

pytestmark = pytest.mark.gpu

SITES = ["D1", "D2", "D3"]


def _instance(n_det, n_lm, n_q, srate, n_t, seed):
    inst = synth.make_instance(SITES[:min(n_det, 3)], n_lm, n_q, srate, n_t, seed)
    if n_det == 4:   # a fourth site with the first one's series
        inst.dets = inst.dets + [(-32.0, 116.0, 20.0)]
        inst.Q = np.concatenate([inst.Q, inst.Q[:1]])
        inst.U = np.concatenate([inst.U, inst.U[:1]])
        inst.V = np.concatenate([inst.V, inst.V[:1]])
    return inst


# (n_det, n_lm, n_t, N): 36 KiB of LDS makes chunks of a few dozen bins
CASES = [(1, 1, 1, 1), (1, 1, 33, 17), (2, 2, 201, 16), (2, 3, 47, 31), (3, 4, 301, 100),
         (4, 5, 161, 65), (3, 9, 463, 50), (3, 21, 465, 33), (3, 13, 929, 40), (1, 21, 1601, 48)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lds_kb", [None, 36])
@pytest.mark.parametrize("n_det,n_lm,n_t,n", CASES)
def test_tile_edges(n_det, n_lm, n_t, n, lds_kb, precision):
    import torch
    from oracle import oracle as O
    srate, n_q = (16384.0, 16384) if n_t > 400 else (4096.0, 4096)
    inst = _instance(n_det, n_lm, n_q, srate, n_t, 31 * n_t + n_lm)
    s, _ = synth.prior_samples(n, 7 * n + n_det)
    octx = O.Ctx(inst)
    want = octx.eval(s)
    tol = dict(tol=1e-9) if precision == "fp64" else dict(tol=1e-4, rel=True)
    with ile.Context(inst, precision=precision, lds_kb=lds_kb) as ctx:
        check_margT(ctx.eval(s), want, s, octx, inst, **tol)
        # some of the samples invalid: theirs alone become NaN
        bad = np.arange(n) % 5 == 3
        sb = s.copy()
        sb[5, bad] = -1.0
        d = torch.from_numpy(sb).cuda()
        out = torch.zeros(n, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        ctx.eval_dev(d, n, out)
        if bad.any():
            with pytest.raises(ile.IleError):
                ctx.sync()
        torch.cuda.synchronize()
        got = out.cpu().numpy()
    assert np.all(np.isnan(got[bad]))
    keep = np.nonzero(~bad)[0]
    check_margT(got[keep], want[keep], s, octx, inst, idx=keep, **tol)


@pytest.mark.parametrize("n_lm", [1, 2, 3, 4, 5, 6, 7, 8, 9, 32])
@pytest.mark.parametrize("n_det", [1, 3])
def test_quadratic_term_rows(n_det, n_lm):
    """The quadratic term's rows in fours, its columns in fours: every remainder
    of each; the tiles' tolerance."""
    from oracle import oracle as O
    inst = synth.make_instance(SITES[:n_det], min(n_lm, 21), 4096, 4096.0, 33, 900 + n_lm)
    if n_lm > 21:   # the first modes once more
        i = np.arange(n_lm) % 21
        inst.modes = [inst.modes[j] for j in i]
        inst.Q, inst.U, inst.V = inst.Q[:, i].copy(), inst.U[:, i][:, :, i].copy(), inst.V[:, i][:, :, i].copy()
    s, _ = synth.prior_samples(150, n_lm)
    octx = O.Ctx(inst)
    with ile.Context(inst, precision="fp64") as ctx:
        check_margT(ctx.eval(s), octx.eval(s), s, octx, inst, tol=1e-9)
