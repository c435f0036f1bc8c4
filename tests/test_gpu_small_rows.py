"""LDS budgets at the least that the phased engine's bin rows take: one unit of
128 bytes (chunks of 15 bins in FP64, 31 in FP32), whether the budget leaves
exactly one, one and more, or less than one; refused where the coefficients
alone take the budget.  Against the FP64 oracle, the parity tests' tolerances."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth
from test_gpu_parity import check_margT

pytestmark = pytest.mark.gpu


def _coef_kb(nd, nl, e):   # [n_det][k-steps][64] and 16 bytes
    return (nd * ((2 * nl + 3) // 4) * 64 * e + 16) / 1024


@pytest.mark.parametrize("precision,e", [("fp64", 8), ("fp32", 4)])
@pytest.mark.parametrize("nd,nl,nt", [(1, 1, 33), (2, 3, 47), (2, 5, 15), (3, 9, 31), (3, 21, 61), (3, 21, 465)])
def test_rows_of_one_unit(nd, nl, nt, precision, e):
    from oracle import oracle as O
    inst = synth.make_instance(["D1", "D2", "D3"][:nd], nl, 16384, 16384.0, nt, nl)
    s, _ = synth.prior_samples(50, nl)
    octx = O.Ctx(inst)
    want = octx.eval(s)
    tol = dict(tol=1e-9) if precision == "fp64" else dict(tol=1e-4, rel=True)
    fixed = _coef_kb(nd, nl, e)
    for kb in range(int(fixed) + 1, int(fixed) + 6):   # a unit of 16 rows is 2 KiB
        with ile.Context(inst, precision=precision, lds_kb=kb) as ctx:
            check_margT(ctx.eval(s), want, s, octx, inst, **tol)
    if int(fixed) > 0:
        with ile.Context(inst, precision=precision, lds_kb=int(fixed)) as ctx:
            with pytest.raises(ile.IleError):
                ctx.eval(s)
