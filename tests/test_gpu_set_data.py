"""The series' way to the device: layout of every mode count (the padding rows
of the matrix steps), series that pass the staging buffer whole, by rows and
by parts of a row, against the oracle (the parity tests' tolerance); a value
that is not finite is refused by its index wherever it is, and the context
keeps the data it had, to the bit."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth
from test_gpu_parity import check_margT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n_det,n_lm,n_q", [(1, 1, 4096), (3, 2, 4096), (2, 3, 5001), (3, 5, 4096),
                                            (2, 5, 1 << 20), (1, 1, 1 << 23)])
def test_series_layout(n_det, n_lm, n_q, precision):
    from oracle import oracle as O
    inst = synth.make_instance(["D1", "D2", "D3"][:n_det], n_lm, n_q, 4096.0, 65, n_lm)
    s, _ = synth.prior_samples(40, n_lm)
    octx = O.Ctx(inst)
    tol = dict(tol=1e-9) if precision == "fp64" else dict(tol=1e-4, rel=True)
    with ile.Context(inst, precision=precision) as ctx:
        check_margT(ctx.eval(s), octx.eval(s), s, octx, inst, **tol)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("at", [(0, 0, 0), (1, 2, 700), (1, 2, 4095)])
def test_not_finite_refused(at, precision):
    inst = synth.make_instance(["D1", "D2"], 3, 4096, 4096.0, 65, 8)
    s, _ = synth.prior_samples(100, 9)
    with ile.Context(inst, precision=precision) as ctx:
        want = ctx.eval(s)
        for bad in (np.nan, np.inf, 1j * np.inf):
            Q = inst.Q * 3.0
            Q[at] = bad
            i = int(np.ravel_multi_index(at, Q.shape))
            with pytest.raises(ile.IleError, match=r"Q\[%d\] not finite" % i):
                ile.ile_set_data(ctx.h, Q, inst.t0_s, inst.U, inst.V, inst.dets)
            assert np.array_equal(ctx.eval(s), want)
        ile.ile_set_data(ctx.h, inst.Q, inst.t0_s, inst.U, inst.V, inst.dets)
        assert np.array_equal(ctx.eval(s), want)


def test_staging_is_given_back():
    """A context holds no staging buffer after its first data, and the same one
    through any number of further ones (device memory as the runtime counts
    it, within the 2 MiB pages it hands out)."""
    import torch
    inst = synth.make_instance(["D1", "D2", "D3"], 21, 16384, 16384.0, 65, 8)   # 16.5 MB of series
    raw = 16 * inst.Q.size

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]
    with ile.Context(inst, precision="fp32"):   # code objects and pools of the first use
        pass
    f0 = free()
    with ile.Context(inst, precision="fp32") as ctx:
        planar = 3 * 44 * 16384 * 4
        f1 = free()
        assert f0 - f1 < planar + (12 << 20)
        for _ in range(3):
            ile.ile_set_data(ctx.h, inst.Q, inst.t0_s, inst.U, inst.V, inst.dets)
        assert f1 - free() < raw + (4 << 20)
    assert f0 - free() < (4 << 20)
