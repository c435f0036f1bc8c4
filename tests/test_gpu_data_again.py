"""A context's first series are laid out by the host, its further ones on the
device (whole through the staging buffer, by rows, by parts of a row): the same
values either way, so the evaluations agree bit for bit, and other series set
in between leave nothing behind."""
import numpy as np
import pytest

from paper_1902_04934_amd import ile, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n_det,n_lm,n_q", [(1, 1, 4096), (3, 2, 4096), (2, 3, 5001), (3, 5, 4096),
                                            (2, 5, 1 << 20), (1, 1, 1 << 23)])
def test_first_and_further_data_agree(n_det, n_lm, n_q, precision):
    if precision == "bf16" and n_q > 1 << 16:
        pytest.skip("the host lays BF16 series out each time")
    inst = synth.make_instance(["D1", "D2", "D3"][:n_det], n_lm, n_q, 4096.0, 65, n_lm)
    s, _ = synth.prior_samples(300, n_lm)
    with ile.Context(inst, precision=precision) as ctx:
        first = ctx.eval(s)
        ile.ile_set_data(ctx.h, inst.Q[:, ::-1] * 1.5, inst.t0_s, inst.U, inst.V, inst.dets)
        other = ctx.eval(s)
        ile.ile_set_data(ctx.h, inst.Q, inst.t0_s, inst.U, inst.V, inst.dets)
        assert np.array_equal(ctx.eval(s), first)
    with ile.Context(inst, precision=precision) as ctx:   # the other series first
        ile.ile_set_data(ctx.h, inst.Q[:, ::-1] * 1.5, inst.t0_s, inst.U, inst.V, inst.dets)
        assert np.array_equal(ctx.eval(s), other)
    assert np.all(np.isfinite(first)) and not np.array_equal(first, other)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_refused_data_keeps_the_old(precision):
    """Series too short, an invalid detector behind a valid one, a value that is
    not finite in a context's first series."""
    inst = synth.make_instance(["D1", "D2"], 3, 4096, 4096.0, 65, 8)
    other = synth.make_instance(["D3", "D1"], 3, 4096, 4096.0, 65, 9)
    s, _ = synth.prior_samples(300, 9)
    h = ile.ile_create(inst.dets, inst.modes, inst.srate_hz, inst.n_t, d_ref_mpc=inst.d_ref_mpc,
                       gmst_rad=inst.gmst_rad, precision=precision)
    Q = inst.Q.copy()
    Q[1, 2, 77] = np.nan
    with pytest.raises(ile.IleError, match=r"Q\[%d\] not finite" % (5 * 4096 + 77)):
        ile.ile_set_data(h, Q, inst.t0_s, inst.U, inst.V, inst.dets)
    with pytest.raises(ile.IleError, match="set_data has not"):
        ile.ile_eval(h, s)
    ile.ile_set_data(h, inst.Q, inst.t0_s, inst.U, inst.V, inst.dets)
    want = ile.ile_eval(h, s)
    with pytest.raises(ile.IleError, match="too short"):
        ile.ile_set_data(h, other.Q, 0.0, other.U, other.V, other.dets)
    assert np.array_equal(ile.ile_eval(h, s), want)
    with pytest.raises(ile.IleError, match="detector 1"):
        ile.ile_set_data(h, other.Q, other.t0_s, other.U, other.V, [other.dets[0], (95.0, 0.0, 0.0)])
    assert np.array_equal(ile.ile_eval(h, s), want)
    ile.ile_destroy(h)
