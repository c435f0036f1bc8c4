"""Device buffers of ile_set_data, counted by the stand-in for the HIP runtime."""
import pytest

import stand_in


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n_q", [4096, 1 << 17])
def test_first_data_gives_nothing_back(tmp_path, n_q, precision):
    """A context's first data allocates its layout, U, V, their packed triangles
    and a staging buffer of at most 4 MiB, and frees nothing (a hipFree there
    costs the next call what it saves); later data allocates a staging buffer
    once (FP64, FP32) and then nothing."""
    stand_in.run(tmp_path, f"""
        inst = synth.make_instance(["D1", "D2"], 5, {n_q}, 4096.0, 65, 3)
        def alloc(kind):
            return [int(c[3][0]) for c in calls() if c[0] == kind]
        def data(c):
            clear()
            ile.ile_set_data(c.h, inst.Q, inst.t0_s, inst.U, inst.V, inst.dets)
        planar, raw, bf16 = 2 * 12 * {n_q} * 4, 16 * inst.Q.size, {precision!r} == "bf16"
        if {precision!r} == "fp64":
            planar *= 2
        c = ile.Context(inst, precision={precision!r})
        first = alloc("hipMalloc")
        assert alloc("hipFree") == []
        big = [n for n in first if n > 64 << 10]
        assert big[0] >= planar and big[1:] == ([] if bf16 else [min(raw, 4 << 20)]), first
        data(c)
        again = [n for n in alloc("hipMalloc") if n > 1 << 10]
        assert again == ([raw] if not bf16 and raw > 4 << 20 else []), again
        assert alloc("hipFree") == []
        data(c)
        assert alloc("hipFree") == [] and alloc("hipMalloc") == []
        c.close()
    """)


@pytest.mark.parametrize("precision", ["fp64", "bf16"])
@pytest.mark.parametrize("call", ["hipMemcpyAsync", "hipLaunchKernel", "hipMalloc"])
def test_failed_data_is_waited_for(tmp_path, call, precision):
    """Whichever call of ile_set_data fails, first data or further, a copy that
    was queued before it (they read the caller's arrays and the call's own) has
    been waited for when it returns."""
    stand_in.run(tmp_path, f"""
        inst = synth.make_instance(["D1", "D2"], 5, 4096, 4096.0, 65, 3)
        def data(c):
            ile.ile_set_data(c.h, inst.Q, inst.t0_s, inst.U, inst.V, inst.dets)
        for further in (0, 1):
            ended = 0
            for nth in range(1, 20):
                c = ile.Context(inst, precision={precision!r}) if further else None
                clear()
                if c is None:
                    h = ile.ile_create(inst.dets, inst.modes, inst.srate_hz, inst.n_t, precision={precision!r})
                    c = type("H", (), {{"h": h, "close": lambda self: ile.ile_destroy(self.h)}})()
                    clear()
                fail({call!r}, nth)
                try:
                    data(c)
                    ended += 1
                except ile.IleError as e:
                    n = [x[0] for x in calls()]
                    queued = [i for i, x in enumerate(n) if x == "hipMemcpyAsync"]
                    assert not queued or "hipStreamSynchronize" in n[queued[-1]:], (further, nth, n)
                clear()
                c.close()
            assert 0 < ended
    """)


def test_refused_data_leaves_the_geometry(tmp_path):
    """Data refused for its length or a detector leaves the evaluations with the
    series that the context holds; data that fails part way leaves none."""
    stand_in.run(tmp_path, """
        inst = synth.make_instance(["D1", "D2"], 5, 4096, 4096.0, 65, 3)
        s, _ = synth.prior_samples(100, 4)
        c = ile.Context(inst)
        def prep():
            clear()
            c.eval(s)
            return [x[3][2:] for x in calls() if x[0] == "hipLaunchKernel" and "k_prep" in x[3][0]]
        def refused(Q, t0, dets):
            try:
                ile.ile_set_data(c.h, Q, t0, inst.U, inst.V, dets)
            except ile.IleError as e:
                return str(e)
        want = prep()
        assert want == [["4096", str(4096 - 65)]], want
        long = np.concatenate([inst.Q] * 2, axis=2)
        assert "too short" in refused(long, 0.0, inst.dets)
        assert prep() == want
        bad = [inst.dets[0], (95.0, 0.0, 0.0)]
        assert "detector 1" in refused(long, inst.t0_s, bad)
        assert prep() == want
        for nth in range(1, 6):
            c2 = ile.Context(inst)
            clear()
            fail("hipMalloc", nth)
            try:
                ile.ile_set_data(c2.h, long, inst.t0_s, inst.U, inst.V, inst.dets)
                break
            except ile.IleError:
                pass
            # the old data, as only the staging was missing, or none
            c, held = c2, True
            try:
                assert prep() == want
            except ile.IleError as e:
                assert "set_data" in str(e), e
                held = False
            assert held == (nth == 1)
            clear()
            ile.ile_set_data(c2.h, long, inst.t0_s, inst.U, inst.V, inst.dets)
            c2.eval(s)
        assert nth == 3
    """)
