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
