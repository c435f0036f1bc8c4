"""ile_integrate's ways out, with the calls recorded and made to fail by the
stand-in for the HIP runtime: whatever ends it, the work it queued on the
caller's arrays has been waited for, its word of the error flag cleared on the
context's stream, and a failure of the device reported as one."""
import pytest

import stand_in

SETUP = """
        inst = synth.make_instance(["D1", "D2"], 5, 4096, 4096.0, 65, 3)
        s, lp = synth.prior_samples(500, 4)
        bad = s.copy()
        bad[5, 77] = -1.0
        c = ile.Context(inst)
        c.integrate(s, lp, lp)

        def status(x):
            try:
                c.integrate(x, lp, lp)
            except ile.IleError as e:
                return str(e)
            return "ok"
        # the last calls: waited for, then the word cleared on the stream
        def ended():
            n = names({"hipLaunchKernel", "hipStreamSynchronize", "hipMemset", "hipMemsetAsync", "hipMemcpyAsync"})
            return n[-2] == "hipStreamSynchronize" and "k_fill_u32" in n[-1] and "hipMemset" not in n
        clear()
"""


def test_refused_arrays(tmp_path):
    stand_in.run(tmp_path, SETUP + """
        assert "sample 77" in status(bad) and ended(), names()
        assert status(s) == "ok"
    """)


@pytest.mark.parametrize("call", ["hipStreamSynchronize", "hipLaunchKernel"])
def test_device_failure_after_refused_arrays(tmp_path, call):
    """A failing wait, and a failing clear of the word (the last launch)."""
    stand_in.run(tmp_path, SETUP + f"""
        assert "sample 77" in status(bad)
        nth = 1 if {call!r} == "hipStreamSynchronize" else len(names({{"hipLaunchKernel"}}))
        clear()
        fail({call!r}, nth)
        assert "ILE_E_DEVICE" in status(bad), names()
        clear()
        assert status(s) == "ok"
    """)


@pytest.mark.parametrize("call,nth", [("hipMemcpyAsync", 2), ("hipLaunchKernel", 1),
                                      ("hipLaunchKernel", 3), ("hipEventRecord", 1)])
def test_failure_while_queueing(tmp_path, call, nth):
    stand_in.run(tmp_path, SETUP + f"""
        fail({call!r}, {nth})
        assert "ILE_E_DEVICE" in status(s) and ended(), names()
        clear()
        fail({call!r}, {nth})
        assert "sample 77" in status(bad) and ended(), names()
    """)
