"""Where a batch's per-sample terms come from, by its terms limit (stand-in for
the HIP runtime: the launches and allocations of one run)."""
import stand_in


def test_terms_limit(tmp_path):
    stand_in.run(tmp_path, """
        pts = [synth.make_instance(["D1", "D2"], 5, 4096, 4096.0, 65, p) for p in (3, 4)]
        b = ile.Batch("fp64")
        for p in pts:
            b.add_point(p)
        n = 1000
        need = 2 * 8 * (2 + 3 * 2 + 2 * 5) * 1008   # whole tiles of each point

        def run():
            clear()
            b.run(1, n)
            return [x for x in names({"hipLaunchKernel"}) if "k_terms" in x], \\
                   [x[3][0] for x in calls() if x[0] == "hipMalloc"].count(str(need))
        kernel, alloc = run()
        assert len(kernel) == 1 and alloc == 1
        assert run() == ([], 0)                 # the recorded graph again
        b.set_terms_limit(need)
        assert len(run()[0]) == 1               # built again
        clear()
        b.set_terms_limit(need - 1)
        assert [x[3][0] for x in calls() if x[0] == "hipFree"] == [str(need)]
        assert run() == ([], 0)
        b.set_terms_limit(0)
        assert run() == ([], 0)
        b.set_terms_limit(1 << 35)
        kernel, alloc = run()
        assert len(kernel) == 1 and alloc == 1
        b.close()
    """)
