"""Which chunks of a run merge the partials of all chunks so far into a result
(one thread, in order): those whose result the host reads."""
import stand_in


def test_chunks_that_merge(tmp_path):
    stand_in.run(tmp_path, """
        inst = synth.make_instance(["D1", "D2"], 5, 4096, 4096.0, 65, 3)
        c = ile.Context(inst)

        def merges(**kw):
            clear()
            c.run(**dict(dict(max_samples=2300, chunk=500), **kw))
            return [x[3][2] for x in calls() if x[0] == "hipLaunchKernel" and "k_red_small" in x[3][0]]
        last, every = ["none"] * 4 + ["result"], ["result"] * 5
        assert merges(sampler="prior") == last
        assert merges(sampler="prior", n_eff_target=1e9) == every
        assert merges(sampler="adaptive", adapt_chunks=0) == last
        assert merges(sampler="adaptive", adapt_chunks=3) == last
        assert merges(sampler="adaptive", adapt_chunks=3, n_eff_target=1e9) == every
        # adaptation that decides for itself reads each result until it ends
        # (here never: the kernels leave zeros)
        assert merges(sampler="adaptive", adapt_chunks=-1) == every
        assert merges(sampler="prior", max_samples=400) == ["result"]
        with ile.Proposal(c, seed=1) as p:
            # five estimation chunks at the end
            assert merges(sampler="learned", prop=p.h, fallback_neff=0.0)[-5:] == last
            assert merges(sampler="learned", prop=p.h, fallback_neff=0.0, n_eff_target=1e9)[-5:] == every
        # chunks of more than 16384 samples
        clear()
        c.run(sampler="prior", max_samples=60_000, chunk=20_000)
        assert [x[3][2] for x in calls() if "k_red_final" in (x[3] or [""])[0]] == ["none"] * 2 + ["result"]
        c.close()
    """)
