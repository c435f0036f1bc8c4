"""Contexts on two devices in one process: every entry point works on its own
context's device whichever device is current (the stand-in for the HIP runtime
refuses a launch on a stream of another device, as the runtime does, and
records where each call went)."""
import stand_in


def test_calls_go_to_the_contexts_device(tmp_path):
    stand_in.run(tmp_path, """
        inst = synth.make_instance(["D1", "D2"], 5, 4096, 4096.0, 65, 3)
        s, lp = synth.prior_samples(500, 4)

        class Dev:   # a device buffer
            def __init__(self, n):
                self.a = np.zeros(n)
            def data_ptr(self):
                return self.a.ctypes.data
        S, P, R, O = Dev(7 * 500), Dev(500), Dev(6), Dev(500)
        c = [ile.Context(inst, device=d) for d in (0, 1)]
        prop = [ile.Proposal(seed=1, device=d) for d in (0, 1)]
        batch = [ile.Batch(device=d) for d in (0, 1)]
        for b in batch:
            b.add_point(inst)
        ops = {
            "sync": lambda d: c[d].sync(),
            "eval": lambda d: c[d].eval(s),
            "eval_dev": lambda d: c[d].eval_dev(S, 500, O),
            "integrate": lambda d: c[d].integrate(s, lp, lp),
            "integrate_dev": lambda d: c[d].integrate_dev(S, P, P, 500, R),
            "noalloc": lambda d: c[d].integrate_dev_noalloc(S, P, P, 500, R),
            "set_data": lambda d: ile.ile_set_data(c[d].h, inst.Q, inst.t0_s, inst.U, inst.V, inst.dets),
            "draw_prior": lambda d: c[d].draw_prior_dev(1, 0, 500, S, 500, P),
            "run_prior": lambda d: c[d].run_prior(1, 1000, 500),
            "run": lambda d: c[d].run(sampler="adaptive", max_samples=1000, chunk=500),
            "params": lambda d: prop[d].set_params(prop[d].get_params()),
            "sample": lambda d: prop[d].sample_dev(1, 0, 500, S, 500, P, O),
            "prop_sync": lambda d: prop[d].sync(),
            "batch": lambda d: batch[d].run(1, 100),
            "batch_lnL": lambda d: batch[d].lnL(100),
        }
        hip = {"hipLaunchKernel", "hipMemcpyAsync", "hipMemsetAsync", "hipMemset", "hipEventRecord",
               "hipMalloc"}
        bad = []
        for name, op in ops.items():
            for d in (0, 1):
                si.hipSetDevice(1 - d)
                clear()
                try:
                    op(d)
                except ile.IleError as e:
                    bad.append((name, d, str(e)))
                wrong = [x[:3] for x in calls() if x[0] in hip and (x[1] != d or x[2] not in (-1, d))]
                if wrong:
                    bad.append((name, d, wrong[0]))
        assert not bad, bad
    """)
