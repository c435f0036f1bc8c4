"""Timed cases of the library: the calls a program built on it makes, from the
smallest integrate to the million-sample evaluation, through the public entry
points of ``paper_1902_04934_amd.ile``.

A case is one call (or the short sequence of calls that belongs together):

  evaluate   ``eval_dev``: ln L_margT per sample, device buffers
  integrate  ``integrate_dev`` / ``integrate_dev_noalloc`` (device buffers) or
             ``integrate`` (host arrays): the reduced result
  batch      ``Batch.run_dev``: many intrinsic points, each on draws of its own
  surrogate  ``ile_rom_integrate_dev``: joint (lambda, theta) samples
  build      ``ile_qvu_fd_dev``: Q, U, V from frequency-domain series
  harvest    ``harvest_dev``: one final iteration with joint posterior draws
  draw       ``Proposal.sample_dev``: draws of the learned defensive mixture
  train      ``Proposal.set_params`` + ``train_dev``: one training of the network
  point      ``ile_set_data`` (host Q, U, V) + an adaptive ``run``: what a loop
             over intrinsic points does for each of them

FP64 is the reference precision and FP32 the fast one; the BF16 form is a
variant for accuracy studies (slower than both) and is not timed here.
"""
import math

import numpy as np
import torch

from paper_1902_04934_amd import ile

# (lat deg, lon deg, x-arm azimuth deg from local East) of the three sites
SITES = [(46.455, -119.408, 126.0), (30.563, -90.774, 198.0), (43.631, 10.504, 71.0)]
# l = 2 .. 4 in the order the configurations take prefixes of (5, 9, 13, 21)
MODES = [(2, 2), (2, -2), (2, 1), (2, -1), (2, 0), (3, 3), (3, -3), (3, 2), (3, -2),
         (4, 4), (4, -4), (4, 3), (4, -3), (3, 1), (3, -1), (3, 0), (4, 2), (4, -2),
         (4, 1), (4, -1), (4, 0)]
C_LIGHT = 299792458.0
R_EARTH = 6378.0e3
D_REF, D_MIN, D_MAX, T_MAX = 100.0, 10.0, 1000.0, 0.010
N_PARAM = 60880


def listed():
    return [
        # the smallest call: a thousand samples of a two-detector point inside
        # a serving loop that may not allocate; latency and launches
        dict(name="integrate_1e3_noalloc", kind="integrate", entry="noalloc", precision="fp64",
             n_det=2, n_lm=5, n_q=4096, n_t=201, n=1000, draws="prior"),
        # the paper's block of 1e4 samples from host arrays
        dict(name="integrate_1e4_host", kind="integrate", entry="host", precision="fp64",
             n_det=2, n_lm=5, n_q=4096, n_t=201, n=10_000, draws="prior"),
        # one chunk of a sampler that has found the source: concentrated draws
        dict(name="integrate_1e5_chunk", kind="integrate", entry="dev", precision="fp64",
             n_det=3, n_lm=9, n_q=16384, n_t=1601, n=100_000, draws="posterior"),
        # the at-scale single-point evaluation (the benchmark's shape)
        dict(name="evaluate_1e6_fp64", kind="evaluate", precision="fp64", n_det=3, n_lm=21,
             n_q=16384, n_t=1601, n=1_000_000, draws="prior"),
        # single precision, odd sizes
        dict(name="evaluate_2e5_fp32_odd", kind="evaluate", precision="fp32", n_det=3, n_lm=13,
             n_q=16384, n_t=1103, n=200_003, draws="prior"),
        # a group of intrinsic points of mixed shape, each on its own draws
        dict(name="batch_8x1e5_fp32", kind="batch", precision="fp32", points=8, n_q=16384,
             n=100_000),
        # the surrogate form: one Monte Carlo over lambda and theta
        dict(name="surrogate_1e5", kind="surrogate", precision="fp64", n_det=3, n_lm=21, n_b=21,
             n_pow=4, n_q=16384, n_t=1601, n=100_000, draws="prior"),
        # set-up of one intrinsic point from spectra
        dict(name="build_3x21x16384", kind="build", n_det=3, n_lm=21, n_q=16384),
        # the final iteration: evaluate, reduce, draw the joint posterior
        dict(name="harvest_2e5", kind="harvest", precision="fp64", n_det=3, n_lm=21, n_q=16384,
             n_t=1601, n=200_000, n_out=20_000, draws="prior"),
        # one chunk of draws from the learned proposal
        dict(name="draw_1e5", kind="draw", n=100_000, eps=0.1),
        # one refit of the learned proposal on its training ring
        dict(name="train_150x16384", kind="train", n=300_000, steps=150, batch=16384),
        # the next intrinsic point of a loop: its data, then an adaptive run
        dict(name="point_adaptive_3e5", kind="point", precision="fp64", n_det=3, n_lm=21,
             n_q=16384, n_t=1601, n=300_000, chunk=100_000),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(rng, lo, hi):
    return 2 * _logint(rng, lo // 2, hi // 2) + 1


# sample x bin x detector x mode products of the largest listed case
_MOST = 1_000_000 * 1601 * 3 * 21


def draw(rng):
    kind = rng.choice(["integrate", "integrate", "integrate", "evaluate", "evaluate", "batch",
                       "surrogate", "build", "harvest", "draw", "train", "point"])
    n_det = rng.choice([1, 2, 3, 3])
    n_lm = rng.choice([5, 9, 13, 21, rng.randint(1, 21)])
    n_q = rng.choice([4096, 16384, 16384])
    n_t = _odd(rng, 101, 1601)
    shape = dict(n_det=n_det, n_lm=n_lm, n_q=n_q, n_t=n_t, draws=rng.choice(["prior", "posterior"]),
                 precision=rng.choice(["fp64", "fp64", "fp32"]))

    def samples(lo, hi, extra=1):
        return max(lo, min(_logint(rng, lo, hi), _MOST // (n_t * n_det * n_lm * extra)))

    if kind == "integrate":
        entry = rng.choice(["dev", "host", "noalloc"])
        return dict(shape, kind=kind, entry=entry,
                    n=samples(500, 60_000 if entry == "noalloc" else 300_000))
    if kind == "evaluate":
        return dict(shape, kind=kind, n=samples(3_000, 1_000_000))
    if kind == "batch":
        points = rng.randint(2, 12)
        return dict(kind=kind, points=points, n_q=n_q, precision=shape["precision"],
                    n=_logint(rng, 3_000, 900_000 // points))
    if kind == "surrogate":
        return dict(shape, kind=kind, n_b=n_lm, n_lm=rng.choice([5, 9, 21]), n_pow=rng.randint(2, 5),
                    precision="fp64", n=samples(3_000, 200_000))
    if kind == "build":
        return dict(kind=kind, n_det=n_det, n_lm=n_lm, n_q=rng.choice([1024, 4096, 8192, 16384, 32768]))
    if kind == "harvest":
        n = samples(5_000, 300_000)
        return dict(shape, kind=kind, precision="fp64", n=n, n_out=max(100, n // rng.randint(4, 30)))
    if kind == "draw":
        return dict(kind=kind, n=_logint(rng, 1_000, 1_000_000), eps=rng.choice([0.0, 0.1, 0.2]))
    if kind == "train":
        batch = rng.choice([4096, 8192, 16384, rng.randint(2_000, 17_000)])
        return dict(kind=kind, n=_logint(rng, 20_000, 400_000), batch=batch,
                    steps=min(rng.randint(20, 200), 150 * 16384 // batch))
    chunk = _logint(rng, 10_000, 100_000)
    return dict(shape, kind="point", precision="fp64", chunk=chunk, n=chunk * rng.randint(2, 4))


# ------------------------------------------------------------------ inputs
class _Point:
    """One intrinsic point: detectors, modes, grid and the stand-in Q, U, V."""

    def __init__(self, rng, n_det, n_lm, n_q, n_t):
        self.dets, self.modes = SITES[:n_det], MODES[:n_lm]
        self.n_det, self.n_lm, self.n_q, self.n_t = n_det, n_lm, n_q, n_t
        self.srate_hz, self.t_ref_max_s = float(n_q if n_q in (4096, 16384) else 16384), T_MAX
        self.d_ref_mpc, self.gmst_rad, self.earth_radius_m = D_REF, 0.0, R_EARTH
        self.t0_s = -(n_q // 2) / self.srate_hz
        # a burst per detector near the event time in unit complex noise, the
        # modes' amplitudes falling off; U, V Gram matrices of that scale
        amp = 20.0 * 0.3 ** np.arange(n_lm)
        off = rng.integers(-int(0.008 * self.srate_hz), int(0.008 * self.srate_hz) + 1, n_det)
        u = (np.arange(n_q)[None] - n_q // 2 - off[:, None]) / self.srate_hz
        burst = np.exp(-u * u / (2 * 0.004 ** 2) + 2j * np.pi * (60.0 * u + 2000.0 * u * u))
        ph = np.exp(2j * np.pi * rng.random((n_det, n_lm)))
        self.Q = burst[:, None, :] * (amp * ph)[:, :, None]
        noise = rng.standard_normal((n_det, n_lm, n_q, 2), dtype=np.float32)
        self.Q += noise.astype(np.float64).view(np.complex128)[..., 0] * math.sqrt(0.5)
        A = rng.standard_normal((n_det, 64, n_lm)) + 1j * rng.standard_normal((n_det, 64, n_lm))
        U, V = A.conj().transpose(0, 2, 1) @ A, A.transpose(0, 2, 1) @ A
        s = np.mean(amp ** 2) * n_lm / np.trace(U, axis1=1, axis2=2).real
        self.U = 0.5 * (U + U.conj().transpose(0, 2, 1)) * s[:, None, None]
        self.V = 0.5 * (V + V.transpose(0, 2, 1)) * s[:, None, None]


def _samples(rng, n, draws):
    """Samples [7][n] and their log prior density: prior draws, or draws
    concentrated as a proposal that has found a source makes them."""
    s = np.empty((7, n))
    if draws == "prior":
        s[0] = rng.uniform(0, 2 * np.pi, n)
        s[1] = np.arcsin(rng.uniform(-1, 1, n))
        s[2] = rng.uniform(0, np.pi, n)
        s[4] = rng.uniform(-1, 1, n)
        s[5] = np.cbrt(D_MIN ** 3 + rng.random(n) * (D_MAX ** 3 - D_MIN ** 3))
        s[6] = rng.uniform(-T_MAX, T_MAX, n)
    else:
        g = rng.standard_normal((5, n))
        c = rng.random(5)
        s[0] = (2 * np.pi * c[0] + 0.05 * g[0]) % (2 * np.pi)
        s[1] = np.clip(1.8 * c[1] - 0.9 + 0.05 * g[1], -1.5, 1.5)
        s[2] = rng.uniform(0, np.pi, n)
        s[4] = np.clip(1.6 * c[2] - 0.8 + 0.15 * g[2], -0.999, 0.999)
        s[5] = np.clip(400.0 + 80.0 * g[3], 50.0, 950.0)
        s[6] = np.clip((c[4] - 0.5) * T_MAX + 5e-4 * g[4], -T_MAX, T_MAX)
    s[3] = rng.uniform(0, 2 * np.pi, n)
    v3 = D_MAX ** 3 - D_MIN ** 3
    lp = (np.log(np.cos(s[1]) / 2) + np.log(3 * s[5] ** 2 / v3)
          - math.log(2 * np.pi) * 2 - math.log(np.pi) - math.log(2.0) - math.log(2 * T_MAX))
    return s, lp


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _eval_inputs(case, seed):
    rng = np.random.default_rng([seed, 1])
    pt = _Point(rng, case["n_det"], case.get("n_b", case["n_lm"]), case["n_q"], case["n_t"])
    s, lp = _samples(rng, case["n"], case["draws"])
    lq = lp + 0.3 * rng.standard_normal(case["n"])
    return rng, pt, s, lp, lq


def _rom_inputs(case, rng):
    lam = rng.uniform(-1, 1, case["n"])
    A = (rng.standard_normal((case["n_lm"], case["n_b"], case["n_pow"], 2))
         .view(np.complex128)[..., 0] / case["n_b"])
    return lam, A


def _batch_inputs(case, seed):
    rng = np.random.default_rng([seed, 2])
    pts, S, LP, LQ = [], [], [], []
    for _ in range(case["points"]):
        n_lm, h = int(rng.choice([5, 9, 13, 21])), int(rng.integers(100, 801))
        pts.append(_Point(rng, 3, n_lm, case["n_q"], 2 * h + 1))
        s, lp = _samples(rng, case["n"], "posterior")
        S.append(s)
        LP.append(lp)
        LQ.append(lp + 0.3 * rng.standard_normal(case["n"]))
    return pts, np.stack(S), np.stack(LP), np.stack(LQ)


def _fd_inputs(case, seed):
    """Transforms of mode series and data, and spectra, on the FFT grid."""
    rng = np.random.default_rng([seed, 3])
    n, nd, nl = case["n_q"], case["n_det"], case["n_lm"]
    srate = 16384.0
    df = srate / n
    i = np.arange(n)
    f = np.where(i < n // 2, i, i - n) * df
    u = np.where(i < n // 2, i, i - n) / srate
    env = np.exp(-u * u / (2 * 0.03 ** 2))
    ph = 2 * np.pi * rng.random(nl)
    chirp = 2 * np.pi * (40.0 * u + 750.0 * u * u)
    h = np.stack([20.0 * 0.3 ** a * env * np.exp(1j * (ph[a] + 0.5 * MODES[a][1] * chirp))
                  for a in range(nl)])
    h_f = np.fft.fft(h, axis=1) / srate
    fs = np.maximum(np.abs(f), df)
    shape = (40.0 / fs) ** 4 + 1.0 + (fs / 320.0) ** 2
    psd = 1e-3 * shape[None] * rng.uniform(0.5, 2.0, (nd, 1))
    noise = rng.standard_normal((nd, n, 2)).view(np.complex128)[..., 0]
    lag = rng.uniform(-0.01, 0.01, (nd, 1))
    d_f = noise * np.sqrt(psd / (4 * df)) + h_f[:1] * np.exp(-2j * np.pi * f * lag)
    return dict(h=h_f, d=d_f, psd=psd, df=df, f=f, f_min=20.0, f_max=4000.0,
                t0=-(n // 2) / srate)


def _net(rng):
    """Network parameters as after some training: seeded weights, mixture
    means spread over the line, scales of a few tenths."""
    P = []
    for size, fan in ((896, 135), (128, 0), (16384, 256), (128, 0), (43008, 464)):
        P.append(rng.uniform(-1, 1, size) * (math.sqrt(6.0 / fan) if fan else 0.1))
    b3 = np.zeros((7, 3, 16))
    b3[:, 1] = np.linspace(-2.0, 2.0, 16)
    b3[:, 2] = math.log(math.expm1(0.4))
    P.append(b3.reshape(-1) + rng.uniform(-0.1, 0.1, 336))
    return np.concatenate(P).astype(np.float32)


def _hist(rng, nb=50):
    h = rng.random((2, nb)) ** 4 + 0.002
    return [x / x.sum() for x in 0.9 * h / h.sum(1, keepdims=True) + 0.1 / nb]


def _context(pt, precision="fp64"):
    return ile.Context(pt, precision=precision)


# ----------------------------------------------------------------- prepare
def prepare(case, seed):
    kind = case["kind"]
    st = dict(kind=kind, case=case)
    if kind in ("integrate", "evaluate", "harvest", "surrogate"):
        rng, pt, s, lp, lq = _eval_inputs(case, seed)
        st["ctx"] = _context(pt, case["precision"])
        if kind == "surrogate":
            lam, A = _rom_inputs(case, rng)
            ile.ile_rom_set(st["ctx"].h, MODES[:case["n_lm"]], A)
            s = np.concatenate([s, lam[None]])
        if kind == "integrate" and case["entry"] == "host":
            st.update(s=s, lp=lp, lq=lq)
            return st
        st.update(s=_dev(s), lp=_dev(lp), lq=_dev(lq))
        st["res"] = torch.zeros(6, dtype=torch.float64, device="cuda")
        if kind == "evaluate":
            st["out"] = torch.zeros(case["n"], dtype=torch.float64, device="cuda")
        if kind == "harvest":
            m = case["n_out"]
            st["u"] = _dev(rng.random((2, m)))
            st["idx"] = torch.zeros(m, dtype=torch.int64, device="cuda")
            st["bin"] = torch.zeros(m, dtype=torch.int32, device="cuda")
            st["theta"] = torch.zeros((7, m), dtype=torch.float64, device="cuda")
    elif kind == "batch":
        pts, S, LP, LQ = _batch_inputs(case, seed)
        st["batch"] = ile.Batch(precision=case["precision"])
        for p in pts:
            st["batch"].add_point(p)
        st.update(s=_dev(S), lp=_dev(LP), lq=_dev(LQ))
    elif kind == "build":
        f = _fd_inputs(case, seed)
        nd, nl, n = case["n_det"], case["n_lm"], case["n_q"]
        st["h"] = ile.ile_create(SITES[:nd], MODES[:nl], 16384.0, 201)
        st["fd"] = f
        st.update(hf=_dev(f["h"]), df=_dev(f["d"]), psd=_dev(f["psd"]))
        for name, shape in (("Q", (nd, nl, n)), ("U", (nd, nl, nl)), ("V", (nd, nl, nl))):
            st[name] = torch.zeros(shape, dtype=torch.complex128, device="cuda")
    elif kind in ("draw", "train"):
        rng = np.random.default_rng([seed, 4])
        st["P"] = _net(rng)
        if kind == "draw":
            st["ctx"] = _context(_Point(rng, 1, 1, 4096, 101))
            ile.ile_hist_set(st["ctx"].h, *_hist(rng))
            st["prop"] = ile.Proposal(st["ctx"], seed=3, sigma_scale=1.2)
            st["prop"].set_params(st["P"])
            st["prop"].set_transform(2 * np.pi * rng.random(3), rng.normal(0, 0.5, 7),
                                     rng.uniform(0.3, 1.5, 7))
            st["seed"] = int(rng.integers(1 << 40))
            st["x"] = torch.zeros((7, case["n"]), dtype=torch.float64, device="cuda")
            st["lnp"] = torch.zeros(case["n"], dtype=torch.float64, device="cuda")
            st["lnq"] = torch.zeros(case["n"], dtype=torch.float64, device="cuda")
        else:
            s, _ = _samples(rng, case["n"], "prior")
            k = case["n"] // 3
            s[:, k:] = _samples(rng, case["n"] - k, "posterior")[0]
            c = s[:, -1:]
            w = np.array([0.1, 0.1, 1.0, 2.0, 0.3, 120.0, 1e-3])[:, None]
            lnw = 150.0 - 0.5 * (((s - c) / w) ** 2).sum(0)
            st["prop"] = ile.Proposal(seed=3)
            st.update(s=_dev(s), lnw=_dev(lnw), seed=int(rng.integers(1 << 40)))
    else:   # point
        rng = np.random.default_rng([seed, 5])
        args = (case["n_det"], case["n_lm"], case["n_q"], case["n_t"])
        st["pt"] = _Point(rng, *args)
        # the loop's context, which held the point before
        st["ctx"] = _context(_Point(rng, *args), case["precision"])
        st["seed"] = int(rng.integers(1 << 40))
    torch.cuda.synchronize()
    return st


# --------------------------------------------------------------------- run
def run(st):
    kind, case = st["kind"], st["case"]
    n = case.get("n")
    if kind == "evaluate":
        st["ctx"].eval_dev(st["s"], n, st["out"])
        return st["out"]
    if kind == "integrate":
        if case["entry"] == "host":
            return st["ctx"].integrate(st["s"], st["lp"], st["lq"])
        call = (st["ctx"].integrate_dev_noalloc if case["entry"] == "noalloc"
                else st["ctx"].integrate_dev)
        call(st["s"], st["lp"], st["lq"], n, st["res"])
        return st["res"]
    if kind == "batch":
        return st["batch"].run_dev(n, st["s"], st["lp"], st["lq"])
    if kind == "surrogate":
        ile.ile_rom_integrate_dev(st["ctx"].h, st["s"], st["lp"], st["lq"], n, st["res"])
        return st["res"]
    if kind == "build":
        f = st["fd"]
        ile.ile_qvu_fd_dev(st["h"], st["hf"], st["df"], st["psd"], case["n_q"], f["df"],
                           f["f_min"], f["f_max"], f["t0"], st["Q"], st["U"], st["V"])
        return dict(Q=st["Q"], U=st["U"], V=st["V"])
    if kind == "harvest":
        st["ctx"].harvest_dev(st["s"], st["lp"], st["lq"], n, st["u"], case["n_out"], st["idx"],
                              st["bin"], st["theta"], st["res"])
        return dict(idx=st["idx"], bin=st["bin"], theta=st["theta"], result=st["res"])
    if kind == "draw":
        st["prop"].sample_dev(st["seed"], 0, n, st["x"], n, st["lnp"], st["lnq"], eps=case["eps"])
        return dict(x=st["x"], ln_p=st["lnp"], ln_q=st["lnq"])
    if kind == "train":
        st["prop"].set_params(st["P"])
        loss = st["prop"].train_dev(st["s"], n, st["lnw"], n, steps=case["steps"],
                                    batch=case["batch"], lr=2e-3, seed=st["seed"])
        return dict(loss=loss, params=st["prop"].get_params())
    pt = st["pt"]
    ile.ile_set_data(st["ctx"].h, pt.Q, pt.t0_s, pt.U, pt.V, pt.dets)
    return st["ctx"].run(sampler="adaptive", seed=st["seed"], chunk=case["chunk"], max_samples=n)


# -------------------------------------------------------------------- work
def work(case):
    kind = case["kind"]
    n = case.get("n", 0)

    def eval_work(n_det, n_lm, n_q, n_t, n, e):
        return (n * 64 + n_det * n_lm * n_q * 2 * e + 32 * n_det * n_lm ** 2,
                n * (4 * n_det * n_lm * n_t + 16 * n_det * n_lm ** 2))

    e = 4 if case.get("precision") == "fp32" else 8
    if kind == "batch":   # the points' shapes vary by seed: the mean of the mix
        b, f = eval_work(3, 12, case["n_q"], 901, n, e)
        return dict(bytes=case["points"] * (b + 16 * n), flops=case["points"] * f)
    if kind == "build":
        nd, nl, q = case["n_det"], case["n_lm"], case["n_q"]
        band = q * 4000.0 / 8192.0
        return dict(bytes=16 * nl * q + 24 * nd * q + 16 * nd * nl * q + 32 * nd * nl * nl,
                    flops=nd * nl * q * (5 * math.log2(q) + 14) + 16 * nd * nl * nl * band)
    net = 2 * (7 * 128 + 128 * 128 + 336 * 128)
    if kind == "draw":   # the ancestral pass (each unit once) and the density
        return dict(bytes=n * 72 + 4 * N_PARAM, flops=2 * net * n)
    if kind == "train":
        return dict(bytes=n * 64 + 4 * N_PARAM * 2,
                    flops=3 * net * case["steps"] * case["batch"])
    nb = case.get("n_b", case["n_lm"])
    b, f = eval_work(case["n_det"], nb, case["n_q"], case["n_t"], n, e)
    if kind == "integrate":
        b += 16 * n
    if kind == "surrogate":
        b += 24 * n
        f += n * 8 * case["n_lm"] * nb * case["n_pow"]
    if kind == "harvest":
        m = case["n_out"]
        b += 16 * n + m * (16 + 12 + 56)
        f += m * 4 * case["n_det"] * nb * case["n_t"]
    if kind == "point":
        b += case["n_det"] * nb * case["n_q"] * 16
    return dict(bytes=b, flops=f)


# ------------------------------------------------------------------- exact
def _frame(det):
    lat, lon, az = (math.radians(x) for x in det)
    e = np.array([-math.sin(lon), math.cos(lon), 0.0])
    nn = np.array([-math.sin(lat) * math.cos(lon), -math.sin(lat) * math.sin(lon), math.cos(lat)])
    x, y = math.cos(az) * e + math.sin(az) * nn, -math.sin(az) * e + math.cos(az) * nn
    r = R_EARTH * np.array([math.cos(lat) * math.cos(lon), math.cos(lat) * math.sin(lon),
                            math.sin(lat)])
    return r, 0.5 * (np.outer(x, x) - np.outer(y, y))


def _ylm(l, m, ci, phi):
    """-2Y_lm by its Wigner-d sum."""
    c, s = torch.sqrt(0.5 * (1 + ci)), torch.sqrt(0.5 * (1 - ci))
    F = math.factorial
    norm = math.sqrt((2 * l + 1) / (4 * math.pi) * F(l + m) * F(l - m) * F(l + 2) * F(l - 2))
    d = torch.zeros_like(ci)
    for k in range(max(0, m - 2), min(l + m, l - 2) + 1):
        a = (-1) ** k * norm / (F(l + m - k) * F(l - 2 - k) * F(k) * F(k + 2 - m))
        d = d + a * c ** (2 * l + m - 2 - 2 * k) * s ** (2 * k + 2 - m)
    return torch.complex(d * torch.cos(m * phi), d * torch.sin(m * phi))


def _lnl(pt, s, rom=None):
    """ln L_margT [n] of Eqs. (7) and (9) in 64 bits: per block of samples the
    products over the union of the block's windows, gathered per sample."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    S = torch.from_numpy(s).to(dev)
    dt, half = 1.0 / pt.srate_hz, (pt.n_t - 1) // 2
    Qr = [torch.from_numpy(np.concatenate([pt.Q[k].real, pt.Q[k].imag])).to(dev)
          for k in range(pt.n_det)]
    U, V = torch.from_numpy(pt.U).to(dev), torch.from_numpy(pt.V).to(dev)
    j = torch.arange(pt.n_t, device=dev)
    out = []
    for b in range(0, S.shape[1], 4096):
        th = S[:, b:b + 4096]
        ra, dec, psi = th[0], th[1], th[2]
        if rom is None:
            Y = torch.stack([_ylm(l, m, th[4], th[3]) for l, m in pt.modes], 1)
        else:
            modes, A = rom
            A = torch.from_numpy(A).to(dev)
            Y = 0
            for a, (l, m) in enumerate(modes):
                c = A[a, :, -1][None].expand(th.shape[1], -1)
                for p in range(A.shape[2] - 2, -1, -1):
                    c = c * th[7][:, None] + A[a, :, p][None]
                Y = Y + c * _ylm(l, m, th[4], th[3])[:, None]
        kap = D_REF / th[5]
        L, q = 0.0, 0.0
        sh, ch, sd, cd = torch.sin(ra), torch.cos(ra), torch.sin(dec), torch.cos(dec)
        E = torch.stack([-sh, ch, 0 * sh])
        N = torch.stack([-sd * ch, -sd * sh, cd])
        X = -torch.cos(psi) * E + torch.sin(psi) * N
        W = torch.sin(psi) * E + torch.cos(psi) * N
        for k in range(pt.n_det):
            r, D = _frame(pt.dets[k])
            DX = torch.from_numpy(D).to(dev) @ X
            DW = torch.from_numpy(D).to(dev) @ W
            fp, fx = (X * DX).sum(0) - (W * DW).sum(0), (X * DW).sum(0) + (W * DX).sum(0)
            Fk = torch.complex(fp, fx)
            tau = -(cd * ch * r[0] + cd * sh * r[1] + sd * r[2]) / C_LIGHT
            st = torch.floor((th[6] + tau - pt.t0_s) / dt + 0.5).long() - half
            lo, hi = int(st.min()), int(st.max())
            c = kap[:, None] * Fk[:, None] * Y
            G = torch.cat([c.real, c.imag], 1) @ Qr[k][:, lo:hi + pt.n_t]
            L = L + torch.gather(G, 1, (st - lo)[:, None] + j[None])
            q = q + (fp * fp + fx * fx) * (Y.conj() * (Y @ U[k].T)).sum(1).real \
                + (Fk * Fk * (Y * (Y @ V[k].T)).sum(1)).real
        out.append(torch.logsumexp(L, 1) - math.log(pt.n_t) - 0.25 * kap * kap * q)
    return torch.cat(out).cpu().numpy()


def _reduce(lnL, lw):
    w = lnL + lw
    M = w.max()
    e = np.exp(w - M)
    s1, s2, n = math.fsum(e), math.fsum(e * e), w.size
    return [M + math.log(s1) - math.log(n), s1, s1 * s1 / s2,
            math.sqrt(max(0.0, s2 / (s1 * s1) - 1.0 / n)), lnL.max(), float(n)]


_FIELDS = ["ln_L_marg", "n_eff", "n_eff_kish", "sigma_ln_L", "max_ln_L"]


def _as_result(r):
    return dict(zip(_FIELDS, map(float, r)), n_samples=int(r[5]))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("integrate", "evaluate", "harvest", "surrogate"):
        rng, pt, s, lp, lq = _eval_inputs(case, seed)
        rom = None
        if kind == "surrogate":
            lam, A = _rom_inputs(case, rng)
            s, rom = np.concatenate([s, lam[None]]), (MODES[:case["n_lm"]], A)
        lnL = _lnl(pt, s, rom)
        if kind == "evaluate":
            return lnL
        r = _reduce(lnL, lp - lq)
        if kind == "integrate" and case["entry"] == "host":
            return _as_result(r)
        r = np.array(r)
        # the picks are decided by comparisons, not computed
        return r if kind != "harvest" else dict(idx=None, bin=None, theta=None, result=r)
    if kind == "batch":
        pts, S, LP, LQ = _batch_inputs(case, seed)
        return [_as_result(_reduce(_lnl(p, S[i]), LP[i] - LQ[i])) for i, p in enumerate(pts)]
    if kind == "build":
        f = _fd_inputs(case, seed)
        n, fr = case["n_q"], np.abs(f["f"])
        w = np.where((fr > f["f_min"]) & (fr < f["f_max"]), 2 * f["df"] / f["psd"], 0.0)
        g = w * f["d"] * np.exp(2j * np.pi * f["f"] * f["t0"])
        Q = np.fft.ifft(f["h"].conj()[None] * g[:, None], axis=2) * n
        hm = f["h"][:, (-np.arange(n)) % n]
        U = np.stack([(f["h"].conj() * x) @ f["h"].T for x in w])
        V = np.stack([(hm * x) @ f["h"].T for x in w])
        return dict(Q=Q, U=U, V=V)
    # draws and training follow the library's own counter-based streams and
    # its network in 16-bit operands; the adaptive run follows its own draws
    return None
