"""Workloads of the library as its users run them, for timing and comparison.

A case is a dict of plain values.  ``prepare`` builds what a program holds
before the call (lattice plans, a bound batch, device tensors), ``run`` makes
one pass through the public entry points and returns its whole outputs.

Kinds:
  chain     one replica, block layout: single runs and the double-precision
            validation mode
  replicas  many replicas of one simple-cubic lattice at a ladder of
            temperatures (replica layout)
  ball      field sweep of the core/shell particle, many seeds
  phases    the particle with an update policy per magnetic phase, its
            per-phase magnetisation after every MCS and its step-end states
  films     diluted films of different sizes, one replica each (site layout)
  gradient  energies and all their gradients for a batch of configurations
  response  derivatives of a thermal average from step-end states
  thermal   thermal averages, reweighting and correlation times of a history
  multihist the multiple-histogram method over a history
Sizes are those of the tests and of bench.py, or lie between them.
"""
import numpy as np
import torch

import synth
from paper_1803_07030_amd import hsim
from paper_1803_07030_amd.energy import fluct_gradients, heisenberg_energy, spins_planar

DEV = "cuda"


def listed():
    return [
        # the double-precision validation run: SC 8^3 cooled through 20
        # temperatures; one replica, so latency is all there is
        dict(name="chain_sc8_f64", kind="chain", L=8, f64=True, steps=20, mcs=25, ani=False),
        # a short equilibration of a small sample, the kind that finite-size
        # scaling repeats by the hundred; odd edge, so more than two colours
        dict(name="replicas_sc15_r24", kind="replicas", L=15, R=24, steps=1, mcs=100, T_lo=0.8, T_hi=2.2),
        # the headline workload of bench.py, a stretch of 200 MCS
        dict(name="replicas_sc64_r64", kind="replicas", L=64, R=64, steps=1, mcs=200, T_lo=0.1, T_hi=3.0),
        # a sample whose spins exceed the last-level cache
        dict(name="replicas_sc80_r64", kind="replicas", L=80, R=64, steps=1, mcs=40, T_lo=0.1, T_hi=3.0),
        # the hysteresis loop of bench.py's ball workload, five of its field steps
        dict(name="ball20_r32_hysteresis", kind="ball", Rad=20, R=32, steps=5, mcs=60),
        # the paper's feature list: an update policy and a magnetisation
        # record per magnetic phase, and the final state of every step
        dict(name="phases_ball10_r32", kind="phases", Rad=10, R=32, steps=2, mcs=50),
        # the diluted films of bench.py's films workload, 64 of the 256
        dict(name="films64", kind="films", n=64, Lmin=16, Lmax=128, mcs=100),
        # one gradient step of a model with per-bond constants, through the
        # C interface as bench.py's energy workload calls it
        dict(name="gradient_sc32_b1024_f32", kind="gradient", L=32, batch=1024, f64=False, autograd=False),
        # the same through autograd in double precision at a test's size
        dict(name="gradient_sc9_b8_f64", kind="gradient", L=9, batch=8, f64=True, autograd=True),
        # response functions of a film (ragged rows) from its sampled states
        dict(name="response_film61_c75_f32", kind="response", L=61, d=5, cfg=75, f64=False, energy=True),
        # the analysis of the headline workload's history
        dict(name="thermal_r64_m10000", kind="thermal", R=64, steps=1, mcs=10000, m0=1000, evals=3),
        # free energies of a temperature ladder and an interpolated curve
        dict(name="multihist_k16_m2000", kind="multihist", K=16, mcs=2200, m0=200, evals=41),
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "replicas", "replicas", "ball", "phases", "films", "gradient", "gradient",
                       "response", "thermal", "multihist"])
    if kind == "chain":
        f64 = rng.random() < 0.6
        return dict(kind=kind, L=rng.randint(4, 16 if f64 else 22), f64=f64, steps=rng.choice([1, 3, 8]),
                    mcs=rng.randint(5, 40), ani=rng.random() < 0.5)
    if kind == "replicas":
        L, R = _log(rng, 6, 72), rng.choice([16, 24, 32, 40, 64, 64, 100])
        # keep the work at or below the headline case's
        mcs = max(10, min(300, int(2.0e9 / (L ** 3 * R))))
        lo = rng.uniform(0.1, 1.0)
        return dict(kind=kind, L=L, R=R, steps=rng.choice([1, 2]), mcs=mcs, T_lo=lo, T_hi=lo + rng.uniform(0.5, 2.0))
    if kind == "ball":
        return dict(kind=kind, Rad=rng.randint(6, 20), R=rng.choice([16, 24, 32, 48, 64]), steps=rng.randint(2, 5),
                    mcs=rng.randint(20, 60))
    if kind == "phases":
        return dict(kind=kind, Rad=rng.randint(5, 16), R=rng.choice([16, 20, 32, 64]), steps=rng.randint(1, 3),
                    mcs=rng.randint(10, 50))
    if kind == "films":
        return dict(kind=kind, n=_log(rng, 3, 48), Lmin=16, Lmax=_log(rng, 24, 128), mcs=rng.randint(20, 100))
    if kind == "gradient":
        L = _log(rng, 5, 32)
        f64 = rng.random() < 0.4
        # at most the listed batch's bytes
        top = min(1024, int(1024 * 32 ** 3 / (L ** 3 * (2 if f64 else 1))))
        return dict(kind=kind, L=L, batch=_log(rng, 1, top), f64=f64, autograd=rng.random() < 0.5)
    if kind == "response":
        return dict(kind=kind, L=rng.randint(16, 90), d=rng.randint(2, 8), cfg=_log(rng, 16, 200),
                    f64=rng.random() < 0.3, energy=rng.random() < 0.5)
    if kind == "thermal":
        mcs = _log(rng, 600, 10000)
        return dict(kind=kind, R=_log(rng, 1, 64), steps=rng.choice([1, 1, 4]) if mcs < 3000 else 1, mcs=mcs,
                    m0=mcs // 10, evals=rng.choice([1, 3, 5]))
    mcs = _log(rng, 400, 2200)
    return dict(kind=kind, K=rng.randint(2, 16), mcs=mcs, m0=mcs // 11, evals=rng.choice([1, 5, 41]))


# ------------------------------------------------------------------ lattices
def _film_shapes(case):
    """Edge and thickness of every film, the same for every seed."""
    n, lo, hi = case["n"], case["Lmin"], case["Lmax"]
    u = synth.uniform01(3, 2 * n, tag=31)
    Ls = lo + np.minimum((u[0::2] * (hi - lo + 1)).astype(int), hi - lo)
    ds = 2 + np.minimum((u[1::2] * 9).astype(int), 8)
    return [(int(a), int(b)) for a, b in zip(Ls, ds)]


def _ball(case):
    return synth.core_shell_ball(R=case["Rad"], Rc=max(2, (4 * case["Rad"]) // 5))


def _ball_sites(rad):
    r = np.arange(-rad, rad + 1) ** 2
    return int((r[:, None, None] + r[None, :, None] + r[None, None, :] <= rad * rad).sum())


def _sites(case):
    """Sites (over all replicas) of a sweep case and their mean degree."""
    k = case["kind"]
    if k == "chain":
        return case["L"] ** 3, 6.0
    if k == "replicas":
        return case["L"] ** 3 * case["R"], 6.0
    if k in ("ball", "phases"):
        return _ball_sites(case["Rad"]) * case["R"], 5.8
    return int(0.9 * sum(L * L * d for L, d in _film_shapes(case))), 5.1


# ------------------------------------------------------------------- prepare
def _sweep_state(plans, batch, steps, mcs, T, B, init):
    batch.bind(steps, mcs)
    return dict(plans=plans, batch=batch, T=T, B=B, init=init)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "chain":
        lat = synth.sc_periodic(case["L"])
        if case["ani"]:
            lat.k = 0.3 * synth.uniform01(seed, lat.n, tag=1)
            lat.axis = synth.unit_vectors(seed, lat.n, tag=2)
        plan = hsim.Plan(lat)
        b = hsim.Batch([plan], seed=seed, precision=hsim.FP64_EXACT if case["f64"] else hsim.FP32)
        T = synth.cooling_schedule(max(case["steps"], 2))[:case["steps"]]
        return _sweep_state([plan], b, case["steps"], case["mcs"], T, 0.0, hsim.INIT_RANDOM)
    if kind == "replicas":
        lat = synth.sc_periodic(case["L"])
        lat.k = np.full(lat.n, 0.1)
        plan = hsim.Plan(lat)
        b = hsim.Batch([plan] * case["R"], seed=seed)
        T = synth.replica_temperatures(case["R"], case["T_lo"], case["T_hi"])
        T = T[:, None] * np.ones((1, case["steps"]))
        return _sweep_state([plan], b, case["steps"], case["mcs"], T, 0.0, hsim.INIT_COLD_Z)
    if kind == "ball":
        plan = hsim.Plan(_ball(case))
        b = hsim.Batch([plan] * case["R"], seed=seed)
        return _sweep_state([plan], b, case["steps"], case["mcs"], np.full(case["steps"], 0.1),
                            synth.hysteresis_fields(401)[200:200 + case["steps"]], hsim.INIT_COLD_Z)
    if kind == "phases":
        lat = _ball(case)
        plan = hsim.Plan(lat)
        plan.set_types(lat.site_type)
        b = hsim.Batch([plan] * case["R"], seed=seed)
        T = synth.replica_temperatures(case["R"], 0.1, 1.5)[:, None] * np.ones((1, case["steps"]))
        st = _sweep_state([plan], b, case["steps"], case["mcs"], T,
                          np.linspace(0.2, -0.2, case["steps"]), hsim.INIT_COLD_Z)
        b.set_policies([(hsim.POLICY_SMALL_STEP, np.pi / 6), (hsim.POLICY_RANDOM, 0.0), (hsim.POLICY_ADAPTIVE, 0.5)])
        b.bind_outputs(type_mag_types=3, snapshots=True)
        return st
    if kind == "films":
        plans = []                       # the same films for every seed, exchange scaled by it
        for f, ((L, d), s) in enumerate(zip(_film_shapes(case), synth.uniform01(seed, case["n"], tag=33))):
            lat = synth.diluted_film(L, d, seed=3000 + f)
            lat.J = lat.J * (0.9 + 0.2 * s)
            plans.append(hsim.Plan(lat))
        T = (0.2 + 1.8 * synth.uniform01(3, case["n"], tag=32))[:, None]
        b = hsim.Batch(plans, seed=seed)
        return _sweep_state(plans, b, 1, case["mcs"], T, 0.0, hsim.INIT_COLD_Z)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    if kind == "gradient":
        dt = torch.float64 if case["f64"] else torch.float32
        lat = synth.gradient_lattice(L=case["L"], seed=seed)
        plan = hsim.Plan(lat)
        S = torch.randn(case["batch"], 3, lat.n, generator=gen, device=DEV, dtype=dt)
        S /= S.norm(dim=1, keepdim=True)
        J = torch.tensor(lat.bonds()[2], dtype=dt, device=DEV)
        k = torch.tensor(lat.k, dtype=dt, device=DEV)
        axis = torch.tensor(lat.axis.T.copy(), dtype=dt, device=DEV)
        gE = torch.rand(case["batch"], generator=gen, device=DEV, dtype=torch.float64) + 0.5
        st = dict(plan=plan, lat=lat, S=S, J=J, k=k, axis=axis, gE=gE)
        if case["autograd"]:
            st["B"] = torch.tensor(0.5, dtype=torch.float64, device=DEV, requires_grad=True)
            for q in (S, J, k):
                q.requires_grad_(True)
        else:
            st["B"] = 0.5
            hsim.hsim_energy_prepare(plan.handle)
        return st
    if kind == "response":
        dt = torch.float64 if case["f64"] else torch.float32
        lat = synth.diluted_film(case["L"], case["d"], seed=12)
        plan = hsim.Plan(lat)
        # step-end states as a run leaves them: mostly ordered along +z
        snap = 0.3 * torch.randn(case["cfg"], lat.n, 3, generator=gen, device=DEV, dtype=torch.float64)
        snap[..., 2] += 1.0
        snap /= snap.norm(dim=2, keepdim=True)
        J = 0.5 + torch.rand(lat.n_bonds, generator=gen, device=DEV, dtype=dt)
        k = torch.tensor(lat.k, dtype=dt, device=DEV)
        axis = torch.tensor(lat.axis.T.copy(), dtype=dt, device=DEV)
        O = None if case["energy"] else snap[..., 2].sum(dim=1)
        return dict(plan=plan, lat=lat, snap=snap, J=J, k=k, axis=axis, B=0.3, beta=1.0, O=O, dt=dt)
    if kind == "thermal":
        h, beta = _history(case["R"], case["steps"], case["mcs"], seed, 4096)
        ev = beta[..., None] * np.linspace(0.98, 1.02, case["evals"]) if case["evals"] > 1 else None
        return dict(h=h, m0=case["m0"], N=4096, beta=beta, ev=ev)
    h, beta = _history(case["K"], 1, case["mcs"], seed, 512)
    series = np.stack([np.arange(case["K"]), np.zeros(case["K"], int)], axis=1)
    return dict(h=h, m0=case["m0"], N=512, beta_k=beta[:, 0], series=series,
                ev=np.linspace(beta.min(), beta.max(), case["evals"]))


def _history(R, S, M, seed, N):
    """History [R][S][M][5] of correlated samples: E normal with mean
    -beta N s^2 and variance N s^2 (a Gaussian density of states, so that
    neighbouring temperatures overlap and reweighting holds), |M| following
    E, both first-order autoregressive with correlation times from 2 to 40
    MCS.  Returns the device tensor and beta [R][S]."""
    rng = np.random.default_rng(seed)
    T = R * S
    beta = 0.4 + (0.8 / np.sqrt(N)) * np.arange(T)
    tau = np.exp(np.linspace(np.log(2.0), np.log(40.0), T))
    phi = np.exp(-1.0 / tau)
    x = rng.standard_normal((M, T, 4))
    amp = np.sqrt(1.0 - phi * phi)
    for m in range(1, M):
        x[m] = phi[:, None] * x[m - 1] + amp[:, None] * x[m]
    h = np.zeros((T, M, 5))
    h[..., 0] = (-beta * N + np.sqrt(N) * x[..., 0]).T
    mz = 0.3 * N + np.sqrt(N) * (x[..., 3] - 0.5 * x[..., 0])
    h[..., 1], h[..., 2], h[..., 3] = np.sqrt(N) * x[..., 1].T, np.sqrt(N) * x[..., 2].T, mz.T
    h[..., 4] = np.floor(0.4 * N + np.sqrt(N) * rng.standard_normal((T, M)))
    return torch.tensor(h.reshape(R, S, M, 5), device=DEV), beta.reshape(R, S)


# ----------------------------------------------------------------------- run
def run(st):
    if "batch" in st:
        b = st["batch"]
        b.init_spins(st["init"])
        b.run(st["T"], st["B"])
        out = dict(history=b.history)
        if getattr(b, "snapshots", None) is not None:
            out.update(type_mag=b.type_mag, snapshots=b.snapshots)
        else:
            out["spins"] = torch.cat([b.spins_user(r) for r in range(b.R)])
        return out
    if "gE" in st:
        plan, S, J, k, axis, B, gE = (st[q] for q in ("plan", "S", "J", "k", "axis", "B", "gE"))
        if isinstance(B, torch.Tensor):
            E = heisenberg_energy(S, J, k, B, plan, axis)
            gS, gJ, gk, gB = torch.autograd.grad(E, (S, J, k, B), gE)
            return dict(E=E.detach(), gS=gS, gJ=gJ, gk=gk, gB=gB)
        prec = hsim.FP64_EXACT if S.dtype == torch.float64 else hsim.FP32
        E, gB = torch.empty_like(gE), gE.new_empty(1)
        gS, gJ, gk = torch.empty_like(S), torch.empty_like(J), torch.empty_like(k)
        hsim.hsim_energy_forward(plan.handle, len(gE), prec, S, J, k, axis, B, None, E)
        hsim.hsim_energy_backward(plan.handle, len(gE), prec, S, J, k, axis, B, None, gE, gS, gJ, gk, gB)
        return dict(E=E, gS=gS, gJ=gJ, gk=gk, gB=gB)
    if "snap" in st:
        cfg = spins_planar(st["snap"], st["dt"])
        gJ, gk, gB, O = fluct_gradients(st["plan"], cfg, st["J"], st["k"], st["axis"], st["B"], st["beta"],
                                        O=st["O"])
        return dict(cfg=cfg, gJ=gJ, gk=gk, gB=gB, O=O)
    if "series" in st:
        f, it, out = hsim.hsim_analysis_multihist(st["h"], st["m0"], st["N"], st["series"], st["beta_k"], st["ev"])
        return dict(f=f, iterations=it, thermal=out)
    th = hsim.hsim_analysis_thermal(st["h"], st["m0"], st["N"], st["beta"], st["ev"])
    tau_e, win_e = hsim.hsim_analysis_tau(st["h"], st["m0"], 0)
    tau_m, win_m = hsim.hsim_analysis_tau(st["h"], st["m0"], 1)
    return dict(thermal=th, tau_e=tau_e, win_e=win_e, tau_m=tau_m, win_m=win_m)


# ---------------------------------------------------------------------- work
def work(case):
    """Bytes and operations one pass cannot do without."""
    kind = case["kind"]
    if kind in ("chain", "replicas", "ball", "phases", "films"):
        n, z = _sites(case)
        mcs = case.get("steps", 1) * case["mcs"]
        el = 8 if case.get("f64") else 4
        reps = case["n"] if kind == "films" else case.get("R", 1)
        table = (n if kind == "films" else n / reps) * (4 + (4 + el) * z)
        io = 5 * 8 * reps * mcs + 24 * n + table          # history, final states, lattice
        # a spin set beyond what the chip's registers and LDS hold is read
        # and written by every MCS, the films' own lattice tables read
        state = 3 * el * n
        if state > 100e6:
            io += mcs * 2 * state
        if kind == "films" and state + table > 100e6:
            io += mcs * table
        if kind == "phases":
            io += 3 * 3 * 8 * reps * mcs + 24 * n * case["steps"]
        # random words (about 60), trial point (25), field (6 per neighbour),
        # energy change and acceptance (25)
        return dict(bytes=io, flops=mcs * n * (110 + 6 * z))
    if kind == "gradient":
        n, b, el = case["L"] ** 3, case["batch"], 8 if case["f64"] else 4
        # the forward's read, the backward's read and its write; lattice tables and gradients once
        return dict(bytes=9 * el * n * b + n * (48 + 12 * el), flops=b * n * (40 + 75))
    if kind == "response":
        n, b, el = int(0.9 * case["L"] ** 2 * case["d"]), case["cfg"], 8 if case["f64"] else 4
        passes = 2 if case["energy"] else 1
        return dict(bytes=n * b * (24 + 3 * el * (1 + passes)) + n * (40 + 12 * el), flops=b * n * (40 * passes + 40))
    s = case.get("R", case.get("K")) * case.get("steps", 1)
    n = case["mcs"] - case["m0"]
    if kind == "thermal":
        # two passes of moments per evaluation; about 100 lags per series and observable
        return dict(bytes=32.0 * s * n, flops=s * n * (case["evals"] * 60 + 2 * 2 * 100))
    # some 200 iterations, two exponentials (about 20 operations) per sample and series
    return dict(bytes=32.0 * s * n, flops=200.0 * 2 * 20 * s * s * n)


# --------------------------------------------------------------------- exact
def exact(case, seed):
    """run()'s values in 64 bits, without the library's kernels; None for a
    Markov chain, whose single-precision trajectory has no such value."""
    kind = case["kind"]
    if kind not in ("gradient", "response", "thermal", "multihist"):
        return None
    st = prepare(case, seed)
    if kind == "gradient":
        w = st["gE"]
        E, gS, gJ, gk, gB = _energy_grad(st["lat"], st["S"].detach(), st["J"].detach(), st["k"].detach(), st["axis"],
                                         0.5, w, True)
        return dict(E=E, gS=gS, gJ=gJ, gk=gk, gB=gB if case["autograd"] else gB.reshape(1))
    if kind == "response":
        cfg = st["snap"].transpose(1, 2).contiguous()
        E, _, _, _, _ = _energy_grad(st["lat"], cfg, st["J"], st["k"], st["axis"], st["B"], None, False)
        O, c = (E, 1.0) if case["energy"] else (st["O"], 0.0)
        w = (c - st["beta"] * (O - O.mean())) / len(O)
        _, _, gJ, gk, gB = _energy_grad(st["lat"], cfg, st["J"], st["k"], st["axis"], st["B"], w, False)
        return dict(cfg=cfg, gJ=gJ, gk=gk, gB=gB.reshape(1), O=O)
    h = st["h"][:, :, st["m0"]:]
    E, A = h[..., 0], torch.linalg.vector_norm(h[..., 1:4], dim=-1)
    if kind == "thermal":
        beta = torch.tensor(st["beta"], device=DEV)
        ev = beta[..., None] if st["ev"] is None else torch.tensor(st["ev"], device=DEV)
        th = _thermal(E[:, :, None], A[:, :, None], -(ev - beta[..., None])[..., None] * E[:, :, None], ev, st["N"])
        tau_e, win_e = _tau(E)
        tau_m, win_m = _tau(A)
        return dict(thermal=th, tau_e=tau_e, win_e=win_e, tau_m=tau_m, win_m=win_m)
    bk = torch.tensor(st["beta_k"], device=DEV)
    e, a = E.reshape(-1), A.reshape(-1)
    ln_n = float(np.log(E.shape[-1]))
    f = torch.zeros_like(bk)
    for _ in range(5000):
        logd = torch.logsumexp(ln_n + f - bk * e[:, None], dim=1)
        fn = -torch.logsumexp(-bk[:, None] * e - logd, dim=1)
        fn = fn - fn[0]
        done = float((fn - f).abs().max()) < 1e-11
        f = fn
        if done:
            break
    logd = torch.logsumexp(ln_n + f - bk * e[:, None], dim=1)
    ev = torch.tensor(st["ev"], device=DEV)
    return dict(f=f, iterations=None, thermal=_thermal(e, a, -ev[:, None] * e - logd, ev, st["N"]))


def _energy_grad(lat, S, J, k, axis, B, w, want_s):
    """Energies [batch], and for weights w the gradients of sum w E."""
    i, j, _ = (torch.tensor(np.asarray(v), device=DEV) for v in lat.bonds())
    J, k, axis = J.double(), k.double(), axis.double()
    nb, E = S.shape[0], []
    gS = torch.empty(S.shape, dtype=torch.float64, device=DEV) if want_s else None
    gJ, gk = torch.zeros_like(J), torch.zeros_like(k)
    gB = torch.zeros((), dtype=torch.float64, device=DEV)
    for c0 in range(0, nb, 64):                            # slices of the batch, to bound memory
        s = S[c0:c0 + 64].double()
        a = (s * axis).sum(1)
        dots = (s[:, :, i] * s[:, :, j]).sum(1)
        E.append(-(dots * J).sum(1) - B * s[:, 2].sum(1) - (k * a * a).sum(1))
        if w is None:
            continue
        wc = w[c0:c0 + 64, None]
        gJ -= (wc * dots).sum(0)
        gk -= (wc * a * a).sum(0)
        gB -= (wc[:, 0] * s[:, 2].sum(1)).sum()
        if want_s:
            g = torch.zeros_like(s)
            g.index_add_(2, i, -J * s[:, :, j])
            g.index_add_(2, j, -J * s[:, :, i])
            g[:, 2] -= B
            g -= 2.0 * (k * a)[:, None] * axis
            gS[c0:c0 + 64] = wc[:, None] * g
    return torch.cat(E), gS, gJ, gk, gB


def _thermal(E, A, logw, beta, N):
    w = torch.exp(logw - logw.max(dim=-1, keepdim=True).values)
    w = w / w.sum(dim=-1, keepdim=True)
    mean = lambda x: (w * x).sum(dim=-1)                   # noqa: E731
    mE, mA, mA2, mA4 = mean(E), mean(A), mean(A ** 2), mean(A ** 4)
    dE, dA, dA2 = E - mE[..., None], A - mA[..., None], A ** 2 - mA2[..., None]
    m2, m4 = mA2 / N ** 2, mA4 / N ** 4
    return torch.stack([mE / N, mA / N, m2, m4, beta ** 2 * mean(dE * dE) / N, beta * mean(dA * dA) / N,
                        1.0 - m4 / (3.0 * m2 * m2), -mean(dA * dE) / mA, -mean(dA2 * dE) / mA2], dim=-1)


def _tau(x, c=6.0):
    n = x.shape[-1]
    d = x - x.mean(dim=-1, keepdim=True)
    p = torch.fft.rfft(d, n=2 * n)                         # linear autocovariance by zero padding
    cov = torch.fft.irfft(p * p.conj(), n=2 * n)[..., :n] / (n - torch.arange(n, device=DEV))
    rho = (cov[..., 1:n // 2 + 1] / cov[..., :1]).cpu().numpy()
    tau, win = np.empty(x.shape[:-1]), np.empty(x.shape[:-1], dtype=np.int32)
    for at in np.ndindex(*x.shape[:-1]):
        t = 0.5 + np.cumsum(rho[at])
        past = np.nonzero(np.arange(1, t.size + 1) >= c * t)[0]
        u = int(past[0]) if past.size else t.size - 1
        tau[at], win[at] = t[u], u + 1
    return torch.tensor(tau), torch.tensor(win)
