"""The work that users of this framework have it do, as cases to be timed.

A case is a dict of plain values.  `prepare` makes what a filter program has in
hand before the call (ensemble, noise, observations, workspaces), `run` is one
pass through the public entry points of `paper_2402_06927_amd.sch`, `work` is
what the path cannot do without, and `exact` gives the same outputs from plain
torch in 64 bits: a periodic tridiagonal solve by cyclic reduction, constant
coefficient operators by FFT, Philox in integer arithmetic.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2402_06927_amd import sch
from paper_2402_06927_amd import workloads as W

DEV = "cuda"
F64 = torch.float64
SEED = W.MASTER_SEED
# physics shared by the workloads (paper_2402_06927_amd/workloads.py)
L, ALPHA, MU, DT, AMP = 40.0, 1.0, 0.01, 0.025, 0.05
KAPPA, ETA, KSOLVES = 1.0, 1.0, 3
PICARD_TOL = 1e-13
TAG_FORECAST, TAG_PCN, TAG_ACCEPT, TAG_RESAMPLE = 1, 2, 3, 4


# --------------------------------------------------------------------------- the cases
def listed():
    return [
        # The smallest calls: one bootstrap cycle of the 256-node filter, where the
        # launches and the read-back of the ESS count as much as the kernels.
        dict(name="bootstrap_256", kind="bootstrap", nx=256, n=32, steps=20, modes=4, n_obs=40,
             sigma=0.05, threads=0),
        # The paper's experiment 1: one tempered + jittered assimilation step on 100
        # nodes with 150 particles and the Matern-type noise.
        dict(name="paper_tempered_100", kind="paper", nx=100, n=150, steps=5, n_obs=80,
             sigma=math.sqrt(0.5), n_jitter=5),
        # The forecast of the headline filter, on the tile its autotuner picks.
        dict(name="forecast_4096", kind="forecast", nx=4096, n=1024, steps=40, modes=8, matern=False,
             threads=256),
        # A forecast on a grid that no tile divides, without tuning.
        dict(name="forecast_ragged_1500", kind="forecast", nx=1500, n=700, steps=20, modes=4,
             matern=False, threads=0),
        # The headline filter's jitter: five pCN moves, each a rerun of the window.
        dict(name="jitter_4096", kind="jitter", nx=4096, n=1024, steps=40, modes=8, matern=False,
             n_obs=256, sigma=0.02, n_jitter=5, rho=0.99, threads=256),
        # The same with the paper's noise: one increment per cell and step.
        dict(name="jitter_matern_4096", kind="jitter", nx=4096, n=1024, steps=40, modes=8,
             matern=True, n_obs=256, sigma=0.02, n_jitter=5, rho=0.99, threads=256),
        # The backward direction: objective and adjoint gradient of nudging.
        dict(name="nudge_grad_2048", kind="grad", nx=2048, n=2048, steps=40, modes=8, n_obs=256,
             sigma=0.02, ckpt=8, threads=0),
        # Gradient-based jitter (pCN-Langevin moves) on a ragged grid.
        dict(name="pcnl_ragged_1000", kind="pcnl", nx=1000, n=300, steps=10, modes=4, n_obs=100,
             sigma=0.05, n_jitter=2, rho=0.99, ckpt=4, threads=0),
        # Many filters of uneven sizes advanced together (one graph replay a cycle).
        dict(name="batch_uneven_16", kind="batch", n_inst=16, steps=20, modes=4, n_obs=100,
             sigma=0.05, n_max=1024, layout=SEED),
        # The weights of one tempering step: bisection, resampling, gather of the rows.
        dict(name="reweight_2048", kind="reweight", nx=2048, n=2048, n_bisect=50, scale=50.0),
        # The warm-start network: inference of an ensemble, and one training step.
        dict(name="network_forward_4096", kind="forward", batch=4096, n_in=4352, hidden=256,
             n_out=320),
        dict(name="network_train_1024", kind="train", batch=1024, n_in=4352, hidden=256, n_out=320),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _particles(rng, nx, lo, hi, nodes):
    """Particles, log-uniform, at most `nodes` grid nodes in all."""
    return max(lo, min(_log(rng, lo, hi), nodes // nx))


def draw(rng):
    kind = rng.choice(["bootstrap", "paper", "forecast", "forecast", "jitter", "jitter", "grad",
                       "pcnl", "batch", "reweight", "forward", "train"])
    modes, n_obs = rng.randint(1, 8), _log(rng, 20, 256)
    if kind == "bootstrap":
        nx = _log(rng, 64, 2048)
        return dict(kind=kind, nx=nx, n=_particles(rng, nx, 8, 1024, 1 << 18),
                    steps=rng.randint(5, 40), modes=modes, n_obs=min(n_obs, nx), sigma=0.05, threads=0)
    if kind == "paper":
        nx = _log(rng, 64, 256)
        return dict(kind=kind, nx=nx, n=_log(rng, 50, 400), steps=rng.randint(2, 8),
                    n_obs=min(n_obs, nx), sigma=math.sqrt(0.5), n_jitter=rng.randint(1, 5))
    if kind == "forecast":
        nx = _log(rng, 64, 8192)
        return dict(kind=kind, nx=nx, n=_particles(rng, nx, 16, 4096, 1 << 21),
                    steps=rng.randint(5, 40), modes=modes, matern=rng.random() < 0.4, threads=0)
    if kind == "jitter":
        nx = _log(rng, 64, 8192)
        return dict(kind=kind, nx=nx, n=_particles(rng, nx, 16, 2048, 1 << 20),
                    steps=rng.randint(5, 40), modes=modes, matern=rng.random() < 0.4,
                    n_obs=min(n_obs, nx), sigma=0.02, n_jitter=rng.randint(1, 5),
                    rho=rng.choice([0.86, 0.99]), threads=0)
    if kind == "grad":
        nx = _log(rng, 64, 4096)
        return dict(kind=kind, nx=nx, n=_particles(rng, nx, 16, 2048, 1 << 21),
                    steps=rng.randint(5, 40), modes=modes, n_obs=min(n_obs, nx), sigma=0.02,
                    ckpt=rng.choice([4, 8]), threads=0)
    if kind == "pcnl":
        nx = _log(rng, 64, 2048)
        return dict(kind=kind, nx=nx, n=_particles(rng, nx, 16, 1024, 1 << 19),
                    steps=rng.randint(4, 20), modes=modes, n_obs=min(n_obs, nx), sigma=0.05,
                    n_jitter=rng.randint(1, 3), rho=0.99, ckpt=rng.choice([4, 8]), threads=0)
    if kind == "batch":
        return dict(kind=kind, n_inst=rng.randint(3, 16), steps=rng.randint(5, 20), modes=modes,
                    n_obs=n_obs, sigma=0.05, n_max=512, layout=rng.randrange(1 << 20))
    if kind == "reweight":
        nx = _log(rng, 64, 4096)
        return dict(kind=kind, nx=nx, n=_particles(rng, nx, 100, 8192, 1 << 22), n_bisect=50,
                    scale=50.0)
    widths = dict(n_in=8 * _log(rng, 32, 544), hidden=rng.choice([64, 96, 256]),
                  n_out=_log(rng, 20, 320))
    return dict(kind=kind, batch=_log(rng, 64, 4096 if kind == "forward" else 1024), **widths)


# --------------------------------------------------------------------------- inputs
def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed(1000 * int(seed) + stream)


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=F64)


def _axis(nx):
    return torch.arange(nx, device=DEV, dtype=F64)


def _symbol(nx, diag, off):
    """Eigenvalues of the circulant (off, diag, off)."""
    th = 2.0 * math.pi * torch.arange(nx // 2 + 1, device=DEV, dtype=F64) / nx
    return diag + 2.0 * off * torch.cos(th)


def _apply(v, ratio):
    return torch.fft.irfft(torch.fft.rfft(v) * ratio, n=v.shape[-1])


def _ops(nx, alpha=ALPHA):
    """Eigenvalues of M and of M + alpha^2 K."""
    h = L / nx
    return (_symbol(nx, 2 * h / 3, h / 6),
            _symbol(nx, 2 * h / 3 + 2 * alpha**2 / h, h / 6 - alpha**2 / h))


def _velocity(nx, n, g):
    """0.2 sech^2((x - L/2)/2) plus a smooth perturbation of pointwise variance 0.01."""
    x = _axis(nx) * (L / nx)
    u = (0.2 / torch.cosh((x - 0.5 * L) / 2.0) ** 2).expand(n, nx).clone()
    coef = _normal(g, n, 8) * math.sqrt(0.01 / 4.0)
    for k in range(4):
        arg = 2.0 * math.pi * (k + 1) * x / L
        u += coef[:, 2 * k:2 * k + 1] * torch.cos(arg) + coef[:, 2 * k + 1:2 * k + 2] * torch.sin(arg)
    return u


def _paper_velocity(nx, n, g):
    """The paper's initial velocities: alpha^2 U + beta^2, U the smoothed |white noise|."""
    h = L / nx
    cells = (_normal(g, n, nx) * math.sqrt(h)).abs()
    U = _matern(cells, nx, 1.0, math.sqrt(h), 3)
    ab = _normal(g, n, 2)
    return ab[:, :1] ** 2 * U + ab[:, 1:] ** 2


def _modes(nx, q):
    return torch.tensor(W.mode_table(L, nx, q, AMP), device=DEV)


def _observe(u, n_obs):
    nx = u.shape[-1]
    num = torch.arange(n_obs, device=DEV) * nx
    e = num // n_obs
    r = (num % n_obs).to(F64) / n_obs
    return (1.0 - r) * u[..., e] + r * u[..., (e + 1) % nx]


def _ensemble(case, seed):
    """(u, m, y, sigma): the ensemble at the window's start and the observations of a
    truth drawn from the same prior."""
    nx, n = case["nx"], case["n"]
    make = _paper_velocity if case["kind"] == "paper" else _velocity
    u = make(nx, n, _gen(seed, 0))
    fm, fh = _ops(nx)
    m = _apply(u, fh / fm)
    y = sig = None
    if "n_obs" in case:
        truth = make(nx, 1, _gen(seed, 1))[0]
        sig = torch.full((case["n_obs"],), case["sigma"], device=DEV, dtype=F64)
        y = _observe(truth, case["n_obs"]) + sig * _normal(_gen(seed, 2), case["n_obs"])
    return u, m, y, sig


def _increments(case, seed, q):
    return _normal(_gen(seed, 3), case["n"], case["steps"], q) * math.sqrt(DT)


def _sizes(case):
    """Grids, ensembles and seeds of a batch's instances."""
    return W.uneven_instances(case["n_inst"], case["layout"], np_range=(64, case["n_max"]))


def _network(case, seed):
    F, H, O = case["n_in"], case["hidden"], case["n_out"]
    g = _gen(seed, 5)

    def rnd(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)

    parts = [rnd(H * F) * math.sqrt(2.0 / F), 0.01 * rnd(H), rnd(H * H) * math.sqrt(2.0 / H),
             0.01 * rnd(H), rnd(O * H) * math.sqrt(2.0 / H), 0.01 * rnd(O)]
    X = rnd(case["batch"], F).to(torch.bfloat16)
    T = rnd(case["batch"], O)
    return torch.cat(parts), X, T


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "kind": kind}
    if kind in ("forward", "train"):
        p, X, T = _network(case, seed)
        F, H, O = case["n_in"], case["hidden"], case["n_out"]
        net = sch.Mlp(F, H, O, p, torch.empty(H * F + H * H + O * H, dtype=torch.bfloat16, device=DEV))
        sch.sch_mlp_sync(net)
        ws = torch.empty(sch.sch_mlp_workspace_bytes(net, case["batch"]), dtype=torch.uint8, device=DEV)
        st.update(net=net, X=X, T=T, ws=ws, Y=torch.empty(case["batch"], O, device=DEV),
                  loss=torch.zeros(1, dtype=F64, device=DEV), grad=torch.zeros_like(p),
                  am=torch.zeros_like(p), av=torch.zeros_like(p), step=0)
        return st
    if kind == "reweight":
        g = _gen(seed, 0)
        n = case["n"]
        phi = 0.5 * case["scale"] * (_normal(g, n, 4) ** 2).sum(1)
        one = lambda: torch.zeros(1, dtype=F64, device=DEV)  # noqa: E731
        st.update(phi=phi, theta=one(), dtheta=one(), ess=one(), u0=torch.full((1,), 0.37, dtype=F64, device=DEV),
                  w=torch.empty(n, dtype=F64, device=DEV), src=_normal(g, n, case["nx"]),
                  dst=torch.empty(n, case["nx"], dtype=F64, device=DEV),
                  idx=torch.empty(n, dtype=torch.int32, device=DEV),
                  ws=sch.workspace(sch.WS_RESAMPLE, None, n))
        return st
    if kind == "batch":
        inst = []
        for i, s in enumerate(_sizes(case)):
            c = dict(case, nx=s.nx, n=s.n_particles)
            u, m, y, sig = _ensemble(c, seed * 64 + i)
            inst.append(sch.Instance(_modes(s.nx, case["modes"]), m, u,
                                     torch.zeros(s.n_particles, dtype=F64, device=DEV),
                                     y.reshape(1, -1).contiguous(), sig, s.seed + seed))
        st["batch"] = sch.Batch(L, ALPHA, MU, DT, case["modes"], case["steps"], case["n_obs"], 0.5, inst)
        st["live"] = [x for i in inst for x in (i.m, i.u, i.logw)]
        st["start"] = [x.clone() for x in st["live"]]
        return st

    # one ensemble on one grid
    nx, n, S = case["nx"], case["n"], case["steps"]
    matern = bool(case.get("matern", kind == "paper"))
    q = case.get("modes", 1)
    model = sch.Model(L, ALPHA, MU, DT, _modes(nx, q), PICARD_TOL, 200 if kind == "paper" else 50)
    u, m, y, sig = _ensemble(case, seed)
    st.update(model=model, matern=sch.Matern(KAPPA, ETA, KSOLVES) if matern else None, seed=SEED + seed,
              threads=case.get("threads", 0), u0=u, m0=m, u=u.clone(), m=m.clone())
    if y is not None:
        st["obs"] = sch.Obs(y, sig)
    if kind == "bootstrap":
        st["logw"] = torch.zeros(n, dtype=F64, device=DEV)
        st["ws"] = sch.workspace(sch.WS_BOOTSTRAP, model, n, S)
    elif kind == "paper":
        st["ws"] = sch.matern_workspace(sch.WS_TEMPERED, model, n, S, case["n_jitter"])
    else:
        st["dW"] = _increments(case, seed, nx if matern else q)
        st["status"] = torch.zeros(n, dtype=torch.int32, device=DEV)
    if kind == "grad":
        st["dLam"] = 0.3 * _normal(_gen(seed, 4), n, S, q) * math.sqrt(DT)
        st["J"] = torch.empty(n, dtype=F64, device=DEV)
        st["grad"] = torch.empty(n, S, q, dtype=F64, device=DEV)
        st["ws"] = sch.workspace(sch.WS_NUDGE_GRAD, model, n, S, case["ckpt"])
    if kind in ("jitter", "pcnl"):
        # the forecast that the filter has made before it jitters
        st["phi"] = torch.empty(n, dtype=F64, device=DEV)
        st["acc"] = torch.zeros(n, dtype=torch.int32, device=DEV)
        st["theta"] = torch.full((1,), 0.02, dtype=F64, device=DEV)
        _tile(st)
        if matern:
            sch.sch_ensemble_step_matern(model, st["matern"], st["m"], st["u"], st["dW"])
            st["ws"] = sch.matern_workspace(sch.WS_JITTER, model, n, S, case["n_jitter"])
        else:
            sch.sch_ensemble_step(model, st["m"], st["u"], st["dW"])
            st["ws"] = (sch.workspace(sch.WS_JITTER, model, n, S, case["n_jitter"]) if kind == "jitter" else
                        sch.pcnl_workspace(sch.WS_JITTER, model, n, S, case["n_jitter"], case["ckpt"]))
        sch.sch_loglik(model, st["obs"], st["u"], st["phi"])
    return st


# --------------------------------------------------------------------------- one pass
def _tile(st):
    """The tile a tuned program has set (0: the library's own choice)."""
    if sch.sch_tune_get(sch.TUNE_THREADS) != st["threads"]:
        sch.sch_tune_set(sch.TUNE_THREADS, st["threads"])


def run(st):
    c, kind = st["case"], st["kind"]
    if kind == "forward":
        sch.sch_mlp_forward(st["net"], st["X"], st["Y"], st["ws"])
        return {"Y": st["Y"]}
    if kind == "train":
        st["step"] += 1
        sch.sch_mlp_forward(st["net"], st["X"], st["Y"], st["ws"])
        sch.sch_mlp_backward(st["net"], st["X"], st["Y"], st["T"], st["loss"], st["grad"], st["ws"])
        sch.sch_mlp_adam(st["net"], st["grad"], st["am"], st["av"], st["step"])
        return {"Y": st["Y"], "loss": st["loss"], "grad": st["grad"], "params": st["net"].params,
                "m": st["am"], "v": st["av"]}
    if kind == "reweight":
        st["theta"].zero_()
        sch.sch_temper_ess(st["phi"], st["theta"], 0.5 * c["n"], c["n_bisect"], st["dtheta"], st["w"], st["ess"])
        sch.sch_resample(st["w"], st["u0"], st["idx"], st["ws"])
        sch.sch_gather(st["idx"], st["src"], st["dst"])
        return {"w": st["w"], "dtheta": st["dtheta"], "ess": st["ess"], "idx": st["idx"], "rows": st["dst"]}
    if kind == "batch":
        torch._foreach_copy_(st["live"], st["start"])  # every pass is the first cycle
        st["batch"].run(0, 1, use_graph=True)
        r = st["batch"].read()
        return {"state": st["live"], "ess": np.array(r["ess"])}
    _tile(st)
    mt, model = st["matern"], st["model"]
    if kind in ("bootstrap", "paper", "forecast"):  # these advance the ensemble in place
        st["m"].copy_(st["m0"])
        st["u"].copy_(st["u0"])
    if kind == "bootstrap":
        st["logw"].zero_()
        s = sch.sch_pf_bootstrap_cycle(model, st["obs"], st["seed"], 3, st["m"], st["u"], st["logw"], c["steps"],
                                       0.5, st["ws"])
        return {"m": st["m"], "u": st["u"], "logw": st["logw"], "ess": s["ess"], "resampled": s["resampled"]}
    if kind == "paper":
        s = sch.sch_pf_tempered_cycle_matern(model, mt, st["obs"], st["seed"], 3, st["m"], st["u"], c["steps"],
                                             80.0 / 150.0 * c["n"], 50, W.PAPER_SHAPE.rho, c["n_jitter"], 100,
                                             st["ws"])
        return {"m": st["m"], "u": st["u"], "ess": s["ess"], "n_temper": s["n_temper"], "n_accept": s["n_accept"]}
    if kind == "forecast":
        if mt:
            sch.sch_ensemble_step_matern(model, mt, st["m"], st["u"], st["dW"], st["status"])
        else:
            sch.sch_ensemble_step(model, st["m"], st["u"], st["dW"], None, st["status"])
        return {"m": st["m"], "u": st["u"], "status": st["status"]}
    if kind == "grad":
        sch.sch_nudge_grad(model, st["obs"], st["m0"], st["u0"], st["dW"], st["dLam"], st["J"], st["grad"],
                           c["ckpt"], st["status"], st["ws"])
        return {"J": st["J"], "grad": st["grad"], "status": st["status"]}
    # jitter: the chain goes on from pass to pass
    args = (model,) + ((mt,) if mt else ()) + (st["obs"], st["seed"], 3, 1, st["m0"], st["u0"], st["dW"],
                                               st["phi"], st["m"], st["u"], st["theta"], c["rho"], c["n_jitter"])
    if kind == "pcnl":
        sch.sch_jitter_pcnl(*args, c["ckpt"], st["acc"], st["ws"])
    elif mt:
        sch.sch_jitter_pcn_matern(*args, st["acc"], st["ws"])
    else:
        sch.sch_jitter_pcn(*args, st["acc"], st["ws"])
    return {"m": st["m"], "u": st["u"], "dW": st["dW"], "phi": st["phi"], "accepted": st["acc"]}


# --------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind in ("forward", "train"):
        B, F, H, O = case["batch"], case["n_in"], case["hidden"], case["n_out"]
        macs, weights = B * (F * H + H * H + H * O), F * H + H * H + H * O
        if kind == "forward":
            return {"bytes": 2 * B * F + 2 * weights + 4 * B * O, "flops": 2 * macs}
        # forward, input errors (not of the features), weight gradients; params, m, v in and out
        return {"bytes": 2 * B * F + 8 * B * O + 4 * weights * 7 + 2 * weights * 2,
                "flops": 2 * (3 * macs - B * F * H)}
    if kind == "reweight":
        n = case["n"]
        return {"bytes": 8 * n * 2 + 4 * n + 16 * n * case["nx"], "flops": 20 * n * (case["n_bisect"] + 2)}
    # per node: 31 operations per implicit iteration (5 of them a step), 2 Q + 5 per step
    # with modes, 34 with the Matern-type noise
    if kind == "batch":
        nodes = sum(s.nx * s.n_particles for s in _sizes(case))
        return {"bytes": 32 * nodes, "flops": nodes * case["steps"] * (155 + 2 * case["modes"] + 5)}
    nodes, S = case["nx"] * case["n"], case["steps"]
    matern = bool(case.get("matern", kind == "paper"))
    q = case["nx"] if matern else case.get("modes", 1)
    step = nodes * (155 + (34 if matern else 2 * q + 5))
    noise = 8 * case["n"] * S * q
    if kind == "bootstrap":
        return {"bytes": 32 * nodes, "flops": S * step}
    if kind == "paper":
        return {"bytes": 32 * nodes, "flops": S * step * (1 + 3 * case["n_jitter"])}
    if kind == "forecast":
        return {"bytes": 32 * nodes + noise, "flops": S * step}
    if kind == "grad":  # a forward and a backward sweep
        return {"bytes": 16 * nodes + 3 * noise, "flops": 2 * S * step}
    if kind == "pcnl":
        return {"bytes": 32 * nodes + 2 * noise, "flops": S * step * (2 * (case["n_jitter"] + 1) + 1)}
    return {"bytes": 32 * nodes + 2 * noise, "flops": S * step * case["n_jitter"]}


# --------------------------------------------------------------------------- the same in plain torch
def _matern(cells, nx, kappa=KAPPA, eta=ETA, k=KSOLVES):
    fm, fa = _ops(nx, 1.0 / kappa)
    b = eta * math.sqrt(L / nx) * 0.5 * (cells.roll(1, -1) + cells)
    return _apply(b, fm ** (k - 1) / fa**k)


def _tridiagonal(a, b, c, r):
    """Periodic tridiagonal solve along the last axis by cyclic reduction."""
    d = 1
    while float(((a.abs() + c.abs()) / b.abs()).max()) > 1e-20:
        if d >= a.shape[-1]:
            return r / (a + b + c)
        qa, qc = a / b.roll(d, -1), c / b.roll(-d, -1)
        b = b - qa * c.roll(d, -1) - qc * a.roll(-d, -1)
        r = r - qa * r.roll(d, -1) - qc * r.roll(-d, -1)
        a, c = -qa * a.roll(d, -1), -qc * c.roll(-d, -1)
        d *= 2
    return r / b


def _step(m, u, dU):
    """One implicit-midpoint step, its velocity iterated to rounding."""
    nx = m.shape[-1]
    h = L / nx
    o, dg = h / 6 - MU * DT / (2 * h), 2 * h / 3 + MU * DT / h
    fm, fh = _ops(nx)
    rhs = 2.0 * (h / 6 * (m.roll(1, -1) + m.roll(-1, -1)) + 2 * h / 3 * m)
    us, prev = u, m
    for _ in range(60):
        dv = 0.5 * DT * (u + us) + dU
        vm, vp = 0.25 * dv.roll(1, -1), 0.25 * dv.roll(-1, -1)
        ms = _tridiagonal(o - vm, dg + vp - vm, o + vp, rhs) - m
        us = _apply(ms, fm / fh)
        if float(((ms - prev).abs().amax(-1) / ms.abs().amax(-1)).max()) < 3e-14:
            break
        prev = ms
    return ms, us


def _window(m, u, noise, steps, keep=None):
    for n in range(steps):
        if keep is not None:
            keep.append((m, u))
        m, u = _step(m, u, noise(n))
    if keep is not None:
        keep.append((m, u))
    return m, u


def _nll(u, y, sig):
    return 0.5 * (((_observe(u, y.numel()) - y) / sig) ** 2).sum(-1)


def _philox(seed, c0, c1, c2, c3):
    """Philox4x32-10 of broadcast counters: four int64 tensors of 32-bit words."""
    lo32 = 0xFFFFFFFF
    w = [torch.as_tensor(x, dtype=torch.int64, device=DEV) & lo32 for x in (c0, c1, c2, c3)]
    w = list(torch.broadcast_tensors(*w))
    ka, kb = seed & lo32, (seed >> 32) & lo32
    for _ in range(10):
        pa, pb = 0xD2511F53 * w[0], 0xCD9E8D57 * w[2]
        w = [((pb >> 32) & lo32) ^ w[1] ^ ka, pb & lo32, ((pa >> 32) & lo32) ^ w[3] ^ kb, pa & lo32]
        ka, kb = (ka + 0x9E3779B9) & lo32, (kb + 0xBB67AE85) & lo32
    return w


def _uniforms(seed, c0, c1, c2, c3):
    w = _philox(seed, c0, c1, c2, c3)
    return [((w[2 * i] << 21) | (w[2 * i + 1] >> 11)).to(F64) * 2.0**-53 for i in (0, 1)]


def _draws(seed, n, step, q, tag, word3):
    """Standard normals [n][q] of one step."""
    p = torch.arange(n, device=DEV).reshape(-1, 1)
    pair = torch.arange((q + 1) // 2, device=DEV) | (tag << 24)
    a, b = _uniforms(seed, p, step, pair, word3)
    rad, ang = torch.sqrt(-2.0 * torch.log(1.0 - a)), 2.0 * math.pi * b
    return torch.stack([rad * torch.cos(ang), rad * torch.sin(ang)], -1).reshape(n, -1)[:, :q]


def _field(case, dW):
    """noise(n) of the increments dW(n) [n][q] of step n."""
    if case.get("matern", case["kind"] == "paper"):
        return lambda n: _matern(dW(n), case["nx"])
    xi = _modes(case["nx"], case["modes"])
    return lambda n: dW(n) @ xi


def _ess(s):
    e = torch.exp(s - s.max())
    return float(e.sum() ** 2 / (e * e).sum())


def _temper(phi, theta, thr, n_bisect):
    """(dtheta, theta, weights, ESS) of one tempering step."""
    rem = 1.0 - theta
    pick = rem
    if not _ess(-rem * phi) >= thr:
        lo, hi = 0.0, rem
        for _ in range(n_bisect):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if _ess(-mid * phi) >= thr else (lo, mid)
        pick = lo if lo > 0 else hi
    e = torch.exp(-pick * (phi - phi.min()))
    return pick, 1.0 if pick == rem else theta + pick, e / e.sum(), _ess(-pick * phi)


def _systematic(w, u0):
    """Systematic resampling on the cumulated weights rounded down to whole numbers."""
    n = w.numel()
    sh = 51 - (n - 1).bit_length() - math.frexp(float(w.max()))[1]
    cum = torch.floor(torch.ldexp(w, torch.tensor(sh, device=DEV))).to(torch.int64).cumsum(0).to(F64)
    T = (torch.arange(n, device=DEV, dtype=F64) + u0) * cum[-1] / n
    return torch.searchsorted(cum, T, right=True).clamp(max=n - 1)


def _pcn(case, seed, cycle, k, m0, u0, dW, phi, m, u, y, sig, theta, rho, n_jitter):
    """pCN moves; dW [n][steps][q].  Returns the chain's state and the accepted moves."""
    n, S, q = dW.shape
    accepted = torch.zeros(n, dtype=torch.int64, device=DEV)
    for j in range(n_jitter):
        w3 = (k << 16) | j
        prop = torch.empty_like(dW)
        for s in range(S):
            z = _draws(seed, n, cycle * S + s, q, TAG_PCN, w3)
            prop[:, s] = rho * dW[:, s] + math.sqrt(1 - rho * rho) * (math.sqrt(DT) * z)
        mn, un = _window(m0, u0, _field(case, lambda s: prop[:, s]), S)
        pn = _nll(un, y, sig)
        v = _uniforms(seed, torch.arange(n, device=DEV), cycle, TAG_ACCEPT << 24, w3)[0]
        ok = v < torch.exp(theta * (phi - pn))
        accepted += ok
        dW = torch.where(ok[:, None, None], prop, dW)
        phi = torch.where(ok, pn, phi)
        m, u = torch.where(ok[:, None], mn, m), torch.where(ok[:, None], un, u)
    return dW, phi, m, u, accepted


def _gradient(case, m0, u0, dW, dLam, y, sig):
    """(Phi, J, dJ/d(increments)) by the adjoint of the discrete window."""
    nx, S = case["nx"], dW.shape[1]
    h = L / nx
    o, dg = h / 6 - MU * DT / (2 * h), 2 * h / 3 + MU * DT / h
    fm, fh = _ops(nx)
    tot = dW if dLam is None else dW + dLam
    noise, xi = _field(case, lambda n: tot[:, n]), _modes(nx, case["modes"])
    states = []
    _, u = _window(m0, u0, noise, S, states)
    n_obs = y.numel()
    num = torch.arange(n_obs, device=DEV) * nx
    e, r = num // n_obs, (num % n_obs).to(F64) / n_obs
    res = (_observe(u, n_obs) - y) / sig**2
    lam = torch.zeros_like(u)
    lam.index_add_(1, e, (1 - r) * res)
    lam.index_add_(1, (e + 1) % nx, r * res)
    lam = _apply(lam, fm / fh)
    grad = torch.empty_like(dW)

    def advect(s, v):
        return 0.5 * (s.roll(1, -1) + s) * v.roll(1, -1) - 0.5 * (s + s.roll(-1, -1)) * v.roll(-1, -1)

    for n in reversed(range(S)):
        s = states[n][0] + states[n + 1][0]
        dv = 0.25 * (0.5 * DT * (states[n][1] + states[n + 1][1]) + noise(n))
        rows = (o + dv, dg + dv.roll(-1, -1) - dv.roll(1, -1), o - dv)
        nu, rhs = torch.zeros_like(lam), lam
        for _ in range(60):
            new = _tridiagonal(*rows, rhs)
            d = float(((new - nu).abs().amax(-1) / new.abs().amax(-1)).max())
            nu = new
            if d < 3e-14:
                break
            rhs = lam - 0.25 * DT * _apply(advect(s, nu), fm / fh)
        grad[:, n] = (-0.5 * advect(s, nu)) @ xi.T + tot[:, n] / DT
        lam = 2.0 * (h / 6 * (nu.roll(1, -1) + nu.roll(-1, -1)) + 2 * h / 3 * nu) - lam
    phi = _nll(u, y, sig)
    J = phi if dLam is None else phi + (0.5 * dLam**2 + dLam * dW).sum((1, 2)) / DT
    return phi, J, grad


def _exact_network(case, seed):
    F, H, O = case["n_in"], case["hidden"], case["n_out"]
    p, X, T = _network(case, seed)
    cut = np.cumsum([0, H * F, H, H * H, H, O * H, O])
    parts = [p[a:b] for a, b in zip(cut[:-1], cut[1:])]
    W1, W2, W3 = (parts[i].to(torch.bfloat16).to(F64).reshape(s) for i, s in ((0, (H, F)), (2, (H, H)), (4, (O, H))))
    b1, b2, b3 = (parts[i].to(F64) for i in (1, 3, 5))
    X, T = X.to(F64), T.to(F64)
    Z1 = X @ W1.T + b1
    H1 = Z1.relu()
    Z2 = H1 @ W2.T + b2
    H2 = Z2.relu()
    Y = H2 @ W3.T + b3
    if case["kind"] == "forward":
        return {"Y": Y}
    dY = 2.0 * (Y - T) / Y.numel()
    dZ2 = (dY @ W3) * (Z2 > 0)
    dZ1 = (dZ2 @ W2) * (Z1 > 0)
    grad = torch.cat([x.reshape(-1) for x in (dZ1.T @ X, dZ1.sum(0), dZ2.T @ H1, dZ2.sum(0), dY.T @ H2, dY.sum(0))])
    m, v = 0.1 * grad, 0.001 * grad**2
    params = p.to(F64) - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return {"Y": Y, "loss": ((Y - T) ** 2).mean().reshape(1), "grad": grad, "params": params, "m": m, "v": v}


def _exact_bootstrap(case, seed, rng_seed, cycle, u, m, y, sig):
    n, S, q = case["n"], case["steps"], case["modes"]
    noise = _field(dict(case, matern=False),
                   lambda s: math.sqrt(DT) * _draws(rng_seed, n, cycle * S + s, q, TAG_FORECAST, 0))
    m, u = _window(m, u, noise, S)
    s = -_nll(u, y, sig)
    logw = s - s.max() - torch.log(torch.exp(s - s.max()).sum())
    ess = _ess(logw)
    if ess < 0.5 * n:
        idx = _systematic(torch.exp(logw), float(_uniforms(rng_seed, 0, cycle, TAG_RESAMPLE << 24, 0)[0]))
        m, u, logw = m[idx], u[idx], torch.zeros_like(logw)
        return m, u, logw, ess, 1
    return m, u, logw, ess, 0


def _exact_paper(case, seed, u, m, y, sig):
    n, S, nx, cycle, sd = case["n"], case["steps"], case["nx"], 3, SEED + seed
    m0, u0 = m, u
    dW = torch.stack([math.sqrt(DT) * _draws(sd, n, cycle * S + s, nx, TAG_FORECAST, 0) for s in range(S)], 1)
    m, u = _window(m0, u0, _field(case, lambda s: dW[:, s]), S)
    phi, theta, k, total = _nll(u, y, sig), 0.0, 0, 0
    while theta < 1.0:
        _, theta, w, ess = _temper(phi, theta, 80.0 / 150.0 * n, 50)
        idx = _systematic(w, float(_uniforms(sd, 0, cycle, TAG_RESAMPLE << 24, k << 16)[0]))
        m0, u0, dW, phi, m, u = (x[idx] for x in (m0, u0, dW, phi, m, u))
        dW, phi, m, u, acc = _pcn(case, sd, cycle, k, m0, u0, dW, phi, m, u, y, sig, theta, W.PAPER_SHAPE.rho,
                                  case["n_jitter"])
        total += int(acc.sum())
        k += 1
    return {"m": m, "u": u, "ess": ess, "n_temper": k, "n_accept": total}


def _exact_pcnl(case, seed, u0, m0, y, sig):
    n, S, q, theta, rho, sd, cycle = case["n"], case["steps"], case["modes"], 0.02, case["rho"], SEED + seed, 3
    x = _increments(case, seed, q)
    phi, _, g = _gradient(case, m0, u0, x, None, y, sig)
    g = g - x / DT
    accepted = torch.zeros(n, dtype=torch.int64, device=DEV)
    sq = lambda t: (t * t).sum((1, 2))  # noqa: E731
    for j in range(case["n_jitter"]):
        w3 = (1 << 16) | j
        z = torch.stack([_draws(sd, n, cycle * S + s, q, TAG_PCN, w3) for s in range(S)], 1)
        c = (1 - rho) * DT * theta
        v = rho * x + math.sqrt(1 - rho * rho) * math.sqrt(DT) * z - c * g
        pv, _, gv = _gradient(case, m0, u0, v, None, y, sig)
        gv = gv - v / DT
        qd = 2 * (1 - rho * rho) * DT
        lr = (-theta * pv - sq(v) / (2 * DT) - sq(x - rho * v + c * gv) / qd) - (
            -theta * phi - sq(x) / (2 * DT) - sq(v - rho * x + c * g) / qd)
        ok = _uniforms(sd, torch.arange(n, device=DEV), cycle, TAG_ACCEPT << 24, w3)[0] < torch.exp(lr)
        accepted += ok
        x, g = (torch.where(ok[:, None, None], a, b) for a, b in ((v, x), (gv, g)))
        phi = torch.where(ok, pv, phi)
    m, u = _window(m0, u0, _field(case, lambda s: x[:, s]), S)
    return {"m": m, "u": u, "dW": x, "phi": phi, "accepted": accepted}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("forward", "train"):
        return _exact_network(case, seed)
    if kind == "reweight":
        g = _gen(seed, 0)
        phi = 0.5 * case["scale"] * (_normal(g, case["n"], 4) ** 2).sum(1)
        src = _normal(g, case["n"], case["nx"])
        dth, _, w, ess = _temper(phi, 0.0, 0.5 * case["n"], case["n_bisect"])
        idx = _systematic(w, 0.37)
        one = lambda v: torch.tensor([v], dtype=F64)  # noqa: E731
        return {"w": w, "dtheta": one(dth), "ess": one(ess), "idx": idx.to(torch.int32), "rows": src[idx]}
    if kind == "batch":
        state, ess = [], []
        for i, s in enumerate(_sizes(case)):
            c = dict(case, nx=s.nx, n=s.n_particles)
            u, m, y, sig = _ensemble(c, seed * 64 + i)
            m, u, logw, e, _ = _exact_bootstrap(c, seed, s.seed + seed, 0, u, m, y, sig)
            state += [m, u, logw]
            ess.append(e)
        return {"state": state, "ess": np.array(ess)}
    u, m, y, sig = _ensemble(case, seed)
    if kind == "bootstrap":
        m, u, logw, ess, res = _exact_bootstrap(case, seed, SEED + seed, 3, u, m, y, sig)
        return {"m": m, "u": u, "logw": logw, "ess": ess, "resampled": res}
    if kind == "paper":
        return _exact_paper(case, seed, u, m, y, sig)
    if kind == "pcnl":
        return _exact_pcnl(case, seed, u, m, y, sig)
    dW = _increments(case, seed, case["nx"] if case.get("matern") else case["modes"])
    if kind == "forecast":
        m, u = _window(m, u, _field(case, lambda s: dW[:, s]), case["steps"])
        return {"m": m, "u": u, "status": None}
    if kind == "grad":
        dLam = 0.3 * _normal(_gen(seed, 4), case["n"], case["steps"], case["modes"]) * math.sqrt(DT)
        _, J, grad = _gradient(case, m, u, dW, dLam, y, sig)
        return {"J": J, "grad": grad, "status": None}
    me, ue = _window(m, u, _field(case, lambda s: dW[:, s]), case["steps"])
    dW, phi, me, ue, acc = _pcn(case, SEED + seed, 3, 1, m, u, dW, _nll(ue, y, sig), me, ue, y, sig, 0.02,
                                case["rho"], case["n_jitter"])
    return {"m": me, "u": ue, "dW": dW, "phi": phi, "accepted": acc}
