"""The slot counts of a thread's rows where they change: the smallest and largest
grid of 6, 8, 12 and 16 slots on every thread count, in the window, the
jitter, the adjoint and the batched runner.  Against the oracle at the parity
tolerance: a row left out, or a dead slot taken for a row, is off by about
1e-3."""
import numpy as np
import pytest

import oracle as O
import pairing as PR
from paper_2402_06927_amd import autotune as A
from paper_2402_06927_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2402_06927_amd import sch as S

    S.lib()
    yield S
    S.sch_tune_set(S.TUNE_THREADS, 0)


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


EDGES = [(nt * k + d, nt) for nt in (64, 128, 256, 512)
         for k, d in ((4, 1), (6, 0), (6, 1), (8, 1), (12, -1), (12, 0), (12, 1), (15, 3))]


@pytest.mark.parametrize("nx,threads", EDGES)
def test_window_and_jitter(sch, nx, threads):
    print("tile edge", nx, threads, A.slots(nx, threads), flush=True)
    n, s, q, moves, theta = 2, 2, 3, 1, 0.5
    wl = W.BOOTSTRAP_256.scaled(nx=nx, n_modes=q, n_steps=s, n_obs=32, sigma_obs=0.05)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    u0, m0, ut, _ = PR.prior(wl, n)
    dW = O.draw_increments(wl.seed, n, s, q, 0, O.TAG_FORECAST, 0, wl.dt)
    worst, m1, u1, _, _ = O.ensemble_window(om, m0, u0, dW)
    assert worst == 0
    y = O.observe(ut, wl.n_obs) + wl.sigma_obs * W.random_state_noise(wl.n_obs, 3)
    sig = np.full(wl.n_obs, wl.sigma_obs)
    phi = O.ensemble_nll(u1, y, sig)
    ref = O.jitter_pcn(om, y, sig, wl.seed, 0, 0, m0, u0, dW, phi, m1, u1, theta, 0.9, moves)
    m, u = _dev(m0), _dev(u0)
    gd, gphi, gm1, gu1 = _dev(dW), _dev(phi), _dev(m1), _dev(u1)
    acc = torch.zeros(n, dtype=torch.int32, device="cuda")
    sch.sch_tune_set(sch.TUNE_THREADS, threads)
    try:
        sch.sch_ensemble_step(gm, m, u, _dev(dW))
        sch.sch_jitter_pcn(gm, sch.Obs(_dev(y), _dev(sig)), wl.seed, 0, 0, _dev(m0), _dev(u0), gd,
                           gphi, gm1, gu1, _dev(np.array([theta])), 0.9, moves, acc)
    finally:
        sch.sch_tune_set(sch.TUNE_THREADS, 0)
    for a, b in ((m, m1), (u, u1), (gm1, ref[2]), (gu1, ref[3]), (gphi, ref[1])):
        assert PR.rel_l2(a.cpu().numpy(), b) < PR.REL_TOL
    assert np.array_equal(acc.cpu().numpy(), ref[4])


@pytest.mark.parametrize("nx,threads", [e for e in EDGES if e[1] in (64, 256)])
def test_gradient(sch, nx, threads):
    n, s, q = 1, 2, 3
    wl = W.NUDGING_2048.scaled(nx=nx, n_modes=q, n_steps=s, n_obs=32)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    u, m, _, _ = PR.prior(wl, n)
    y = PR.oracle_observations(wl, 1)[0]
    dW = O.draw_increments(wl.seed, n, s, q, 0, O.TAG_NUDGE, 0, wl.dt)
    J = torch.empty(n, dtype=torch.float64, device="cuda")
    g = torch.empty((n, s, q), dtype=torch.float64, device="cuda")
    obs = sch.Obs(_dev(y), _dev(np.full(wl.n_obs, wl.sigma_obs)))
    sch.sch_tune_set(sch.TUNE_THREADS, threads)
    try:
        sch.sch_nudge_grad(gm, obs, _dev(m), _dev(u), _dev(dW), None, J, g, 2)
    finally:
        sch.sch_tune_set(sch.TUNE_THREADS, 0)
    rs, Jr, gr = O.nudge_grad(om, y, wl.sigma_obs, m[0], u[0], dW[0], np.zeros_like(dW[0]))
    assert rs == 0
    assert abs(float(J[0]) - Jr) <= 1e-10 * abs(Jr)
    assert PR.rel_l2(g[0].cpu().numpy(), gr) < PR.REL_TOL


def test_batch_of_every_class(sch):
    """One instance a tile class, their threads given (20 classes)."""
    base = W.BOOTSTRAP_256.scaled(n_steps=2, n_modes=3, n_obs=32)
    sizes = [(nt * k + 1, nt) for nt in (64, 128, 256, 512) for k in (1, 4, 6, 8, 12)]
    n, insts, ref = 3, [], []
    for i, (nx, nt) in enumerate(sizes):
        wl = base.scaled(nx=nx, n_particles=n, seed=base.seed + 2 * i)
        u, m, _, _ = PR.prior(wl, n)
        y = PR.oracle_observations(wl, 1)
        insts.append(sch.Instance(
            xi=_dev(W.mode_table(wl.L, nx, wl.n_modes, wl.mode_amp)), m=_dev(m), u=_dev(u),
            logw=torch.zeros(n, dtype=torch.float64, device="cuda"), y=_dev(y),
            sigma=_dev(np.full(wl.n_obs, wl.sigma_obs)), seed=wl.seed, threads=nt))
        ref.append(O.bootstrap_cycle(PR.oracle_model(wl), y[0], np.full(wl.n_obs, wl.sigma_obs),
                                     wl.seed, 0, m, u, np.zeros(n), wl.n_steps, wl.ess_frac))
    b = sch.Batch(base.L, base.alpha, base.mu, base.dt, base.n_modes, base.n_steps, base.n_obs,
                  base.ess_frac, insts, base.picard_tol, base.picard_max)
    b.run(0, 1, use_graph=False)
    assert not any(b.read()["status"])
    for (nx, nt), g, (rc, m, u, _, _) in zip(sizes, insts, ref):
        assert rc == 0
        assert PR.rel_l2(g.m.cpu().numpy(), m) < PR.REL_TOL, (nx, nt)
        assert PR.rel_l2(g.u.cpu().numpy(), u) < PR.REL_TOL, (nx, nt)
    b.close()
