"""The reverse sweep's own row layout and its mode products where they can go
wrong: chunk lengths of both parities (a last pair that not every chunk holds,
slots left over one by one), odd grids (rows 8-byte aligned, a single last
node), one row and odd numbers of modes, every tile's smallest and largest
grid; three steps in segments of two, so that both a recomputed and a kept
segment are read.  Against the oracle's reverse sweep at its bars: a value read
from another slot is off by about 1e-3."""
import numpy as np
import pytest

import oracle as O
import pairing as PR
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


def _check(sch, wl, q, ref, run):
    n, s = 2, 3
    u, m, _, _ = PR.prior(wl, n)
    y = PR.oracle_observations(wl, 1)[0]
    dW = O.draw_increments(wl.seed, n, s, q, 0, O.TAG_NUDGE, 0, wl.dt)
    dLam = 0.5 * np.sqrt(wl.dt) * np.random.default_rng(wl.nx).standard_normal(dW.shape)
    J = torch.empty(n, dtype=torch.float64, device="cuda")
    g = torch.empty((n, s, q), dtype=torch.float64, device="cuda")
    st = torch.full((n,), 99, dtype=torch.int32, device="cuda")
    obs = sch.Obs(_dev(y), _dev(np.full(wl.n_obs, wl.sigma_obs)))
    run(obs, _dev(m), _dev(u), _dev(dW), _dev(dLam), J, g, 2, st)
    assert int(st.abs().max()) == 0
    for p in range(n):
        rs, Jr, gr = ref(y, wl.sigma_obs, m[p], u[p], dW[p], dLam[p])
        assert rs == 0
        assert abs(float(J[p]) - Jr) <= 1e-10 * abs(Jr)
        gg, gir = g[p].cpu().numpy(), (dLam[p] + dW[p]) / wl.dt
        assert PR.rel_l2(gg, gr) < PR.REL_TOL
        assert PR.rel_l2(gg - gir, gr - gir) < 1e-9  # the data part, on its own scale


@pytest.mark.parametrize("nx,threads,q", [
    (64, 64, 1), (65, 64, 2), (129, 64, 3), (191, 64, 1), (256, 64, 8), (257, 64, 3), (383, 64, 5),
    (449, 64, 2), (511, 64, 1), (512, 64, 7), (1023, 128, 3), (1024, 128, 2), (1025, 256, 1),
    (1535, 256, 5), (2047, 256, 3), (4095, 512, 2), (4097, 512, 1), (4608, 512, 3), (8191, 512, 5),
    (8192, 512, 2)])
def test_modes(sch, nx, threads, q):
    print("adjoint rows", nx, threads, q, flush=True)
    wl = W.NUDGING_2048.scaled(nx=nx, n_modes=q, n_steps=3, n_obs=32)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    sch.sch_tune_set(sch.TUNE_THREADS, threads)
    try:
        _check(sch, wl, q, lambda *a: O.nudge_grad(om, *a),
               lambda *a: sch.sch_nudge_grad(gm, *a))
    finally:
        sch.sch_tune_set(sch.TUNE_THREADS, 0)


@pytest.mark.parametrize("nx,threads", [(65, 64), (129, 64), (383, 64), (513, 64), (577, 64),
                                        (1023, 64), (1024, 64), (2047, 128), (4097, 512)])
def test_cells(sch, nx, threads):
    print("adjoint rows, matern", nx, threads, flush=True)
    wl = W.MATERN_4096.scaled(nx=nx, n_steps=3, n_obs=32)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    mt = (wl.kappa, wl.eta, wl.k_solves)
    omt, gmt = O.matern(*mt), sch.Matern(*mt)
    sch.sch_tune_set(sch.TUNE_THREADS, threads)
    try:
        _check(sch, wl, nx, lambda *a: O.nudge_grad_matern(om, omt, *a),
               lambda *a: sch.sch_nudge_grad_matern(gm, gmt, *a))
    finally:
        sch.sch_tune_set(sch.TUNE_THREADS, 0)
