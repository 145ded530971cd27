"""Weights, resampling and gather where their kernels change paths: the last
particle kept in registers and in LDS and the first that is not, failed
particles (infinite or NaN potential) in each place, rows that 16-byte loads
cannot take, and the tile that the number of particles picks.

Weights against the oracle at relative L2 1e-12 (each side errs by a few ulp in
the exponential and n eps in the sum), bisected steps at the parity test's
bars; indices and rows exactly."""
import math

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
    return S


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a), device="cuda")


def _temper(sch, phi, theta, thr, n_bisect, extra=None):
    n = len(phi)
    th, dth, ess = _dev([float(theta)]), _dev([0.0]), _dev([0.0])
    w, lo = _dev(np.zeros(n)), _dev(np.zeros(n))
    sch.sch_temper_ess(_dev(phi), th, thr, n_bisect, dth, w, ess,
                       *(() if extra is None else (_dev(extra), lo)))
    return (float(th), float(dth), float(ess), w.cpu().numpy(), lo.cpu().numpy())


def _phi(n, bad):
    phi = W.random_phi(n, n, 20.0)
    if bad and n > 2:
        phi[0], phi[n // 2], phi[n - 1] = np.inf, np.nan, np.inf
    return phi


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 8192, 8193, 12001])
def test_weights(sch, n, bad):
    phi, extra = _phi(n, bad), W.random_state_noise(n, 6)
    for x in (None, extra):
        _, dth, ess, w, lo = _temper(sch, phi, 0.25, 0.0, 0, x)
        e_ref, w_ref, lo_ref = O.weights(phi, 0.75, x)
        assert dth == 0.75 and abs(ess - e_ref) <= 1e-12 * e_ref
        assert PR.rel_l2(w, w_ref) < 1e-12
        if x is not None:
            ok = np.isfinite(lo_ref)
            assert np.array_equal(ok, np.isfinite(lo)) and PR.rel_l2(lo[ok], lo_ref[ok]) < 1e-12
    if n > 1:
        _, dth, ess, w, _ = _temper(sch, phi, 0.0, 0.5 * n, 50)
        d_ref, w_ref, e_ref = O.temper(phi, 0.0, 0.5 * n, 50)
        assert abs(dth - d_ref) <= 1e-12 * d_ref + 2.0 ** -40
        assert abs(ess - e_ref) < 1e-9 * e_ref and PR.rel_l2(w, w_ref) < 1e-9


@pytest.mark.parametrize("offset", [1e5, 1e8])
@pytest.mark.parametrize("n", [5, 1024, 8193])
def test_weights_of_potentials_far_from_zero(sch, n, offset):
    """A common offset drops out of the weights: beta phi is rounded once, alike
    for the largest exponent, the sum and the weights (an ulp of beta phi is
    7e-12 at 1e5 and 7e-9 at 1e8).  Both sides then exponentiate the same
    differences, so test_weights' bar holds; the weights add up to 1."""
    phi = offset + _phi(n, False)
    for x in (None, np.zeros(n)):
        for beta in (1.0, 0.75):
            _, _, ess, w, _ = _temper(sch, phi, 1.0 - beta, 0.0, 0, x)
            e_ref, w_ref, _ = O.weights(phi, beta, x)
            assert abs(ess - e_ref) <= 1e-12 * e_ref, (beta, ess, e_ref)
            assert PR.rel_l2(w, w_ref) < 1e-12, beta
            assert abs(math.fsum(w) - 1.0) < 1e-12, beta


def test_no_particle_left(sch):
    for x in (None, np.zeros(70)):
        _, _, ess, w, _ = _temper(sch, np.full(70, np.inf), 0.0, 0.0, 0, x)
        assert ess == 0.0 and not w.any()


@pytest.mark.parametrize("n", [1, 2, 65, 1023, 8191, 8192, 8193])
def test_resample(sch, n):
    w = W.random_weights(n, n, spread=2.0)
    idx = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    sch.sch_resample(_dev(w), _dev([0.61]), idx, sch.workspace(sch.WS_RESAMPLE, None, n))
    st, ref = O.resample_systematic(w, 0.61)
    assert st == 0 and np.array_equal(idx.cpu().numpy(), ref)


@pytest.mark.parametrize("row_len", [1, 2, 255, 256, 1000, 1001, 5000])
@pytest.mark.parametrize("shift", [0, 1])
def test_gather(sch, row_len, shift):
    n = 7
    base = _dev(np.random.default_rng(1).standard_normal(n * row_len + 1))
    src = base[shift:shift + n * row_len].view(n, row_len)
    dst = torch.full((n, row_len), 5.0, dtype=torch.float64, device="cuda")
    idx = torch.tensor([3, 3, 0, 6, -1, 2, 7], dtype=torch.int32, device="cuda")
    sch.sch_gather(idx, src, dst)
    for j, r in enumerate(idx.tolist()):
        want = src[r] if 0 <= r < n else torch.full_like(dst[j], 5.0)
        assert torch.equal(dst[j], want)


@pytest.mark.parametrize("nx,n,threads", [(1000, 256, 128), (1000, 257, 64), (1500, 512, 256),
                                          (1500, 513, 128), (3000, 2, 256), (500, 600, 64),
                                          (4100, 2, 512)])
def test_default_tile_by_ensemble(sch, nx, n, threads):
    """The default tile's bits are those of the tile asked for by name, on both
    sides of every line."""
    wl = W.BOOTSTRAP_256.scaled(nx=nx, n_modes=2, n_steps=1)
    gm = PR.gpu_model(wl)
    u0, m0, _, _ = PR.prior(wl, 2)
    u0, m0 = (np.resize(a, (n, nx)) for a in (u0, m0))
    dW = O.draw_increments(wl.seed, n, 1, 2, 0, O.TAG_FORECAST, 0, wl.dt)
    out = []
    try:
        for nt in (0, threads):
            sch.sch_tune_set(sch.TUNE_THREADS, nt)
            m, u = _dev(m0), _dev(u0)
            sch.sch_ensemble_step(gm, m, u, _dev(dW))
            out.append((m, u))
    finally:
        sch.sch_tune_set(sch.TUNE_THREADS, 0)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("nx,n", [(65, 17), (100, 512), (100, 513)])
def test_rows_resampled_in_a_cycle(sch, nx, n):
    """The state's rows after a resampling, on both sides of the ensemble size
    up to which they change places in LDS."""
    wl = W.BOOTSTRAP_256.scaled(nx=nx, n_modes=3, n_steps=2, n_obs=40, n_particles=n)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    u0, m0, _, _ = PR.prior(wl, n)
    y, sig = PR.oracle_observations(wl, 1)[0], np.full(wl.n_obs, wl.sigma_obs)
    rc, m_o, u_o, _, st_o = O.bootstrap_cycle(om, y, sig, wl.seed, 0, m0, u0, np.zeros(n),
                                              wl.n_steps, 1.01)
    assert rc == 0 and st_o.resampled
    m, u, lw = _dev(m0), _dev(u0), _dev(np.zeros(n))
    st = sch.sch_pf_bootstrap_cycle(gm, sch.Obs(_dev(y), _dev(sig)), wl.seed, 0, m, u, lw,
                                    wl.n_steps, 1.01,
                                    sch.workspace(sch.WS_BOOTSTRAP, gm, n, wl.n_steps))
    assert st["resampled"] == 1 and abs(st["ess"] - st_o.ess) < 1e-9 * st_o.ess
    assert PR.rel_l2(m.cpu().numpy(), m_o) < PR.REL_TOL
    assert PR.rel_l2(u.cpu().numpy(), u_o) < PR.REL_TOL


@pytest.mark.parametrize("row_len", [2, 510, 512, 514, 1024, 1026, 32766, 32768, 32770])
def test_gather_of_pairs_at_the_grids_edges(sch, row_len):
    """Rows of whole 16-byte pairs at the lengths where another workgroup starts."""
    src = torch.arange(5 * row_len, dtype=torch.float64, device="cuda").reshape(5, row_len)
    idx = torch.tensor([4, 0, 0, 3, 2], dtype=torch.int32, device="cuda")
    dst = torch.full_like(src, -1.0)
    sch.sch_gather(idx, src, dst)
    assert torch.equal(dst, src[idx.long()])


@pytest.mark.parametrize("n,n_steps", [(128, 256), (129, 256)])
def test_long_rows_resampled_in_a_cycle(sch, n, n_steps):
    """A tempered cycle whose increments' rows are long (one value per cell and
    step, over 256 MiB in all), on both sides of the rows up to which these change
    places in LDS.  Each step of either side errs by the
    tolerance 1e-13 at most: 5e-11 in all."""
    wl = W.MATERN_4096.scaled(nx=1024, n_steps=n_steps, n_obs=40, n_particles=n, eta=0.1, dt=0.01)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    omt = O.matern(wl.kappa, wl.eta, wl.k_solves)
    gmt = sch.Matern(wl.kappa, wl.eta, wl.k_solves)
    u0, m0, _, _ = PR.prior(wl, n)
    y, sig = O.observe(u0[0], wl.n_obs), np.full(wl.n_obs, 1.0)
    args = (n_steps, 0.9 * n, 50, 0.9, 1, 3)
    rc, out, st_o = O.tempered_cycle_matern(om, omt, y, sig, wl.seed, 0, m0, u0, *args)
    m, u = _dev(m0), _dev(u0)
    st = sch.sch_pf_tempered_cycle_matern(gm, gmt, sch.Obs(_dev(y), _dev(sig)), wl.seed, 0, m, u,
                                          *args,
                                          sch.matern_workspace(sch.WS_TEMPERED, gm, n, n_steps, 1))
    assert rc == 0 and st["n_temper"] == st_o.n_temper and st["n_accept"] == st_o.n_accept
    assert PR.rel_l2(m.cpu().numpy(), out["m"]) < PR.REL_TOL
    assert PR.rel_l2(u.cpu().numpy(), out["u"]) < PR.REL_TOL
