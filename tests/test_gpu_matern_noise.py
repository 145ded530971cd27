"""The normals behind the increments and the Matern-type noise whose cells,
drawn or read in pairs, change threads through LDS, where they can go wrong:
the whole range of the normals, odd grids (a last cell without a partner),
chunk starts of both parities, every tile's smallest and largest grid."""
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


@pytest.mark.parametrize("seed,n,s,q", [(1, 1, 1, 1), (7, 3, 5, 7), (2**63 + 5, 64, 16, 2048)])
def test_normals(sch, seed, n, s, q):
    """A normal is r cos or r sin of 2 pi u with r <= sqrt(-2 ln 2^-53) < 8.6.
    Each side errs by less than an ulp or two in r (relative 5e-16), in the
    angle (2 pi u rounded: absolute 5e-16) and in the trigonometric value
    (2e-16): 2e-15 r between them.  At 2 million draws r reaches 5.4 and falls
    below 2e-3."""
    dt = 0.25
    out = torch.zeros((n, s, q), dtype=torch.float64, device="cuda")
    sch.sch_draw_increments(seed, 3, 0, sch.TAG_FORECAST, out, dt)  # cycle 3
    ref = O.draw_increments(seed, n, s, q, 3 * s, O.TAG_FORECAST, 0, dt)
    assert np.abs(out.cpu().numpy() - ref).max() <= 2e-15 * 8.6 * np.sqrt(dt)


TILES = [(64, 64), (65, 64), (127, 64), (129, 64), (256, 64), (257, 64), (511, 64), (513, 64),
         (1023, 64), (1024, 128), (1025, 128), (2047, 128), (1025, 256), (2049, 256), (4095, 256),
         (4096, 256), (4097, 512), (8191, 512)]


@pytest.mark.parametrize("nx,threads", TILES)
def test_window_on_every_tile_edge(sch, nx, threads):
    """At the parity tolerance: a node given its neighbour's cell is off by
    about 1e-3."""
    print("matern window", nx, threads, flush=True)
    n, s = 2, 2
    wl = W.MATERN_4096.scaled(nx=nx, n_steps=s)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    u0, m0, _, _ = PR.prior(wl, n)
    cells = O.draw_increments(wl.seed, n, s, nx, 0, O.TAG_FORECAST, 0, wl.dt)
    worst, m_ref, u_ref, _, _ = O.ensemble_window_matern(
        om, O.matern(wl.kappa, wl.eta, wl.k_solves), m0, u0, cells)
    assert worst == 0
    m, u = _dev(m0), _dev(u0)
    status = torch.full((n,), 99, dtype=torch.int32, device="cuda")
    sch.sch_tune_set(sch.TUNE_THREADS, threads)
    sch.sch_ensemble_step_matern(gm, sch.Matern(wl.kappa, wl.eta, wl.k_solves), m, u, _dev(cells),
                                 status)
    sch.sch_tune_set(sch.TUNE_THREADS, 0)
    assert int(status.abs().max()) == 0
    assert PR.rel_l2(m.cpu().numpy(), m_ref) < PR.REL_TOL
    assert PR.rel_l2(u.cpu().numpy(), u_ref) < PR.REL_TOL


@pytest.mark.parametrize("nx,threads", [(65, 64), (129, 64), (513, 64), (1025, 128), (2049, 256),
                                        (4097, 512)])
def test_jitter_on_odd_grids(sch, nx, threads):
    """Proposals drawn in pairs inside the kernel: the accepted cells are the
    oracle's (to the normals' rounding), the last one of an odd grid too."""
    print("matern jitter", nx, threads, flush=True)
    n, s, moves, theta = 3, 2, 2, 0.5
    wl = W.MATERN_4096.scaled(nx=nx, n_steps=s, n_obs=32, sigma_obs=0.05)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    omt = O.matern(wl.kappa, wl.eta, wl.k_solves)
    u0, m0, ut, _ = PR.prior(wl, n)
    cells = O.draw_increments(wl.seed, n, s, nx, 0, O.TAG_FORECAST, 0, wl.dt)
    _, m1, u1, _, _ = O.ensemble_window_matern(om, omt, m0, u0, cells)
    y = O.observe(ut, wl.n_obs) + wl.sigma_obs * W.random_state_noise(wl.n_obs, 3)
    sig = np.full(wl.n_obs, wl.sigma_obs)
    phi = O.ensemble_nll(u1, y, sig)
    ref = O.jitter_pcn_matern(om, omt, y, sig, wl.seed, 2, 3, m0, u0, cells, phi, m1, u1, theta,
                              0.9, moves)
    gc, gphi, gm1, gu1 = _dev(cells), _dev(phi), _dev(m1), _dev(u1)
    acc = torch.zeros(n, dtype=torch.int32, device="cuda")
    sch.sch_tune_set(sch.TUNE_THREADS, threads)
    sch.sch_jitter_pcn_matern(gm, sch.Matern(wl.kappa, wl.eta, wl.k_solves),
                              sch.Obs(_dev(y), _dev(sig)), wl.seed, 2, 3, _dev(m0), _dev(u0), gc,
                              gphi, gm1, gu1, _dev(np.array([theta])), 0.9, moves, acc)
    sch.sch_tune_set(sch.TUNE_THREADS, 0)
    assert np.array_equal(acc.cpu().numpy(), ref[4])
    assert ref[4].sum() > 0
    assert PR.rel_l2(gc.cpu().numpy(), ref[0]) < 1e-12
    assert PR.rel_l2(gphi.cpu().numpy(), ref[1]) < PR.REL_TOL
    assert PR.rel_l2(gm1.cpu().numpy(), ref[2]) < PR.REL_TOL
    assert PR.rel_l2(gu1.cpu().numpy(), ref[3]) < PR.REL_TOL
