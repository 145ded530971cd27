"""The modes form's noise sum, whose nodes change threads through LDS, where its
map can go wrong: odd grids (a single last node, rows of the mode table 8-byte
aligned), one row and odd numbers of modes, every tile's smallest and largest
grid.  Against the oracle's window at the parity tolerance: a node given its
neighbour's noise is off by about 1e-3."""
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


@pytest.mark.parametrize("nx,threads,q", [
    (64, 64, 1), (127, 64, 3), (129, 64, 1), (256, 64, 8), (257, 64, 3), (511, 64, 2), (512, 64, 5),
    (513, 64, 7), (1023, 64, 1), (1024, 64, 4), (1023, 128, 3), (1024, 128, 2), (1025, 128, 1),
    (2047, 128, 5), (2048, 128, 8), (1025, 256, 3), (2047, 256, 1), (2048, 256, 7), (2049, 256, 2),
    (4095, 256, 5), (4096, 256, 3), (2049, 512, 1), (4095, 512, 3), (4096, 512, 8), (4097, 512, 2),
    (8191, 512, 3), (8192, 512, 1)])
def test_window_noise_on_every_tile_edge(sch, nx, threads, q):
    print("modes noise", nx, threads, q, flush=True)
    n, s = 2, 2
    wl = W.BOOTSTRAP_256.scaled(nx=nx, n_modes=q, n_steps=s)
    om, gm = PR.oracle_model(wl), PR.gpu_model(wl)
    u0, m0, _, _ = PR.prior(wl, n)
    dW = O.draw_increments(wl.seed, n, s, q, 0, O.TAG_FORECAST, 0, wl.dt)
    worst, m_ref, u_ref, _, _ = O.ensemble_window(om, m0, u0, dW)
    assert worst == 0
    m, u, d = (torch.tensor(np.ascontiguousarray(a), device="cuda") for a in (m0, u0, dW))
    status = torch.full((n,), 99, dtype=torch.int32, device="cuda")
    sch.sch_tune_set(sch.TUNE_THREADS, threads)
    sch.sch_ensemble_step(gm, m, u, d, None, status)
    sch.sch_tune_set(sch.TUNE_THREADS, 0)
    assert int(status.abs().max()) == 0
    assert PR.rel_l2(m.cpu().numpy(), m_ref) < PR.REL_TOL
    assert PR.rel_l2(u.cpu().numpy(), u_ref) < PR.REL_TOL
