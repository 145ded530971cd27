"""The chunks' interface system in each of its regimes: two, four and six sweeps
of the even unknowns, the same after a reduction level, the whole system in
every wavefront, and on one wavefront a particle the sweeps after no, one and
several reduction levels.  The viscosity sets how far the
couplings reach (a chunk of c nodes couples its ends by about r^c, r the root of
the step matrix), so the same grids walk through the regimes.  Against the
oracle's pivoted solve at the parity tolerance; a regime taken one step too
early is off by its bound's square root and more."""
import re
from pathlib import Path

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


def coupling(wl, threads):
    """Largest |A| + |C| over |B| of the interface rows at dv = 0."""
    h = wl.L / wl.nx
    o, d = h / 6 - wl.mu * wl.dt / (2 * h), 2 * h / 3 + wl.mu * wl.dt / h
    x = d / (2 * abs(o))
    r = x - np.sqrt(x * x - 1)
    return 2.0 / (r ** -(wl.nx // threads) + r ** (wl.nx // threads))


CASES = [(nx, threads, mu)
         for nx, threads in ((64, 64), (100, 64), (250, 64), (1000, 64), (1024, 64), (1024, 128),
                             (2000, 128), (1100, 256), (2048, 256), (4096, 256), (3000, 512),
                             (4096, 512), (8192, 512))
         for mu in (0.0, 0.01, 0.03, 0.2, 1.0, 10.0)]


@pytest.mark.parametrize("nx,threads,mu", CASES)
def test_window_across_coupling_regimes(sch, nx, threads, mu):
    n, s, q = 2, 2, 3
    wl = W.BOOTSTRAP_256.scaled(nx=nx, n_modes=q, n_steps=s, mu=mu)
    print("interface", nx, threads, mu, "coupling %.1e" % coupling(wl, threads), flush=True)
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


def test_cases_reach_every_regime():
    from collections import Counter

    def halve(e):  # couplings after every other unknown is eliminated
        return e * e / 2 / (1 - e * e / 2)

    def sweeps(e):
        return 2 if e <= 2.0 ** -19 else 4 if e <= 3.4e-4 else 6 if e <= 3.4e-3 else 0

    one, several = Counter(), Counter()
    for nx, threads, mu in CASES:
        e = coupling(W.BOOTSTRAP_256.scaled(nx=nx, mu=mu), threads)
        if threads == 64:
            levels = 0
            while e > 3.4e-4 and levels < 6:
                e, levels = halve(e), levels + 1
            one[min(levels, 2), sweeps(e)] += 1
        else:
            e = halve(e)
            several[("", e and sweeps(e)) if sweeps(e) else ("level", sweeps(halve(e)))] += 1
    assert all(several["", k] for k in (2, 4, 6)) and several["level", 0], several
    assert any(several["level", k] for k in (2, 4, 6)), several
    assert all(any(one[n, k] for k in (2, 4)) for n in (0, 1, 2)), one


def device_bounds():
    """The device's bounds on the couplings, by the number of sweeps."""
    src = (Path(__file__).parents[1] / "paper_2402_06927_amd" / "csrc" / "device.hpp").read_text()
    line = re.search(r"constexpr double kSweep2 = .*?;", src, re.S).group()
    got = {int(k): float.fromhex(v) if "x" in v else float(v)
           for k, v in re.findall(r"kSweep(\d) = ([^,;]+)", line)}
    assert sorted(got) == [2, 4, 6]
    return got


def test_sweeps_cut_off_below_rounding():
    """K sweeps of couplings below eps leave eps^(K+1) of the largest unknown: at
    most a sixteenth of a rounding."""
    for k, eps in device_bounds().items():
        assert eps ** (k + 1) <= 2.0 ** -57, (k, eps)


# couplings that the reduction's last level still sees
REDUCED = [(64, 64, 1000.0), (100, 64, 1000.0), (1000, 64, 1000.0), (1024, 128, 1000.0),
           (1100, 256, 1000.0), (2100, 512, 1000.0)]


@pytest.mark.parametrize("nx,threads,mu", REDUCED)
def test_window_reduced_to_the_last_level(sch, nx, threads, mu):
    test_window_across_coupling_regimes(sch, nx, threads, mu)


def test_cases_reach_every_regime_of_the_device():
    """As test_cases_reach_every_regime, by the device's own bounds, and with the
    reduction that goes to its end: on one wavefront, and on several after the
    elimination of interface_solve()."""
    bounds = device_bounds()

    def halve(e):  # couplings after every other unknown is eliminated
        return e * e / 2 / (1 - e * e / 2)

    def sweeps(e):
        return next((k for k in (2, 4, 6) if e <= bounds[k]), 0)

    one, several, to_the_end = set(), set(), set()
    for nx, threads, mu in CASES + REDUCED:
        e = coupling(W.BOOTSTRAP_256.scaled(nx=nx, mu=mu), threads)
        if threads > 64:
            e = halve(e)
            after = sweeps(halve(e))
            several.add(("window", sweeps(e)) if sweeps(e) else ("level", after))
            if sweeps(e) or after:
                continue
            # the whole system: 64 equations, one for every threads / 64 chunks
            e = coupling(W.BOOTSTRAP_256.scaled(nx=64 * (nx // 64), mu=mu), 64)
        levels = 0
        while e > bounds[4] and levels < 6:
            e, levels = halve(e), levels + 1
        if levels == 6:
            to_the_end.add(threads)
        if threads == 64:
            one.add((min(levels, 2), 0 if levels == 6 else sweeps(e)))
    assert {("window", k) for k in (2, 4, 6)} | {("level", 0)} <= several, several
    assert any(("level", k) in several for k in (2, 4, 6)), several
    assert all(any((n, k) in one for k in (2, 4)) for n in (0, 1, 2)), one
    assert {64, 128, 256, 512} <= to_the_end, to_the_end
