"""Systems that grow in the interface elimination alone: the chunks' rows and the
odd interface equations eliminate quietly, but an even equation's pivot all but
vanishes beside its couplings, and the reduction level that follows leaves
couplings small enough for sweeps.  What the neighbours' equations said is then
lost in the rounding of the eliminated ones: the solve has to go another way or
to say so (SCH_E_UNSTABLE).

One Picard iteration (a plain solve) against the oracle's pivoted one; dv is one
mode's field (u = 0, one increment of 1).  A numpy emulation of the elimination
places the pivot and checks that the case goes the way that it is meant to.
Elsewhere the growth is below 2^14, so that the solve errs by about 2^14
roundings, 2e-12; taken without care, the couplings cost 1e-10 to 6e-8."""
import numpy as np
import pytest

import oracle as O
import pairing as PR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GROWTH_MAX = 2.0 ** 16
P, L = 8, 40.0  # rows a chunk, length of the domain


@pytest.fixture(scope="module")
def sch():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2402_06927_amd import sch as S

    S.lib()
    yield S
    S.sch_tune_set(S.TUNE_THREADS, 0)


@np.errstate(divide="ignore", invalid="ignore")  # at a root of the pivot itself
def eliminate(dv, NT, mu, dt):
    """The elimination on chunks of P rows: the largest |c'| of the
    chunks and of the odd interface equations, the even equations' pivots and
    couplings, the largest |a| + |c| after the reduction level, and the odd
    equations' pivots and couplings."""
    h = L / len(dv)
    o, d = h / 6 - mu * dt / (2 * h), 2 * h / 3 + mu * dt / h
    vm, vp = np.roll(dv, 1) / 4, np.roll(dv, -1) / 4
    a, b, c = (x.reshape(NT, P).T for x in (o - vm, d + vp - vm, o + vp))
    cp, g = np.zeros((P, NT)), np.ones((P, NT))
    for j in range(1, P):
        inv = 1 / (b[j] - a[j] * cp[j - 1])
        cp[j], g[j] = c[j] * inv, -a[j] * g[j - 1] * inv
    gn, kn = g[P - 1], -cp[P - 1]
    tail = np.roll(gn, 1), np.roll(kn, 1)
    for j in range(P - 2, 0, -1):
        gn, kn = g[j] - cp[j] * gn, -cp[j] * kn
    A, B, C = a[0] * tail[0], b[0] + c[0] * gn + a[0] * tail[1], c[0] * kn
    go, ko = -A[1::2] / B[1::2], -C[1::2] / B[1::2]
    pivot = B[::2] + A[::2] * np.roll(ko, 1) + C[::2] * go
    a, c = A[::2] * np.roll(go, 1) / pivot, C[::2] * ko / pivot
    inv = 1 / (1 - a * np.roll(c, 1) - c * np.roll(a, -1))
    after = np.abs(a * np.roll(a, 1) * inv) + np.abs(c * np.roll(c, -1) * inv)
    quiet = max(np.abs(cp).max(), np.abs(ko).max())
    return quiet, pivot, np.maximum(np.abs(a), np.abs(c)), after.max(), (B[1::2], go, ko)


def one_iteration(sch, dv, NT, mu, dt, seed):
    """Status, and the errors of m and u against the oracle (of a refused step,
    none: its input is kept)."""
    nx = len(dv)
    om = O.Model(L, 1.0, mu, dt, dv[None], picard_max=1)
    m0, u0 = np.random.default_rng(seed + 1).standard_normal((1, nx)), np.zeros((1, nx))
    _, m_ref, u_ref, _, _ = O.ensemble_window(om, m0, u0, np.ones((1, 1, 1)))
    dev = dict(dtype=torch.float64, device="cuda")
    gm = sch.Model(L, 1.0, mu, dt, torch.tensor(dv[None], **dev), picard_max=1)
    m, u = torch.tensor(m0, **dev), torch.tensor(u0, **dev)
    status = torch.full((1,), 99, dtype=torch.int32, device="cuda")
    sch.sch_tune_set(sch.TUNE_THREADS, NT)
    sch.sch_ensemble_step(gm, m, u, torch.ones((1, 1, 1), **dev), None, status)
    sch.sch_tune_set(sch.TUNE_THREADS, 0)
    err = [PR.rel_l2(a.cpu().numpy(), b) for a, b in ((m, m_ref), (u, u_ref))]
    print(f"nx {nx}: status {int(status)}, error of m {err[0]:.2g}, of u {err[1]:.2g}", flush=True)
    if int(status) == sch.SCH_E_UNSTABLE:
        assert np.array_equal(m.cpu().numpy(), m0)
    return int(status), *err


# threads, a random field (its seed, mu, dt and scale), the even equation and the
# node beside its first one that is moved by an amount between lo and hi, where
# its pivot changes sign, and the couplings to reach
FIELDS = [(256, 260, 1.0, 0.025, 2.5860416666666666, 91, 1, 1.1026646269800986,
           1.3231975523761195, 2.0 ** 23),
          (256, 996, 0.1, 0.05, 1.0760833333333335, 29, 1, -2.974347630361155,
           -2.799386005045793, 2.0 ** 18),
          (512, 196, 0.01, 0.1, 0.21782083333333335, 159, 1, 0.09627975815606658,
           0.10269840869980439, 2.0 ** 18),
          (512, 260, 1.0, 0.025, 5.133020833333333, 91, 1, 2.1886733595302634,
           2.6264080314363185, 2.0 ** 23)]


@pytest.mark.parametrize("NT,seed,mu,dt,scale,eq,side,lo,hi,reach", FIELDS)
def test_solve_with_a_small_even_pivot(sch, NT, seed, mu, dt, scale, eq, side, lo, hi, reach):
    nx = NT * P
    base = scale * np.random.default_rng(seed).standard_normal(nx)
    node = (2 * eq * P + side) % nx

    def field(s):
        dv = base.copy()
        dv[node] += s
        return dv

    def pivot(s):
        return eliminate(field(s), NT, mu, dt)[1][eq]

    sign = pivot(lo) > 0
    assert (pivot(hi) > 0) != sign
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if (pivot(mid) > 0) == sign else (lo, mid)
    for e in range(4, 44):  # towards the root until the couplings are reached
        dv = field(lo * (1 + 2.0 ** -e))
        quiet, _, couplings, after, _ = eliminate(dv, NT, mu, dt)
        if couplings.max() > reach:
            break
    print(f"nx {nx}: quiet {quiet:.3g}, even couplings {couplings.max():.3g}, after {after:.2g}",
          flush=True)
    # quiet everywhere else, and within the sweeps' bound after the level
    assert quiet < GROWTH_MAX / 4 and couplings.max() > reach and after < 2e-3

    status, err_m, err_u = one_iteration(sch, dv, NT, mu, dt, seed)
    assert status == sch.SCH_E_UNSTABLE or max(err_m, err_u) < PR.REL_TOL


# the same for an odd equation (not the first of an eliminated run)
ODD = [(256, 42, 0.01, 0.05, 0.30896666666666667, 55, 1, -0.07108192231364736,
        -0.0609273619831263),
       (256, 182, 1.0, 0.05, 10.292083333333334, 219, -1, -1.921542099556944,
        -1.537233679645555),
       (256, 379, 0.1, 0.025, 1.128166666666667, 231, 1, 1.254648844460772,
        1.3442666190651127),
       (512, 181, 0.01, 0.1, 0.02722760416666667, 275, -1, 0.023138679609350305,
        0.02399566774302995),
       (512, 652, 0.1, 0.1, 2.061020833333334, 173, 1, 1.3623273242984089,
        1.5326182398357093)]


@pytest.mark.parametrize("NT,seed,mu,dt,scale,eq,side,lo,hi", ODD)
def test_solve_with_a_small_odd_pivot(sch, NT, seed, mu, dt, scale, eq, side, lo, hi):
    """Systems that the order of interface_solve() solves to 1e-12 in m (it does
    not meet this pivot): neither refused nor less accurate."""
    nx = NT * P
    base = scale * np.random.default_rng(seed).standard_normal(nx)
    node = (eq * P + side) % nx

    def field(s):
        dv = base.copy()
        dv[node] += s
        return dv

    def odd(s):
        B, left, right = eliminate(field(s), NT, mu, dt)[4]
        return B[eq // 2], max(abs(left[eq // 2]), abs(right[eq // 2]))

    sign = odd(lo)[0] > 0
    assert (odd(hi)[0] > 0) != sign
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if (odd(mid)[0] > 0) == sign else (lo, mid)
    s = next(s for s in (lo * (1 + 2.0 ** -e) for e in range(4, 44)) if odd(s)[1] > 2.0 ** 19)
    status, err_m, err_u = one_iteration(sch, field(s), NT, mu, dt, seed)
    assert status != sch.SCH_E_UNSTABLE and err_m < 1e-12 and err_u < PR.REL_TOL
