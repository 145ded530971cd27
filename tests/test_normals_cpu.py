"""The two factors of the device's Box-Muller pair at the points that random
counters hardly ever hit: v = 1 (no reciprocal root), 2^-53 and 1 - 2^-53, the
switch of the mantissa at sqrt(1/2) and at powers of two, u at and beside the
eighths of a turn, and the wrap below 1.

box_radius and turn_sincos are compiled from the device's source for the host,
with the hardware's estimates (rcp, rsq: single-precision values, as good as
theirs) in their places, and compared with 64-bit-mantissa values.  Bars: the
logarithm errs by its argument's sum, its quotient and its own sum (3 roundings
of 2^-53, halved by the root), the root by one: 2.5, taken as 3; the angle by
two roundings of at most pi / 4 and the polynomial by one: 2^-52."""
import ctypes
import re
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

EPS = 2.0 ** -53
SHIM = r"""
#include <cmath>
#include <cstdint>
using std::fma; using std::rint;
#define __device__
#define __forceinline__ inline
static double emu_rcp(double x) { return 1.0f / (float)x; }
static double emu_rsq(double x) { return 1.0f / std::sqrt((float)x); }
static double emu_mant(double x) { int e; return std::frexp(x, &e); }
static int emu_exp(double x) { int e; std::frexp(x, &e); return e; }
#define __builtin_amdgcn_rcp emu_rcp
#define __builtin_amdgcn_rsq emu_rsq
#define __builtin_amdgcn_frexp_mant emu_mant
#define __builtin_amdgcn_frexp_exp emu_exp
%s
extern "C" void factors(int n, const double* v, const double* u, double* r, double* s, double* c) {
  for (int i = 0; i < n; ++i) { r[i] = box_radius(v[i]); turn_sincos(u[i], s[i], c[i]); }
}
"""


@pytest.fixture(scope="module")
def factors(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    src = (Path(__file__).parents[1] / "paper_2402_06927_amd" / "csrc" / "device.hpp").read_text()
    body = "\n".join(re.search(r"__device__ __forceinline__ \w+ %s\(.*?\n}\n" % f, src, re.S).group()
                     for f in ("rcp64", "box_radius", "turn_sincos"))
    d = tmp_path_factory.mktemp("normals")
    (d / "f.cpp").write_text(SHIM % body)
    subprocess.run([gxx, "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", "-o",
                    d / "f.so", d / "f.cpp"], check=True)
    lib = ctypes.CDLL(str(d / "f.so"))

    def call(v, u):
        v, u = np.ascontiguousarray(v), np.ascontiguousarray(u)
        out = [np.empty(len(v)) for _ in range(3)]
        p = lambda a: a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))  # noqa: E731
        lib.factors(len(v), p(v), p(u), *(p(o) for o in out))
        return out

    return call


def _radius_points():
    k = {1, 2, 3, 4, 2 ** 53, 2 ** 53 - 1, 2 ** 53 - 2, 2 ** 53 - 3}
    for e in range(1, 53):
        for c in (2 ** e, int(2 ** e * np.sqrt(0.5))):
            k |= {c + j for j in range(-3, 4)}
    k |= {int(x) for x in np.random.default_rng(1).integers(1, 2 ** 53, 20000)}
    return np.array(sorted(x for x in k if 1 <= x <= 2 ** 53), dtype=np.float64) * EPS


def _angle_points():
    k = {j * 2 ** 50 + d for j in range(9) for d in (-3, -2, -1, 0, 1, 2, 3)}
    k |= {int(x) for x in np.random.default_rng(2).integers(0, 2 ** 53, 20000)}
    return np.array(sorted(x for x in k if 0 <= x < 2 ** 53), dtype=np.float64) * EPS


def test_radius(factors):
    v = _radius_points()
    r, _, _ = factors(v, np.zeros_like(v))
    ref = np.sqrt(-2 * np.log(v.astype(np.longdouble)))
    assert v[-1] == 1.0 and r[-1] == 0.0 and v[0] == EPS
    assert np.abs((r[:-1] - ref[:-1]) / ref[:-1]).max() <= 3 * EPS


def test_radius_no_worse_than_the_library(factors):
    """The device library's sqrt(-2 log v) errs by 1.66e-16 at most, the factor by
    no more than its root's rounding, half a rounding of the sum's first part
    (which lies in its log, at most 1.25 times as large) and half of three
    roundings of the quarter that the series makes: 2 EPS, 2.2e-16.  Where the
    exponent is 0 (v in [0.707, 1)) that first part is exact, and the series a
    sixth: 1.25 EPS, 1.4e-16."""
    v = _radius_points()[:-1]
    k = np.random.default_rng(3).integers(int(2 ** 53 * 0.3), 2 ** 53, 400000)
    v = np.concatenate([v, k.astype(np.float64) * EPS])
    r, _, _ = factors(v, np.zeros_like(v))
    ref = np.sqrt(-2 * np.log(v.astype(np.longdouble)))
    err = np.abs((r - ref) / ref)
    assert err.max() <= 2 * EPS
    assert err[v >= 0.7072].max() <= 1.25 * EPS


def test_sine_and_cosine(factors):
    u = _angle_points()
    _, s, c = factors(np.full_like(u, 0.5), u)
    q = np.rint(4 * u).astype(int)
    x = np.longdouble("6.283185307179586476925286766559") * (u.astype(np.longdouble)
                                                             - q / np.longdouble(4))
    a, b = np.sin(x), np.cos(x)
    sref = np.choose(q & 3, (a, b, -a, -b))
    cref = np.choose(q & 3, (b, -a, -b, a))
    assert q.max() == 4 and np.abs(s - sref).max() <= 2 * EPS and np.abs(c - cref).max() <= 2 * EPS
    # the small one of the two to the same number of its own roundings, and 0 at
    # the quarter turns
    small, ref = np.where(q & 1, c, s), np.where(q & 1, cref, sref)
    assert np.abs(small - ref).max() <= 2 * EPS and not small[ref == 0].any()
    near = (ref != 0) & (np.abs(ref) < 1e-3)
    assert near.any() and np.abs((small[near] - ref[near]) / ref[near]).max() <= 3 * EPS
