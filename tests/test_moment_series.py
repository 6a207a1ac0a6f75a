"""The series that the moment forms ship, from the header the library compiles: a pair's whole window against the profile
itself over all offsets from the nearest sample, with the window's edge on either side of half a sample, the
numbers of terms at their limits, and where the form is refused."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
JMAX, MOM_MAX = 40, 12
GAUSS, EXPONENTIAL, POWER, UNIFORM = range(4)
FM_TOL, AM_TOL = 2e-7, 2.5e-8
ROUND = 2e-7                               # coefficients in FP32: 6e-8 of at most three peaks


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("series") / "series.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2604_09643_amd", "csrc"), "-o", so,
                    os.path.join(ROOT, "tests", "series", "series_driver.cpp")], check=True)
    return ctypes.CDLL(so)


def series(lib, kernel, sigma, trunc, nu=2.0, exact=True, delta=1.0):
    terms, edge, coef = np.zeros(5, np.int32), np.zeros(6, np.float32), np.zeros((3, JMAX + 1, MOM_MAX), np.float32)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    d = ctypes.c_double
    lib.series(kernel, d(delta), d(sigma), d(trunc), d(nu), int(exact), p(terms), p(edge), p(coef))
    return terms, edge.astype(np.float64), coef.astype(np.float64)


def phi(kernel, x, w, nu):
    a = np.abs(x) / w
    return x * {GAUSS: np.exp(-0.5 * a * a), EXPONENTIAL: np.exp(-a), POWER: (1 + a * a) ** -nu}[kernel]


def dphi(kernel, x, w, nu):
    a = np.abs(x) / w
    return {GAUSS: (1 - a * a) * np.exp(-0.5 * a * a), EXPONENTIAL: (1 - a) * np.exp(-a),
            POWER: (1 + a * a) ** -nu * (1 - 2 * nu * a * a / (1 + a * a))}[kernel]


def window(terms, edge, coef, which, t, jt, derivative=False):
    """Rows -jt .. jt of a pair at offsets t, as the kernels add them up."""
    rows = np.zeros((2 * jt + 1, t.size))
    n = np.arange(MOM_MAX)
    for j in range(-jt, jt + 1):
        c = coef[which, abs(j)] * (np.where(n % 2 == 0, -1.0, 1.0) if j < 0 else 1.0)
        rows[j + jt] = sum(c[i] * i * t ** (i - 1) for i in range(1, MOM_MAX)) if derivative else sum(c[i] * t ** i for i in n)
    if terms[3]:
        a = np.abs(t)
        inside = a >= np.float32(edge[0])
        far = (t < 0) == bool(terms[4])    # row + jt
        if derivative:
            v = edge[2] + 2 * edge[3] * a + 3 * edge[4] * a * a
        else:
            v = np.copysign(1.0, t) * (edge[1] + a * (edge[2] + a * (edge[3] + a * edge[4])))
        np.add.at(rows, (np.where(far, 2 * jt, 0), np.arange(t.size)), np.where(inside, v, 0.0))
    if terms[3] == 2:
        e = np.exp2(edge[5] * np.abs(t))
        rows[jt] += 0.5 * e * (1 + np.log(2.0) * edge[5] * np.abs(t)) if derivative else 0.5 * t * e
    return rows


CASES = [(GAUSS, 1 / 0.40, 6.0, 1.0, 6), (GAUSS, 1 / 0.42, 6.0, 1.0, 7), (GAUSS, 1 / 0.63, 6.0, 1.0, 7), (GAUSS, 1 / 0.65, 6.0, 1.0, 8),
         (GAUSS, 1 / 0.74, 6.0, 1.0, 8), (GAUSS, 1 / 1.04, 6.0, 1.0, 8), (GAUSS, 2.08, 6.0, 1.0, 7),
         (EXPONENTIAL, 2.078, 12.0, 1.0, 6), (EXPONENTIAL, 1.558, 12.0, 1.0, 8), (EXPONENTIAL, 3.247, 9.0, 1.0, 6),
         (EXPONENTIAL, 2.0, 12.2, 1.0, 6), (POWER, 2.078, 10.0, 2.0, 10), (POWER, 1.43, 10.0, 3.0, 12), (POWER, 3.117, 9.2, 2.0, 8),
         (POWER, 1.974, 10.2, 2.0, 10)]


@pytest.mark.parametrize("kernel,w,trunc,nu,fwd", CASES)
def test_windows(lib, kernel, w, trunc, nu, fwd):
    jt = int(np.floor(trunc * w + 0.5))
    terms, edge, coef = series(lib, kernel, w, trunc, nu)
    assert terms[0] == fwd and terms[3] == {GAUSS: 0, POWER: 1, EXPONENTIAL: 2}[kernel]
    t = np.linspace(-1.0, 1.0, 2001)
    if terms[3]:                           # the indicator's own step aside
        t = t[np.abs(np.abs(t) - abs(2.0 * (jt - trunc * w))) > 1e-5]
    u = 0.5 * t[None] - np.arange(-jt, jt + 1)[:, None]
    keep = (np.abs(u) <= trunc * w) if kernel != GAUSS else np.ones(u.shape, dtype=bool)
    want = np.where(keep, phi(kernel, u, w, nu), 0.0)
    peak = np.abs(phi(kernel, np.linspace(0.0, trunc * w, 20001), w, nu)).max()
    for which, tol in ((0, FM_TOL), (1, FM_TOL), (2, AM_TOL)):
        if terms[which]:
            got = window(terms, edge, coef, which, t, jt)
            # four terms of the edge sample are within FM_TOL too
            assert np.abs(got - want).max() <= ((FM_TOL if terms[3] else tol) + ROUND) * peak
    if terms[2]:                           # the derivative in t: a Chebyshev term's grows by its order squared at most
        got, want = window(terms, edge, coef, 2, t, jt, True), np.where(keep, 0.5 * dphi(kernel, u, w, nu), 0.0)
        inner = slice(1, -1) if terms[3] else slice(None)      # the edge sample's four terms have a coarser derivative
        assert np.abs(got - want)[inner].max() <= (64 * AM_TOL + 8 * ROUND) * peak


def test_where_the_form_ends(lib):
    assert series(lib, GAUSS, 1 / 1.10, 6.0)[0][0] == 8 and series(lib, GAUSS, 1 / 1.13, 6.0)[0][0] == 0
    assert list(series(lib, GAUSS, 1 / 0.76, 6.0)[0][:3]) == [8, 8, 0]
    assert list(series(lib, GAUSS, 1 / 0.56, 5.9)[0][1:3]) == [0, 0]       # short windows: the adjoints test their edges
    assert list(series(lib, GAUSS, 1 / 0.55, 5.9)[0][:3]) == [7, 7, 8]
    assert series(lib, GAUSS, 5.0, 5.9, exact=False)[0][0] == 0
    assert series(lib, GAUSS, 5.0, 6.0, exact=False)[0][0] == 6
    assert series(lib, POWER, 2.078, 9.0, 2.0)[0][0] == 0 and series(lib, POWER, 2.078, 9.2, 2.0)[0][0] > 0
    assert series(lib, EXPONENTIAL, 2.078, 8.6)[0][0] == 0 and series(lib, EXPONENTIAL, 2.078, 8.8)[0][0] > 0
    assert series(lib, UNIFORM, 3.0, 1.0)[0][0] == 0
