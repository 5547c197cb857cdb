"""The search for the trust-region multiplier (csrc/trbracket.h, the code that the solver's
kernel runs), compiled for the host and driven by factorisations in numpy, a round of four
multipliers at a time: the number of rounds, and what it ends with.

  * a step inside the region or on its boundary is found within the search's rounds, and its
    multiplier is the eigen-decomposition's;
  * where there is no multiplier (B singular or indefinite, no gradient along the least
    eigenvalue's direction, and a short step in the others), the search gives up: in the first
    round if B and the gradient vanish in whole coordinates (a type weight of exactly 0 or 1),
    by the fifth if B is singular, and in any case before an eigen-decomposition's time (17
    rounds) has gone."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N, WAVES = 27, 4
MORE, NONE = -1, -2

SHIM = """
#include "trbracket.h"
using celmi::TrBracket;
extern "C" {
int tr_rounds() { return celmi::kTrRounds; }
int tr_size() { return sizeof(TrBracket); }
void tr_start(TrBracket* b, double below, double disc, double gnorm, double r, int dec) { b->start(below, disc, gnorm, r, dec); }
double tr_first(const TrBracket* b, int w) { return b->first(w); }
int tr_take(TrBracket* b, int round, const double (*rs)[3]) { return b->take(round, rs); }
double tr_next(const TrBracket* b, int w) { return b->next(w); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("bracket")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1803_00113_amd", "csrc"),
                    str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    l = C.CDLL(str(d / "shim.so"))
    l.tr_start.argtypes = [C.c_void_p, C.c_double, C.c_double, C.c_double, C.c_double, C.c_int]
    for f in (l.tr_first, l.tr_next):
        f.argtypes, f.restype = [C.c_void_p, C.c_int], C.c_double
    l.tr_take.argtypes = [C.c_void_p, C.c_int, C.c_void_p]
    return l


def factorise(B, pivot, g):
    """|p|, p . (B + D)^-1 p by an unpivoted L D L^T factorisation; None if a pivot is not positive."""
    A = B + np.diag(pivot)
    z, d = g.copy(), np.zeros(N)
    L = np.eye(N)
    for j in range(N):
        d[j] = A[j, j]
        if not d[j] > 1e-290:
            return None
        l = A[j + 1:, j] / d[j]
        A[j + 1:, j + 1:] -= np.outer(l, A[j, j + 1:])
        z[j + 1:] -= l * z[j]
        L[j + 1:, j] = l
    back = lambda v: np.linalg.solve(L.T, v)
    p = back(z / d)
    q = np.linalg.solve(L, p)
    return float(np.sqrt(p @ p)), float((q * q / d).sum())


def search(lib, B, g, radius):
    """(rounds, what take returned, the winning multiplier) of one source's search."""
    off = np.abs(B).sum(1) - np.abs(np.diag(B))
    dec = (off == 0) & (np.diag(B) == 0) & (g == 0)
    br = C.create_string_buffer(lib.tr_size())
    lib.tr_start(br, float(max(0, -np.diag(B).min())), float(max(0, (off - np.diag(B)).max())),
                 float(np.linalg.norm(g)), radius, int(dec.any()))
    lam = [lib.tr_first(br, w) for w in range(WAVES)]
    for rnd in range(lib.tr_rounds()):
        rs = np.zeros((WAVES, 3))
        for w in range(WAVES):
            f = factorise(B, lam[w] + dec * 1.0, g)
            rs[w] = (-1.0, 0.0, lam[w]) if f is None else (
                f[0], lam[w] + f[0] ** 2 / f[1] * (f[0] - radius) / radius, lam[w])
        got = lib.tr_take(br, rnd, rs.ctypes.data)
        if got != MORE:
            return rnd + 1, got, lam[got] if got >= 0 else None
        lam = [lib.tr_next(br, w) for w in range(WAVES)]
    return lib.tr_rounds(), NONE, None


def matrix(rng, lam):
    Q, _ = np.linalg.qr(rng.normal(size=(len(lam), len(lam))))
    B = (Q * lam) @ Q.T
    return 0.5 * (B + B.T), Q


@pytest.mark.parametrize("n_zero", [1, 2, 13])
@pytest.mark.parametrize("seed", range(6))
def test_interior_step_with_vanishing_coordinates(lib, seed, n_zero):
    """Coordinates that are zero throughout B and g, the others' step inside the region."""
    rng = np.random.default_rng(seed)
    z = np.sort(rng.choice(N, n_zero, replace=False))
    rest = np.setdiff1d(np.arange(N), z)
    B, g = np.zeros((N, N)), np.zeros(N)
    B[np.ix_(rest, rest)] = matrix(rng, 10.0 ** rng.uniform(-2, 5, len(rest)))[0]
    g[rest] = B[np.ix_(rest, rest)] @ (0.3 * rng.normal(size=len(rest)) / np.sqrt(len(rest)))
    assert np.linalg.norm(np.linalg.solve(B[np.ix_(rest, rest)], g[rest])) < 1.0
    rounds, got, _ = search(lib, B, g, 1.0)
    assert got == NONE and rounds == 1
    # on the boundary the search goes on as for any other source
    radius = 0.5 * np.linalg.norm(np.linalg.solve(B[np.ix_(rest, rest)], g[rest]))
    rounds, got, lam = search(lib, B, g, radius)
    assert got >= 0 and rounds <= 8
    assert abs(np.linalg.norm(np.linalg.solve(B + lam * np.eye(N), g)) / radius - 1) <= 1.1e-7


@pytest.mark.parametrize("least", [0.0, -1e-3, -3.0, -2e4])
@pytest.mark.parametrize("seed", range(6))
def test_hard_case(lib, seed, least):
    """The least eigenvalue zero or negative, no gradient along its direction, and the step in
    the other directions at the pole half the radius or less."""
    rng = np.random.default_rng(100 + seed)
    lam = np.concatenate([[least], np.abs(least) + 10.0 ** rng.uniform(-1, 5, N - 1)])
    B, Q = matrix(rng, lam)
    y = np.concatenate([[0.0], rng.normal(size=N - 1)])
    y *= 0.45 / np.linalg.norm(y)
    g = Q @ ((lam - least) * y)
    rounds, got, lam_w = search(lib, B, g, 1.0)
    if got >= 0:   # (rounding left a gradient along the direction: a step of almost no curvature)
        d = np.linalg.eigvalsh(B).min() + lam_w
        assert d <= 1e-6 * np.linalg.norm(g)
    assert rounds <= (5 if least == 0.0 else 12 if got < 0 else 16)


@pytest.mark.parametrize("seed", range(20))
def test_ordinary_steps(lib, seed):
    """Definite and indefinite matrices of eight decades, with a gradient everywhere: the
    multiplier of the eigen-decomposition."""
    rng = np.random.default_rng(200 + seed)
    lam = 10.0 ** rng.uniform(-2, 5, N)
    k = rng.integers(0, 4)
    lam[:k] *= -(10.0 ** rng.uniform(-3, 0, k))
    B, Q = matrix(rng, lam)
    gt = rng.normal(size=N) * np.abs(lam) ** rng.uniform(0.3, 0.8)
    g = Q @ gt
    norm = lambda m: np.linalg.norm(gt / (lam + m))
    for radius in (1e-3, 1.0, 1e3):
        rounds, got, m = search(lib, B, g, radius)
        if got < 0:   # given up: only where the root is next to the pole
            assert rounds == 12 and lam.min() < 0 and norm(-lam.min() + 1e-4 * np.abs(lam).max()) <= radius
        elif lam.min() > 0 and norm(0.0) <= radius:
            assert rounds == 1 and m == 0.0
        else:
            assert lam.min() + m > 0 and abs(norm(m) / radius - 1) <= 1e-6


def test_decoupled_coordinate_with_a_gradient_is_not_left_out(lib):
    """A row of zeros in B with a gradient there: the step lies on the boundary."""
    rng = np.random.default_rng(5)
    B, g = np.zeros((N, N)), np.zeros(N)
    B[1:, 1:] = matrix(rng, 10.0 ** rng.uniform(0, 4, N - 1))[0]
    g[1:] = 0.1 * rng.normal(size=N - 1)
    g[0] = 0.5
    rounds, got, lam = search(lib, B, g, 1.0)
    assert got >= 0 and rounds <= 8
    assert abs(np.linalg.norm(np.linalg.solve(B + lam * np.eye(N), g)) - 1) <= 1.1e-7
