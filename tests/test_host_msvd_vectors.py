"""Host build of the recurrences that the projected SVD's kernels run (csrc/msvd.hpp), on the CPU.

The pairs of a chain, the twisted solves and the maps of the setup's scan against plain loops, at every length around
their groups; and whole singular triples, formed from the same functions in the kernels' order, against the acceptance test's
bound and, with the perturbation bound residual / gap, against LAPACK's.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(os.path.dirname(HERE), "_build", "msvd_vectors_host.so")
EPS = np.finfo(float).eps
pd = ctypes.POINTER(ctypes.c_double)
ci, cd = ctypes.c_int, ctypes.c_double
LENGTHS = [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 13, 15, 16, 17, 23, 24, 25, 31, 32, 33, 60]


@pytest.fixture(scope="module")
def lib():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-o", OUT,
                           os.path.join(HERE, "host", "msvd_vectors_host.cpp")])
    L = ctypes.CDLL(OUT)
    L.chain_host.argtypes, L.chain_host.restype = [pd, pd, ci, cd, cd, pd, pd], None
    L.twisted_host.argtypes, L.twisted_host.restype = [pd, ci, ci, ci, ci, pd], None
    L.triple_host.argtypes, L.triple_host.restype = [pd, pd, ci, ci, ci, pd, pd, pd], cd
    L.rhobar2_host.argtypes, L.rhobar2_host.restype = [pd, pd, ci], cd
    return L


def _p(a):
    return a.ctypes.data_as(pd)


def _bidiagonal(kind, l, rng):
    d, e = 0.1 + rng.random(l), 0.1 + rng.random(l)
    if kind == "graded":
        g = 10.0 ** -np.linspace(0, 12, l)
        d, e = d * g, e * g
    elif kind == "reversed":
        g = 10.0 ** -np.linspace(12, 0, l)
        d, e = d * g, e * g
    elif kind == "large":
        d, e = np.ldexp(d, 400), np.ldexp(e, 400)
    elif kind == "small":
        d, e = np.ldexp(d, -400), np.ldexp(e, -400)
    return d, e


@pytest.mark.parametrize("l", LENGTHS)
@pytest.mark.parametrize("kind", ["random", "graded", "reversed"])
def test_chain_equals_its_steps(lib, kind, l):
    rng = np.random.default_rng(l)
    d, e = _bidiagonal(kind, l, rng)
    for w0 in (0.0, float(d[-1] ** 2)):
        for lam in (0.3, 1e-9, 1e-30):
            s, plain = np.zeros(l), np.zeros(l)
            lib.chain_host(_p(d ** 2), _p(e ** 2), l, w0, lam, _p(s), _p(plain))
            assert np.array_equal(s, plain)


@pytest.mark.parametrize("n", LENGTHS)
def test_twisted_solve_in_both_directions(lib, n):
    """From every start: the products of the negated multipliers in order, and nothing past them."""
    rng = np.random.default_rng(n)
    for st in (1, 2):
        mul = rng.standard_normal(st * n)
        for r in range(n):
            z = np.full(n, 7.0)
            ref = z.copy()
            ref[r] = 1.0
            for i in range(r - 1, -1, -1):
                ref[i] = -mul[st * i] * ref[i + 1]
            lib.twisted_host(_p(mul), st, n, r, -1, _p(z))
            assert np.array_equal(z, ref)
            for i in range(r, n - 1):
                ref[i + 1] = -mul[st * i] * ref[i]
            lib.twisted_host(_p(mul), st, n, r, 1, _p(z))
            assert np.array_equal(z, ref)


def _apart(kind, l, rng):
    """Bidiagonals with singular values that keep their distance, whose pairs vanish or lose range."""
    d, e = 0.1 + rng.random(l), 0.1 + rng.random(l)
    if kind == "decoupled":  # zero off-diagonal entries, 1 x 1 blocks among them
        e[rng.random(l) < 0.4] = 0.0
    elif kind == "diagonal":
        e[:] = 0.0
    elif kind == "squares":  # pivots that vanish exactly
        d, e = 0.25 * (1 + np.arange(l)), np.where(np.arange(l) % 3 == 1, 0.25, 0.0)
    elif kind != "random":
        g = 10.0 ** -np.linspace(0, int(kind[6:]), l)
        d, e = (d * g, e * g) if kind.startswith("graded") else (d * g[::-1], e * g[::-1])
    return d, e


@pytest.mark.parametrize("l", [1, 2, 3, 5, 8, 13, 24, 33, 60])
@pytest.mark.parametrize("kind", ["random", "decoupled", "diagonal", "squares", "graded22", "graded30", "graded60", "rising30"])
def test_vectors_pass_the_acceptance_test(lib, kind, l):
    """Residuals and Gram matrices of all vectors within the bounds that the kernels accept: a zero off-diagonal entry
    behind a vanishing pivot, and entries that fall by tens of decades, do not send a problem to the QR iteration."""
    for seed in range(4):
        d, e = _apart(kind, l, np.random.default_rng(100 * l + seed))
        V, U, res = np.zeros((l, l)), np.zeros((l, l)), 0.0
        for j in range(l):
            res = max(res, lib.triple_host(_p(d), _p(e), l, j, 64, _p(V[j]), _p(U[j]), _p(np.zeros(1))))
        assert res <= 1.0
        for M in (V, U):
            assert np.max(np.abs(M @ M.T - np.eye(l))) <= 1e-9


@pytest.mark.parametrize("l", [7, 10, 12, 13, 16, 31, 33, 34, 49, 56, 64, 71, 104])
@pytest.mark.parametrize("kind", ["ones", "ladder", "whole"])
def test_vectors_where_a_pivot_vanishes(lib, kind, l):
    """A zero pivot between off-diagonal entries that are not zero, also where the chain is scaled: what stands for it
    in the pivot and in the quotient after it is one number, and the acceptance test's bounds hold."""
    i = np.arange(l)
    d, e = np.ones(l), np.ones(l)
    if kind == "ladder":  # the triangular factor of the l + 1 by l bidiagonal of ones
        d, e = np.sqrt((i + 2) / (i + 1)), np.sqrt((i + 1) / (i + 2))
    elif kind == "whole":
        d, e = (np.random.default_rng(l).integers(1, 4, (2, l))).astype(float)
    V, U, res = np.zeros((l, l)), np.zeros((l, l)), 0.0
    for j in range(l):
        res = max(res, lib.triple_host(_p(d), _p(e), l, j, 64, _p(V[j]), _p(U[j]), _p(np.zeros(1))))
    assert res <= 1.0
    for M in (V, U):
        assert np.max(np.abs(M @ M.T - np.eye(l))) <= 1e-9


@pytest.mark.parametrize("l", LENGTHS)
@pytest.mark.parametrize("kind", ["random", "graded", "reversed", "large", "small"])
def test_triples(lib, kind, l):
    """Every triple passes the acceptance test's residual; its vectors stand at LAPACK's up to residual / gap."""
    rng = np.random.default_rng(1000 + l)
    d, e = _bidiagonal(kind, l, rng)
    scale = {"large": 400, "small": -400}.get(kind, 0)
    B = np.diag(np.ldexp(d, -scale)) + np.diag(np.ldexp(e[: l - 1], -scale), 1)
    U, s, Vt = np.linalg.svd(B)
    for j in range(l):
        v, u, sg = np.zeros(l), np.zeros(l), np.zeros(1)
        res = lib.triple_host(_p(d), _p(e), l, j, 64 + 64 * (j % 2), _p(v), _p(u), _p(sg))
        assert res <= 1.0, (j, res)
        assert abs(np.ldexp(sg[0], -scale) - s[j]) <= 8 * l * EPS * s[0]
        # the residual admitted above with LAPACK's own, over the distance to the next value
        gap = np.min(np.abs(np.delete(s, j) - s[j])) if l > 1 else s[0]
        slack = (1e-9 * s[j] + (64 + 8) * l * EPS * s[0]) * np.sqrt(2) / gap
        if slack < 0.1:
            assert abs(v @ Vt[j]) >= 1 - slack and abs(u @ U[:, j]) >= 1 - slack
            assert (v @ Vt[j]) * (u @ U[:, j]) > 0  # u and v of one triple


@pytest.mark.parametrize("decades", [60, 100, 107, 120, 140])
def test_values_far_below_the_largest(lib, decades):
    """A value many decades under the others is bracketed: of diag(1, 0.7, 10^-decades) with off-diagonal entries
    that leave it alone, to high relative accuracy (its square down to 1e-280 of theirs)."""
    d, e = np.array([1.0, 0.7, 10.0 ** -decades]), np.array([0.3, 10.0 ** (-2 * decades), 0.0])
    v, u, sg = np.zeros(3), np.zeros(3), np.zeros(1)
    lib.triple_host(_p(d), _p(e), 3, 2, 256, _p(v), _p(u), _p(sg))
    assert abs(sg[0] / d[2] - 1.0) <= 8 * EPS


@pytest.mark.parametrize("l", LENGTHS + [300])
@pytest.mark.parametrize("ratio", [0.01, 0.6, 1.0])
def test_maps_of_the_rotations(lib, l, ratio):
    """rhobar^2 of the composed maps against its recurrence in extended precision: positive terms only, so about
    four roundings a step and level, whatever the order."""
    rng = np.random.default_rng(l)
    a, b = np.exp(rng.standard_normal(l)), ratio * np.exp(rng.standard_normal(l))
    r2 = np.longdouble(a[0]) ** 2
    for i in range(l - 1):
        r2 = np.longdouble(a[i + 1]) ** 2 * r2 / (r2 + np.longdouble(b[i]) ** 2)
    got = lib.rhobar2_host(_p(a), _p(b), l)
    assert abs(got - float(r2)) <= 4 * (l + 10) * EPS * float(r2)
