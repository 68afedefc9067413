"""The division-free eigenvalue count of csrc/msvd.hpp against the one by quotients, on the CPU.

Both count the eigenvalues of B^T B below x from d^2 and e^2, each exactly for a matrix whose entries
are perturbed by a few roundings; B^T B's factors determine its eigenvalues to high relative accuracy, so
the counts have to bracket each other at x (1 -+ 8 n eps).
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(os.path.dirname(HERE), "_build", "msvd_count_host.so")
EPS = np.finfo(float).eps
pd = ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def counts():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-o", OUT,
                           os.path.join(HERE, "host", "msvd_count_host.cpp")])
    L = ctypes.CDLL(OUT)
    fs = []
    for name in ("count_pairs", "count_quotients", "count_pairs_reversed"):
        f = getattr(L, name)
        f.argtypes, f.restype = [pd, pd, ctypes.c_int, ctypes.c_double], ctypes.c_int
        fs.append(lambda d2, e2, x, f=f: f(d2.ctypes.data_as(pd), e2.ctypes.data_as(pd), len(d2), float(x)))
    return fs


def _squares(kind, n, rng):
    d2, e2 = rng.random(n), rng.random(n)  # e2[n-1] is not read
    if kind == "graded":  # squares over 60 decades
        g = 10.0 ** -np.linspace(0, 60, n)
        d2, e2 = d2 * g, e2 * g
    elif kind == "decoupled":
        e2[:: max(n // 3, 1)] = 0.0
    elif kind == "integers":  # exact zero pivots at x = 1, 2, ..
        d2, e2 = np.full(n, 2.0 ** -3), np.full(n, 2.0 ** -3)
    elif kind == "tiny":  # pairs that leave their range between two rescalings
        d2, e2 = d2 * 1e-200, e2 * 1e-200
        d2[0] = 1.0
    return d2, e2


@pytest.mark.parametrize("kind", ["random", "graded", "decoupled", "integers", "tiny"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 10, 16, 17, 18, 19, 25, 26, 33, 300])
def test_counts_bracket_each_other(counts, kind, n):
    pairs, quotients, backwards = counts
    rng = np.random.default_rng(n)
    d2, e2 = _squares(kind, n, rng)
    xs = np.concatenate([10.0 ** rng.uniform(-70, 0.5, 100), rng.random(100), 2.0 ** -3 * np.arange(1, 9),
                         1e-200 * rng.random(20)])
    dr, er = d2[::-1].copy(), np.concatenate([e2[: n - 1][::-1], [0.0]])
    delta = 8 * n * EPS
    for x in xs:
        lo, hi = quotients(d2, e2, x * (1 - delta)), quotients(d2, e2, x * (1 + delta))
        assert lo <= pairs(d2, e2, x) <= hi
        lo, hi = quotients(dr, er, x * (1 - delta)), quotients(dr, er, x * (1 + delta))
        assert lo <= backwards(d2, e2, x) <= hi
