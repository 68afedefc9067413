"""Host build of the parameter choice's terms (csrc/filter.hpp) on the CPU.

The filter factors s^2 / (s^2 + lambda^2) and lambda^2 / (s^2 + lambda^2) are quotients of ordinary size whatever the
scale of s and lambda; the kernel forms them from one reciprocal.  References: the divisions themselves (numpy, correctly
rounded), and the sums of the unscaled spectrum, which a power of two times s, lambda and f leaves alone up to its own power.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(os.path.dirname(HERE), "_build", "filter_host.so")
EPS = np.finfo(float).eps
pd = ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def lib():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-o", OUT, os.path.join(HERE, "host", "filter_host.cpp")])
    L = ctypes.CDLL(OUT)
    L.factors_host.argtypes, L.factors_host.restype = [pd, pd, pd, ctypes.c_int, pd], None
    L.sums_host.argtypes, L.sums_host.restype = [pd, pd, ctypes.c_int, ctypes.c_double, pd], None
    return L


def _factors(lib, s2, l2, f2):
    out = np.zeros((3, s2.size))
    lib.factors_host(*(a.ctypes.data_as(pd) for a in (s2, l2, f2)), s2.size, out.ctypes.data_as(pd))
    return out


def _spread(k, n=4000):
    """Values over twelve decades around 2^k."""
    rng = np.random.default_rng(abs(k))
    return np.ldexp(10.0 ** rng.uniform(-6, 6, (2, n)), k)


@pytest.mark.parametrize("k", [-1050, -1000, -700, 0, 700, 990])
def test_factors_over_the_whole_range(lib, k):
    """At every scale of the squares, subnormal ones too, the factors are the divisions' up to their roundings."""
    s2, l2 = _spread(k)
    s2, l2 = s2[s2 + l2 > 0], l2[s2 + l2 > 0]
    phi, psi, _ = _factors(lib, s2, l2, np.ones_like(s2))
    den = s2 + l2
    for got, ref in ((phi, s2 / den), (psi, l2 / den)):
        assert np.all(np.abs(got - ref) <= EPS * ref)


@pytest.mark.parametrize("k", [-900, -100, 0, 100, 900])
def test_factors_round_as_divisions(lib, k):
    """One rounding a quotient: bit for bit the correctly rounded divisions."""
    s2, l2 = _spread(k, 100000)
    f2 = np.ldexp(_spread(7, 100000)[0], k)
    den = s2 + l2
    for got, num in zip(_factors(lib, s2, l2, f2), (s2, l2, f2)):
        assert np.array_equal(got, num / den)


@pytest.mark.parametrize("k", [-520, -512, -500, 0, 500, 508])
def test_sums_do_not_depend_on_the_scale(lib, k):
    """GCV and L-curve sums of 2^k (s, lambda, f): the first's of degree 2 and 0, the others' as they are made of."""
    rng = np.random.default_rng(3)
    s, f = np.sort(10.0 ** rng.uniform(-1, 0, 40))[::-1].copy(), rng.standard_normal(40)

    def sums(c):
        out = np.zeros(8)
        a, b = np.ldexp(s, c), f.copy()
        lib.sums_host(a.ctypes.data_as(pd), b.ctypes.data_as(pd), 40, float(np.ldexp(0.3, c)), out.ctypes.data_as(pd))
        out[5:] = np.ldexp(out[5:], 2 * c)  # E, E1, E2: f^2 / s^2
        return out

    a, b = sums(0), sums(k)
    # a term's roundings, and those of squares that have become subnormal: down to 2^-1048 with a
    # step of 2^-1074
    tol = 64 * EPS + (2.0 ** -24 if k <= -512 else 0.0)
    # E's terms of order 2^-2k overflow from about 2^1024 on
    keep = slice(None) if k > -508 else slice(0, 5)
    assert np.all(np.abs(a - b)[keep] <= tol * np.abs(a)[keep])
