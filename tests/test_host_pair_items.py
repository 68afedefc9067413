"""Host build of the pair products' work items (csrc/pair_items.hpp) on the CPU: every unordered pair of blocks
is evaluated once, and every partial sum has a place of its own that the reduction reads.

The sizes reach every shape of the rule, with classes that leave the last super-row and segment partial.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
OUT = os.path.join(os.path.dirname(HERE), "_build", "pair_items_host.so")
pi = ctypes.POINTER(ctypes.c_int32)
i64 = ctypes.c_int64


@pytest.fixture(scope="module")
def lib():
    os.makedirs(os.path.dirname(OUT), exist_ok=True)
    subprocess.check_call(["g++", "-O2", "-shared", "-fPIC", "-o", OUT, os.path.join(HERE, "host", "pair_items_host.cpp")])
    L = ctypes.CDLL(OUT)
    L.pair_layout.argtypes, L.pair_layout.restype = [i64, i64, ctypes.c_int, pi, pi, pi, i64], i64
    L.pair_col_base.argtypes, L.pair_col_base.restype = [ctypes.c_int, ctypes.c_int], i64
    return L


# n_int, n_bnd, FP64 form, the shape that the rule takes: block, F, Lb
SIZES = [(1, 0, 1, (64, 1, 2)), (0, 130, 1, (64, 1, 2)), (63, 1, 1, (64, 1, 2)), (1700, 333, 1, (64, 1, 2)),
         (3300, 900, 1, (128, 1, 2)), (15361, 4740, 1, (128, 1, 4)), (24001, 6005, 1, (128, 2, 4)),
         (33003, 8101, 1, (128, 2, 8)), (51000, 9001, 1, (128, 4, 8)), (88001, 22013, 1, (128, 8, 14)),
         (100003, 30001, 1, (128, 8, 14)), (1, 1, 0, (128, 1, 2)), (4001, 1007, 0, (128, 1, 2)),
         (16477, 4119, 0, (128, 2, 4)), (30001, 7777, 0, (128, 4, 8)), (80000, 20000, 0, (128, 8, 14))]


@pytest.mark.parametrize("n_int,n_bnd,fp64,shape", SIZES)
def test_items_cover_every_pair_once(lib, n_int, n_bnd, fp64, shape):
    room = 400000
    out, it, first = (np.zeros(k, dtype=np.int32) for k in (9, 4 * room, room))
    cols = lib.pair_layout(n_int + n_bnd, n_int, fp64, *(a.ctypes.data_as(pi) for a in (out, it, first)), room)
    nb_int, nb, blk, F, Lb, nsr, nitems, max_f, max_lb = (int(v) for v in out)
    assert (blk, F, Lb) == shape and F <= max_f and Lb <= max_lb and F & (F - 1) == 0
    assert nb_int == -(-n_int // blk) and nb == nb_int - (-n_bnd // blk) and nsr == -(-nb // F)
    items = it[: 4 * nitems].reshape(nitems, 4)
    first = first[: nsr + 1]
    # a super-row's items follow each other; the reduction counts them by itself
    assert first[0] == 0 and first[nsr] == nitems
    assert np.array_equal(np.diff(first), [-(-(nb - k * F) // Lb) for k in range(nsr)])
    assert np.array_equal(items[:, 2], first[items[:, 0]] + items[:, 1])
    assert np.array_equal(np.sort(items[:, 2]), np.arange(nitems))
    # pairs b <= c, and one column partial per (block, super-row up to its own)
    pairs, places = np.zeros((nb, nb), dtype=np.int32), np.zeros(cols, dtype=np.int32)
    base = np.array([lib.pair_col_base(c, F) for c in range(nb)])
    size = []
    for k, sg, _, _ in items:
        b0, b1 = k * F, min(k * F + F, nb)
        c0, c1 = b0 + sg * Lb, min(b0 + sg * Lb + Lb, nb)
        assert c0 < c1
        for b in range(b0, b1):
            pairs[b, max(b, c0):c1] += 1
        places[base[c0:c1] + k] += 1
        size.append(sum(max(0, c1 - max(b, c0)) for b in range(b0, b1)))
    assert np.array_equal(pairs, np.triu(np.ones((nb, nb), dtype=np.int32)))
    assert np.all(places == 1)
    # the reduction of block c reads c // F + 1 places from its base on, which end where the next one's begin
    assert np.array_equal(np.append(base[1:], cols) - base, np.arange(nb) // F + 1)
    assert np.all(np.diff(size) <= 0)  # launched largest first
