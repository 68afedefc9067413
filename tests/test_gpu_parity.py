"""GPU parity: the HIP path (through the C ABI) against the FP64 CPU oracle.

Rows of the hot path covered here: matrix entries (assembly / generation),
the products A x and A^T x in all three operator modes, the Golub-Kahan
bidiagonalisation with full reorthogonalisation, the projected SVD, the
parameter choice, the projected solution, the lift, the evaluation and the
whole solve, at small sizes (several tiles plus a ragged tail) element by
element; at full size (unit ball, n = 100000) the products on sampled rows,
the Golub-Kahan relations, and the benchmark's stored FP64 HKT + GCV solve
step by step against the oracle on the GPU's Krylov scalars.

Tolerances (derivations in the design notes):
* FP64 entries: |dA_ij| <= 4e-15 |A_ij| (both sides evaluate the same closed
  form with a few roundings each);
* FP64 products: |dy_i| <= 1e-13 (|A||x|)_i, the natural error scale of a
  length-n dot product in FP64 with different summation orders;
* FP32-evaluated entries: |dA_ij| <= 4e-6 |A_ij| (nodes rounded to FP32,
  one FP32 rsqrt and a few FP32 operations); products |dy_i| <= 4e-6 (|A||x|)_i;
* leading Ritz values (top 10): relative 1e-12 (the required bar); all Ritz
  values: absolute 64 l eps s_1 (dense SVD accuracy of the oracle);
* solution u at the evaluation points: relative 1e-8 at the oracle's lambda;
  coefficients: relative 1e-6.
"""
import math
import sys

import numpy as np
import pytest

from paper_2511_09798_amd import inputs as I

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def say(*a):
    print("[gpu-case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def mq():
    from paper_2511_09798_amd import mqhelm

    return mqhelm


def _problem(mq, p, mode):
    say("create", p.name, "mode", mode, "n", p.n)
    return mq.Problem(p.x_int, p.x_bnd, p.kappa, p.eps, mode)


SMALL = [
    ("cube_ragged", lambda: I.cube_scaled(333, 190, kappa=6.0, eps=2.0, ell=40)),
    ("sphere_ragged", lambda: I.sphere_scaled(517, 260, kappa=9.0, eps=3.0, ell=40)),
]


# ---------------------------------------------------------------------------
# entries
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("name,make", SMALL)
@pytest.mark.parametrize("mode", ["stored_fp64", "matfree_fp64", "matfree_fp32"])
def test_entries(mq, orc, name, make, mode):
    p = make()
    A = orc.assemble(p.nodes, p.n_int, p.kappa, p.eps)
    with _problem(mq, p, mode) as pr:
        say("matrix_rows", name, mode)
        R = pr.matrix_rows(0, p.n)
    tol = 4e-6 if mode == "matfree_fp32" else 4e-15
    assert np.all(np.abs(R - A) <= tol * np.abs(A)), float(np.max(np.abs(R - A) / np.abs(A)))


# ---------------------------------------------------------------------------
# products
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("name,make", SMALL + [("cube_n1800", I.cube_small)])
@pytest.mark.parametrize("mode", ["stored_fp64", "matfree_fp64", "matfree_fp32"])
def test_products(mq, orc, name, make, mode):
    p = make()
    A = orc.assemble(p.nodes, p.n_int, p.kappa, p.eps)
    x = I.random_vector(p.n, 11)
    z = I.random_vector(p.n, 12)
    tol = 4e-6 if mode == "matfree_fp32" else 1e-13
    with _problem(mq, p, mode) as pr:
        for trans in (False, True):
            say("apply", name, mode, "trans", trans)
            y = pr.apply(x, trans=trans)
            ref = orc.apply(A, p.nodes, p.n_int, p.kappa, p.eps, x, trans=trans)
            scale = (np.abs(A.T) if trans else np.abs(A)) @ np.abs(x)
            assert np.all(np.abs(y - ref) <= tol * scale), float(np.max(np.abs(y - ref) / scale))
            say("apply shifted", name, mode, "trans", trans)
            y2 = pr.apply(x, trans=trans, shift=0.75, z=z)
            scale2 = scale + 0.75 * np.abs(z)
            assert np.all(np.abs(y2 - (ref - 0.75 * z)) <= tol * scale2)


@pytest.mark.parametrize("n_int,n_bnd", [(1, 1), (127, 129), (128, 128), (257, 1), (130, 0), (0, 131), (1300, 500)])
@pytest.mark.parametrize("row_scale", [0, 1])
def test_stored_pair_values(mq, orc, n_int, n_bnd, row_scale):
    """Stored tiles hold one value per pair of nodes: rows and both products at tile edges and with an
    empty class (the interior row's mixed entries are formed from phi)."""
    nodes = I.random_nodes_cube(n_int + n_bnd, 77)
    xi, xb = (nodes[:n_int] if n_int else None), (nodes[n_int:] if n_bnd else None)
    kappa, eps = 7.0, 2.5
    A = orc.assemble(nodes, n_int, kappa, eps)
    A[:n_int] *= 1.0 / (3 * eps * eps + kappa * kappa) if row_scale else 1.0
    x, z = I.random_vector(n_int + n_bnd, 3), I.random_vector(n_int + n_bnd, 4)
    with mq.Problem(xi, xb, kappa, eps, "stored_fp64") as pr:
        say("stored pairs", n_int, n_bnd, row_scale)
        R = pr.matrix_rows(0, pr.n, row_scale=row_scale)
        ys = [pr.apply(x, trans=t, shift=0.5, z=z, row_scale=row_scale) for t in (False, True)]
    # the interior row's mixed entry adds the rounding of phi and of its reciprocal: about 8 eps
    assert np.all(np.abs(R - A) <= 4e-15 * np.abs(A))
    for y, M in zip(ys, (A, A.T)):
        assert np.all(np.abs(y - (M @ x - 0.5 * z)) <= 1e-13 * (np.abs(M) @ np.abs(x) + np.abs(z)))


@pytest.mark.parametrize("row_scale", [0, 1])
@pytest.mark.parametrize("kappa,eps", [(7.0, 2.5), (0.5, 12.0), (40.0, 0.3)])
def test_stored_entries_round_once(mq, kappa, eps, row_scale):
    """The stored matrix holds the entries that the formula gives, bit for bit, whatever its tiles keep."""
    nodes = I.random_nodes_cube(700, 79)
    R = {}
    for mode in ("stored_fp64", "matfree_fp64"):
        with mq.Problem(nodes[:430], nodes[430:], kappa, eps, mode) as pr:
            say("stored entries", mode, kappa, eps, row_scale)
            R[mode] = pr.matrix_rows(0, pr.n, row_scale=row_scale)
    assert np.array_equal(R["stored_fp64"], R["matfree_fp64"])


@pytest.mark.parametrize("n_int,n_bnd", [(63, 1), (64, 65), (3300, 900), (15361, 4740)])
def test_fp64_pair_product_shapes(mq, n_int, n_bnd):
    """The FP64 pair products' work shapes (blocks of 64 nodes; 1 x 2 and 1 x 4 blocks of 128) with ragged
    classes against the stored products; all entries are positive, so |A||x| = A|x|."""
    nodes = I.random_nodes_cube(n_int + n_bnd, 78)
    x = I.random_vector(n_int + n_bnd, 5)
    ys = {}
    for mode in ("stored_fp64", "matfree_fp64"):
        with mq.Problem(nodes[:n_int], nodes[n_int:], 9.0, 3.0, mode) as pr:
            say("pair product shapes", mode, n_int, n_bnd)
            ys[mode] = [(pr.apply(x, trans=t), pr.apply(np.abs(x), trans=t)) for t in (False, True)]
    for (y, sc), (ref, _) in zip(ys["matfree_fp64"], ys["stored_fp64"]):
        assert np.all(np.abs(y - ref) <= 2e-13 * sc)  # 1e-13 for each side


@pytest.mark.parametrize("n_int,n_bnd", [(24001, 6005), (33003, 8101), (51000, 9001), (88001, 22013)])
def test_fp64_pair_product_super_rows(mq, n_int, n_bnd):
    """The FP64 pair products' shapes with several fixed blocks an item (2 x 4, 2 x 8, 4 x 8 and 8 x 14 blocks of
    128), the last super-row and segment partial, against the stored products (positive entries: |A||x| = A|x|)."""
    nodes = I.random_nodes_cube(n_int + n_bnd, 80)
    x = I.random_vector(n_int + n_bnd, 5)
    ys = {}
    for mode in ("stored_fp64", "matfree_fp64"):
        with mq.Problem(nodes[:n_int], nodes[n_int:], 9.0, 3.0, mode) as pr:
            say("pair product super-rows", mode, n_int, n_bnd)
            ys[mode] = [(pr.apply(x, trans=t), pr.apply(np.abs(x), trans=t)) for t in (False, True)]
    for (y, sc), (ref, _) in zip(ys["matfree_fp64"], ys["stored_fp64"]):
        assert np.all(np.abs(y - ref) <= 2e-13 * sc)  # 1e-13 for each side


@pytest.mark.parametrize("n,ell", [(70, 60), (2047, 140), (2049, 40)])
def test_reorthogonalisation_forms(mq, orc, n, ell):
    """Runs across the small form's limits (64 blocks of 32 rows, 8192 partials): Golub-Kahan relations and
    orthonormal bases, and lockstep runs equal to single ones bit for bit."""
    n_int = int(0.8 * n)
    p = I.cube_scaled(n_int, n - n_int, kappa=12.0, eps=3.4, ell=ell)
    A = orc.assemble(p.nodes, p.n_int, p.kappa, p.eps)
    F = np.stack([p.rhs, I.random_vector(n, 6)])
    with _problem(mq, p, "matfree_fp64") as pr:
        say("gkb", n, ell)
        g = [pr.gkb(f, ell) for f in F]
        m = pr.gkb_multi(F, ell)
    for k in range(2):
        W, Z, C = g[k]["W"].T, g[k]["Z"].T, orc.bidiag_matrix(g[k]["alpha"], g[k]["beta"])
        assert g[k]["ell_done"] == ell
        assert np.linalg.norm(A @ Z - W @ C) / np.linalg.norm(C, 2) < 1e-12
        assert np.max(np.abs(W.T @ W - np.eye(ell + 1))) < 1e-12 and np.max(np.abs(Z.T @ Z - np.eye(ell))) < 1e-12
        for key in ("W", "Z", "alpha", "beta"):
            assert np.array_equal(g[k][key], m[key][k]), key


@pytest.mark.parametrize("mode", ["stored_fp64", "matfree_fp64"])
@pytest.mark.parametrize("n,nrhs,ell", [(2100, 16, 40), (4003, 9, 12), (20001, 2, 5)])
def test_lockstep_sums_by_their_own_launch(mq, mode, n, nrhs, ell):
    """Groups whose row blocks no longer fit one round sum the projection coefficients by a launch of their
    own, a run alone in the kernel that needs them: the bits are the same."""
    n_int = int(0.8 * n)
    p = I.cube_scaled(n_int, n - n_int, kappa=12.0, eps=3.4, ell=ell)
    F = np.stack([I.random_vector(n, 60 + k) for k in range(nrhs)])
    with _problem(mq, p, mode) as pr:
        say("lockstep sums", mode, n, nrhs, ell)
        m = pr.gkb_multi(F, ell)
        for k in (0, nrhs - 1):
            g = pr.gkb(F[k], ell)
            assert g["ell_done"] == ell
            for key in ("W", "Z", "alpha", "beta"):
                assert np.array_equal(g[key], m[key][k]), key


@pytest.mark.parametrize("m", [1, 63, 64, 65, 1025])
@pytest.mark.parametrize("n", [1, 48, 49, 385, 2100])
def test_evaluation_shapes(mq, orc, n, m):
    """Points and centres around a wave and a slice, from host and device arrays (equal
    bit for bit), and a point that is not finite: refused, u left as it was."""
    import torch

    n_int = n // 2
    nodes, pts, coef = I.random_nodes_cube(n, 3), I.random_nodes_cube(m, 4), I.random_vector(n, 5)
    r2 = np.sum((pts[:, None, :] - nodes[None, :, :]) ** 2, axis=2)
    phi = np.sqrt(1.0 + 9.0 * r2)
    with mq.Problem(nodes[:n_int], nodes[n_int:], 9.0, 3.0, "matfree_fp64") as pr:
        say("evaluation shapes", n, m)
        u = pr.eval(coef, pts)
        cd, xd, ud = torch.from_numpy(coef).cuda(), torch.from_numpy(pts).cuda(), torch.full((m,), 7.0).cuda().double()
        torch.cuda.synchronize()
        pr.eval(cd, xd, ud)
        assert np.array_equal(ud.cpu().numpy(), u)
        xd[m - 1, 2] = float("nan")
        ud.fill_(7.0)
        with pytest.raises(mq.MQHError):
            pr.eval(cd, xd, ud)
        assert bool((ud == 7.0).all())
        xd.copy_(torch.from_numpy(pts))
        assert np.array_equal(pr.eval(cd, xd).cpu().numpy(), u)
    # n roundings of the sum, about eight of a term
    assert np.all(np.abs(u - phi @ coef) <= (n + 8) * EPS * (phi @ np.abs(coef)))


@pytest.mark.parametrize("mode", ["stored_fp64", "matfree_fp64", "matfree_fp32"])
@pytest.mark.parametrize("trans", [False, True])
def test_products_in_place_vectors(mq, mode, trans):
    """Device vectors read and written where they are: at an odd element, z the output itself, z one element off
    it, and x the output; the bits of the staged product of host arrays every time."""
    import torch

    n = 1003
    nodes, x, z = I.random_nodes_cube(n, 8), I.random_vector(n, 5), I.random_vector(n, 6)
    with mq.Problem(nodes[:700], nodes[700:], 9.0, 3.0, mode) as pr:
        say("products in place", mode, trans)
        ref = pr.apply(x, trans=trans, shift=0.7, z=z)
        buf = torch.zeros(4 * n, dtype=torch.float64, device="cuda:0")
        xd, zd = buf[1:n + 1], buf[n + 2:2 * n + 2]
        yd = buf[2 * n + 5:3 * n + 5]

        def run(xv, zv, yv):
            xv.copy_(torch.from_numpy(x))
            zv.copy_(torch.from_numpy(z))
            torch.cuda.synchronize()
            mq.mqh_apply(pr.h, trans, xv, 0.7, zv, yv)
            return yv.cpu().numpy()

        assert np.array_equal(run(xd, zd, yd), ref)
        assert np.array_equal(run(xd, yd, yd), ref)
        assert np.array_equal(run(xd, zd, buf[n + 3:2 * n + 3]), ref)
        assert np.array_equal(run(xd, zd, xd), ref)


class _DeviceBytes:
    """hipMalloc'ed bytes of exactly the size asked for (the page they end in is mapped whole)."""

    def __init__(self, mq, size):
        import ctypes

        self.lib, self.p = mq.lib, ctypes.c_void_p()
        self.lib.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
        self.lib.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
        self.lib.hipFree.argtypes = [ctypes.c_void_p]
        assert self.lib.hipMalloc(ctypes.byref(self.p), size) == 0
        self.size = size

    def put(self, a, off=0):
        assert off + a.nbytes <= self.size
        assert self.lib.hipMemcpy(self.p.value + off, a.ctypes.data, a.nbytes, 1) == 0
        return self.p.value + off

    def get(self, count, off=0):
        a = np.empty(count)
        assert self.lib.hipMemcpy(a.ctypes.data, self.p.value + off, a.nbytes, 2) == 0
        return a

    def free(self):
        self.lib.hipFree(self.p)


@pytest.mark.parametrize("mode", ["stored_fp64", "matfree_fp64"])
@pytest.mark.parametrize("off", [2, 4])
def test_device_arrays_at_any_address(mq, mode, off):
    """Device arrays that do not start at a double's address (2 or 4 bytes past one): the bits of host arrays."""
    n, m = 1003, 130
    nodes, x, z, pts = I.random_nodes_cube(n, 8), I.random_vector(n, 5), I.random_vector(n, 6), I.random_nodes_cube(m, 9)
    bufs = [_DeviceBytes(mq, 8 * k + 8) for k in (n, n, n, 3 * m, m)]
    with mq.Problem(nodes[:700], nodes[700:], 9.0, 3.0, mode) as pr:
        say("device arrays at any address", mode, off)
        ref, uref = pr.apply(x, trans=True, shift=0.7, z=z), pr.eval(x, pts)
        xp, zp, yp = bufs[0].put(x, off), bufs[1].put(z, off), bufs[2].p.value + off
        assert mq.lib.mqh_apply(pr.h, 1, xp, 0.7, zp, yp, mq.MQH_FLAG_DEVICE_PTRS) == 0
        assert np.array_equal(bufs[2].get(n, off), ref)
        ep, up = bufs[3].put(pts.ravel(), off), bufs[4].p.value + off
        assert mq.lib.mqh_eval(pr.h, xp, ep, m, up, mq.MQH_FLAG_DEVICE_PTRS) == 0
        assert np.array_equal(bufs[4].get(m, off), uref)
    for b in bufs:
        b.free()


def test_device_arrays_too_short(mq):
    """A device array one element short of what the call takes is refused, whichever it is, and outputs that do
    fit stay as they were.  (The missing element lies in the array's last page: nothing outside mapped memory.)"""
    n, m = 1003, 130
    nodes, x, z, pts = I.random_nodes_cube(n, 8), I.random_vector(n, 5), I.random_vector(n, 6), I.random_nodes_cube(m, 9)
    mark = np.full(n, 7.0)
    with mq.Problem(nodes[:700], nodes[700:], 9.0, 3.0, "matfree_fp64") as pr:
        for short in range(3):
            say("device arrays too short", "apply", short)
            bufs = [_DeviceBytes(mq, 8 * (n - (k == short))) for k in range(3)]
            ps = [b.put(a[: n - (k == short)]) for k, (b, a) in enumerate(zip(bufs, (x, z, mark)))]
            assert mq.lib.mqh_apply(pr.h, 0, ps[0], 0.7, ps[1], ps[2], mq.MQH_FLAG_DEVICE_PTRS) < 0
            left = n - (short == 2)
            assert np.array_equal(bufs[2].get(left), mark[:left])
            for b in bufs:
                b.free()
        for short in range(3):
            say("device arrays too short", "eval", short)
            data = (x, pts.ravel(), mark[:m])
            bufs = [_DeviceBytes(mq, a.nbytes - 8 * (k == short)) for k, a in enumerate(data)]
            ps = [b.put(a[: a.size - (k == short)]) for k, (b, a) in enumerate(zip(bufs, data))]
            assert mq.lib.mqh_eval(pr.h, ps[0], ps[1], m, ps[2], mq.MQH_FLAG_DEVICE_PTRS) < 0
            left = m - (short == 2)
            assert np.array_equal(bufs[2].get(left), mark[:left])
            for b in bufs:
                b.free()
        R = pr.matrix_rows(0, n)  # and the problem still works
        assert np.all(np.abs(pr.apply(x) - R @ x) <= 1e-13 * (R @ np.abs(x)))


def test_products_device_pointers(mq, orc):
    import torch

    p = I.cube_scaled(300, 200, kappa=4.0, eps=2.0, ell=10)
    A = orc.assemble(p.nodes, p.n_int, p.kappa, p.eps)
    x = I.random_vector(p.n, 5)
    with _problem(mq, p, "matfree_fp64") as pr:
        say("apply device pointers")
        xd = torch.from_numpy(x).cuda()
        yd = pr.apply(xd, trans=True)
        torch.cuda.synchronize()
        y = yd.cpu().numpy()
    ref = orc.apply(A, p.nodes, p.n_int, p.kappa, p.eps, x, trans=True)
    assert np.all(np.abs(y - ref) <= 1e-13 * (np.abs(A.T) @ np.abs(x)))


# ---------------------------------------------------------------------------
# Golub-Kahan bidiagonalisation
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("mode", ["stored_fp64", "matfree_fp64"])
def test_gkb_against_oracle(mq, orc, mode):
    p = I.cube_small()
    A = orc.assemble(p.nodes, p.n_int, p.kappa, p.eps)
    g = orc.gkb(A, p.nodes, p.n_int, p.kappa, p.eps, p.rhs, p.ell)
    with _problem(mq, p, mode) as pr:
        say("gkb", mode)
        r = pr.gkb(p.rhs, p.ell)
    assert r["ell_done"] == g.ell == p.ell and r["status"] == 0
    W, Z = r["W"].T, r["Z"].T
    C = orc.bidiag_matrix(r["alpha"], r["beta"])
    c2 = np.linalg.norm(C, 2)
    # Krylov relations and orthonormality of the GPU bases
    assert np.linalg.norm(A @ Z - W @ C) / c2 < 1e-12
    assert np.max(np.abs(W.T @ W - np.eye(p.ell + 1))) < 1e-12
    assert np.max(np.abs(Z.T @ Z - np.eye(p.ell))) < 1e-12
    assert r["beta"][0] == pytest.approx(g.beta[0], rel=1e-14)
    # leading Ritz values (top 10) and the first Krylov scalars
    s_gpu = np.linalg.svd(C, compute_uv=False)
    s_orc = np.linalg.svd(orc.bidiag_matrix(g.alpha, g.beta), compute_uv=False)
    assert np.max(np.abs(s_gpu[:10] - s_orc[:10]) / s_orc[:10]) < 1e-12
    assert np.max(np.abs(r["alpha"][:5] - g.alpha[:5]) / g.alpha[:5]) < 1e-12


def test_gkb_fp32_entries_close_to_fp64(mq, orc):
    p = I.cube_small()
    g = orc.gkb(None, p.nodes, p.n_int, p.kappa, p.eps, p.rhs, 20)
    with _problem(mq, p, "matfree_fp32") as pr:
        say("gkb fp32")
        r = pr.gkb(p.rhs, 20)
    s_gpu = np.linalg.svd(orc.bidiag_matrix(r["alpha"], r["beta"]), compute_uv=False)
    s_orc = np.linalg.svd(orc.bidiag_matrix(g.alpha, g.beta), compute_uv=False)
    assert np.max(np.abs(s_gpu[:5] - s_orc[:5]) / s_orc[:5]) < 1e-5
    W, Z = r["W"].T, r["Z"].T
    assert np.max(np.abs(W.T @ W - np.eye(21))) < 1e-12  # reorthogonalisation stays FP64


def test_gkb_breakdown_full_space(mq, orc):
    n = 16
    X = I.random_nodes_cube(n, 116)
    f = I.random_vector(n, 7)
    say("gkb breakdown l = n")
    with mq.Problem(X[:8], X[8:], 2.0, 6.0, "stored_fp64") as pr:
        r = pr.gkb(f, n)
    g = orc.gkb(None, X, 8, 2.0, 6.0, f, n)
    assert r["ell_done"] == g.ell == n
    assert r["status"] == mq.MQH_WBREAKDOWN and r["beta"][n] == 0.0
    s_gpu = np.linalg.svd(orc.bidiag_matrix(r["alpha"], r["beta"]), compute_uv=False)
    A = orc.assemble(X, 8, 2.0, 6.0)
    sv = np.linalg.svd(A, compute_uv=False)
    assert np.max(np.abs(s_gpu - sv) / sv) < 1e-10


def test_gkb_zero_rhs(mq):
    X = I.random_nodes_cube(40, 3)
    say("gkb zero rhs")
    with mq.Problem(X[:20], X[20:], 2.0, 3.0, "matfree_fp64") as pr:
        r = pr.gkb(np.zeros(40), 5)
        assert r["ell_done"] == 0 and r["status"] == mq.MQH_WBREAKDOWN
        out = pr.solve(np.zeros(20), np.zeros(20), 5)
        assert out.status == mq.MQH_WBREAKDOWN and np.all(out.coef == 0.0)


# ---------------------------------------------------------------------------
# projected problem
# ---------------------------------------------------------------------------

@pytest.fixture(scope="module")
def proj_case(orc):
    p = I.cube_scaled(400, 240, kappa=3.0, eps=0.7, ell=80)
    g = orc.gkb(None, p.nodes, p.n_int, p.kappa, p.eps, p.rhs, p.ell)
    s, ft, V = orc.proj_svd(g.alpha, g.beta)
    return p, g, s, ft, V


def test_proj_svd(mq, orc, proj_case):
    p, g, s, ft, V = proj_case
    say("proj_svd l =", g.ell)
    sv, ftg, Vg = mq.mqh_proj_svd(g.alpha, g.beta)
    Vg = Vg.T  # columns v~_i
    assert np.max(np.abs(sv[:10] - s[:10]) / s[:10]) < 1e-12
    assert np.max(np.abs(sv - s)) < 64 * g.ell * EPS * s[0]
    assert abs(abs(ftg[-1]) - abs(ft[-1])) < 1e-12 * g.beta[0]
    assert np.sum(ftg ** 2) == pytest.approx(g.beta[0] ** 2, rel=1e-13)
    assert np.max(np.abs(Vg.T @ Vg - np.eye(g.ell))) < 1e-12
    # sign-invariant comparison: projected Tikhonov solutions at a few lambdas
    for lam in (s[0] * 1e-1, s[5], s[30], s[-1] * 10):
        y = Vg @ (sv / (sv ** 2 + lam ** 2) * ftg[:-1])
        yo = orc.y_tikhonov(s, ft, V, lam)
        assert np.linalg.norm(y - yo) <= 1e-9 * np.linalg.norm(yo)


@pytest.mark.parametrize("ell", [1, 2, 7])
def test_proj_svd_small(mq, orc, ell):
    rng = np.random.default_rng(ell)
    a = rng.random(ell) + 0.2
    b = np.concatenate([[1.5], rng.random(ell) + 0.2])
    say("proj_svd small", ell)
    sv, ftg, Vg = mq.mqh_proj_svd(a, b)
    s, ft, V = orc.proj_svd(a, b)
    assert np.max(np.abs(sv - s) / s) < 1e-13
    assert np.max(np.abs(np.abs(ftg) - np.abs(ft))) < 1e-13


@pytest.mark.parametrize("kind", ["positive", "signed", "steep"])
@pytest.mark.parametrize("ell", [1, 2, 8, 9, 17, 63, 65, 128, 256, 257, 512, 513, 1000])
def test_projected_problem_shapes(mq, orc, kind, ell):
    """Lengths around the kernels' groups, strips and thread rules, with the coefficients that the scan of
    the rotations takes (positive), leaves to the rotations (signed), or gives back to them from about
    80 steps on (steep: rhobar falls by 30 a step).  LAPACK's backward error, l eps s_1, is the bound of a value."""
    rng = np.random.default_rng(ell)
    a = np.exp(0.3 * rng.standard_normal(ell)) * (rng.choice([-1.0, 1.0], ell) if kind == "signed" else 1.0)
    b = np.concatenate([[2.0], np.exp(0.3 * rng.standard_normal(ell)) * (30.0 if kind == "steep" else 0.6)])
    C = orc.bidiag_matrix(a, b)
    rhs = np.zeros(ell + 1)
    rhs[0] = b[0]
    U, s, Vt = np.linalg.svd(C)
    say("projected shapes", kind, ell)
    sv, ft, V = mq.mqh_proj_svd(a, b)
    assert np.max(np.abs(sv - s)) <= 8 * ell * EPS * s[0]
    assert np.max(np.abs(V @ V.T - np.eye(ell))) <= 64 * ell * EPS
    assert np.max(np.abs(np.linalg.norm(C @ V.T, axis=0) - sv)) <= 64 * ell * EPS * s[0]  # ||C v_i|| = s_i
    # the Tikhonov solution at s_1 / 10: a condition of 101 on a backward error of l eps
    lam = 0.1 * s[0]
    f = U.T @ rhs
    y0 = Vt.T @ (s / (s ** 2 + lam ** 2) * f[:ell])
    y = mq.mqh_proj_solution(sv, ft, V, mq.MQH_METHOD_HKT, lam)
    assert np.linalg.norm(y - y0) <= 101 * 8 * ell * EPS * np.linalg.norm(y0)
    # the GCV curve over grids below, at and past one pass: sums of positive terms, then (l + 1) - tr, from
    # which at least 1 is left of l
    for J in (3, 256, 259):
        ch = mq.mqh_param_choice(sv, ft, mq.MQH_METHOD_HKT, mq.MQH_RULE_GCV, n_grid=J, want_curve=True)
        lo = max(sv[-1], 16 * EPS * sv[0])
        lo = lo if lo < sv[0] else 16 * EPS * sv[0]
        lams = np.exp(np.linspace(np.log(lo), np.log(sv[0]), J))[:, None]
        psi, phi = lams ** 2 / (sv ** 2 + lams ** 2), sv ** 2 / (sv ** 2 + lams ** 2)
        ref = (np.sum((psi * ft[:-1]) ** 2, axis=1) + ft[-1] ** 2) / (ell + 1 - np.sum(phi, axis=1)) ** 2
        # exp of a logarithm of up to 40 in size: 40 eps of lambda, four times that of the squared terms
        assert np.max(np.abs(ch["curve"] - ref) / ref) <= (8 * ell * ell + 1024) * EPS


@pytest.mark.parametrize("k", [-520, 508])
def test_gcv_does_not_depend_on_the_scale(mq, k):
    """The GCV curve of 2^k times the singular values: the same values at 2^k times the grid, also where the
    squares are subnormal or near the largest number; a given lambda's criterion too."""
    rng = np.random.default_rng(3)
    s, f = np.sort(10.0 ** rng.uniform(-1, 0, 70))[::-1].copy(), rng.standard_normal(71)
    say("gcv scale", k)
    a = mq.mqh_param_choice(s, f, mq.MQH_METHOD_HKT, mq.MQH_RULE_GCV, n_grid=300, want_curve=True)
    b = mq.mqh_param_choice(np.ldexp(s, k), f, mq.MQH_METHOD_HKT, mq.MQH_RULE_GCV, n_grid=300, want_curve=True)
    # lambda as exp of a logarithm of up to 362: 362 eps of it; squares down to 2^-1047 with a step of 2^-1074
    # (both sums are of positive terms, and at least 1 of 71 is left of the trace term)
    tol = 71 * (8 * 362 * EPS + 2.0 ** -25)
    assert np.all(np.abs(a["curve"] - b["curve"]) <= tol * a["curve"])
    lam = 0.3
    c = [mq.mqh_param_choice(np.ldexp(s, q), f, mq.MQH_METHOD_HKT, mq.MQH_RULE_FIXED, lambda_fixed=float(np.ldexp(lam, q)))
         for q in (0, k)]
    assert abs(c[0]["crit"] - c[1]["crit"]) <= tol * c[0]["crit"]


@pytest.mark.parametrize("ell", [2, 9, 30, 65, 300])
@pytest.mark.parametrize("kind", ["zero_beta", "zero_beta_signed", "one_by_one", "graded30", "rising30"])
def test_proj_svd_fast_path_accepts(mq, kind, ell):
    """The fast path alone on C_l with zero beta (B then falls apart; a singular value may be a coefficient
    itself) and with coefficients over 30 decades: accepted, with the QR iteration's values."""
    rng = np.random.default_rng(ell)
    a, b = rng.random(ell) + 0.1, np.concatenate([[2.0], rng.random(ell) + 0.1])
    if kind.startswith("zero_beta"):
        b[1:][rng.random(ell) < 0.3] = 0.0
        a *= rng.choice([-1.0, 1.0], ell) if kind.endswith("signed") else 1.0
    elif kind == "one_by_one":
        a, b[1:] = 0.25 * (1 + np.arange(ell)), 0.0
    else:
        g = 10.0 ** -np.linspace(0, 30, ell)
        g = g if kind == "graded30" else g[::-1]
        a, b[1:] = a * g, b[1:] * g
    say("fast path accepts", kind, ell)
    sv, ft, V = mq.mqh_proj_svd(a, b, path="fast")
    s2, f2, _ = mq.mqh_proj_svd(a, b, path="qr")
    assert np.max(np.abs(sv / s2 - 1.0)) <= 256 * EPS
    assert np.max(np.abs(V @ V.T - np.eye(ell))) <= 64 * ell * EPS
    # a bidiagonal fixes a vector to eps over the relative distance of its value to the next
    gap = np.minimum(np.abs(np.diff(s2, prepend=np.inf)), np.abs(np.diff(s2, append=-np.inf))) / s2
    assert np.all(np.abs(np.abs(ft[:-1]) - np.abs(f2[:-1])) <= 64 * ell * EPS * b[0] / np.minimum(gap, 1.0))


@pytest.mark.parametrize("ell", [20, 33, 49, 56, 71, 111])
@pytest.mark.parametrize("flip", [False, True])
def test_proj_svd_fast_path_accepts_vanishing_pivots(mq, flip, ell):
    """alpha and beta of ones: the chains of a value meet zero pivots, also where they are scaled.  The fast path alone
    is accepted, with the values 2 cos(k pi / (2 ell + 2)) that such a bidiagonal has."""
    sg = np.random.default_rng(ell).choice([-1.0, 1.0], 2 * ell) if flip else np.ones(2 * ell)
    say("vanishing pivots", ell, flip)
    sv, ft, V = mq.mqh_proj_svd(sg[:ell], np.concatenate([[2.0], sg[ell:]]), path="fast")
    want = 2.0 * np.cos(np.arange(1, ell + 1) * np.pi / (2 * ell + 2))
    assert np.all(np.abs(sv - want) <= 4 * ell * EPS * want[0])
    assert np.max(np.abs(V @ V.T - np.eye(ell))) <= 1e-9


def _decaying(l, seed):
    # a spectrum like that of a Golub-Kahan run on an ill-posed operator
    rng = np.random.default_rng(seed)
    a = np.logspace(0, -7, l) * (1.0 + 0.3 * rng.random(l))
    b = np.concatenate([[1.0], np.logspace(-0.3, -7.3, l) * (1.0 + 0.3 * rng.random(l))])
    return a, b


@pytest.mark.parametrize("source", ["gkb", "decaying300", "decaying1024"])
def test_proj_svd_fast_path_and_qr(mq, orc, proj_case, source):
    # the fast path alone (multisection + twisted factorisations) and the QR
    # iteration alone, each against the oracle's one-sided Jacobi SVD (values,
    # |f~|) and against each other (projected Tikhonov solutions)
    if source == "gkb":
        g = proj_case[1]
        a, b = g.alpha, g.beta
    else:
        a, b = _decaying(int(source[8:]), 5)
    l = len(a)
    say("proj_svd paths", source, "l =", l)
    sf, ff, Vf = mq.mqh_proj_svd(a, b, path="fast")
    sq, fq, Vq = mq.mqh_proj_svd(a, b, path="qr")
    sd, fd, Vd = mq.mqh_proj_svd(a, b)
    assert np.array_equal(sd, sf) and np.array_equal(fd, ff) and np.array_equal(Vd, Vf)  # no fallback needed
    s, ft, V = orc.proj_svd(a, b)
    for sv, ftg, Vg in ((sf, ff, Vf), (sq, fq, Vq)):
        assert np.max(np.abs(sv[:10] - s[:10]) / s[:10]) < 1e-12
        assert np.max(np.abs(sv - s)) < 64 * l * EPS * s[0]
        assert abs(abs(ftg[-1]) - abs(ft[-1])) < 1e-12 * b[0]
        assert np.sum(ftg ** 2) == pytest.approx(b[0] ** 2, rel=1e-13)
        assert np.max(np.abs(Vg @ Vg.T - np.eye(l))) < 1e-12
    assert np.max(np.abs(sf - sq) / sq) < 256 * EPS
    assert np.max(np.abs(np.abs(ff) - np.abs(fq))) < 1e-12 * b[0]
    for lam in (sq[0] * 1e-2, sq[l // 3], sq[-1] * 10):
        yf = Vf.T @ (sf / (sf ** 2 + lam ** 2) * ff[:-1])
        yq = Vq.T @ (sq / (sq ** 2 + lam ** 2) * fq[:-1])
        assert np.linalg.norm(yf - yq) <= 1e-9 * np.linalg.norm(yq)


def test_proj_svd_exact_cluster_falls_back(mq, orc):
    # two identical decoupled blocks: double singular values, rejected by the
    # fast path's acceptance test and computed by the QR iteration
    blk_a = np.array([1.0, 0.7, 0.4])
    blk_b = np.array([0.6, 0.3, 0.0])
    a = np.concatenate([blk_a, blk_a])
    b = np.concatenate([[1.0], blk_b, blk_b])
    say("proj_svd exact cluster")
    with pytest.raises(mq.MQHError) as ex:
        mq.mqh_proj_svd(a, b, path="fast")
    assert "acceptance test" in str(ex.value)
    sd, fd, Vd = mq.mqh_proj_svd(a, b)
    sq, fq, Vq = mq.mqh_proj_svd(a, b, path="qr")
    assert np.array_equal(sd, sq) and np.array_equal(fd, fq) and np.array_equal(Vd, Vq)
    s = np.linalg.svd(orc.bidiag_matrix(a, b), compute_uv=False)
    assert np.max(np.abs(sd - s) / s) < 1e-13
    assert np.max(np.abs(Vd @ Vd.T - np.eye(6))) < 1e-13


def test_param_choice(mq, orc, proj_case):
    p, g, s, ft, V = proj_case
    say("param_choice gcv")
    r = mq.mqh_param_choice(s, ft, mq.MQH_METHOD_HKT, mq.MQH_RULE_GCV, want_curve=True)
    lam, gv, edge, grid, vals = orc.choose_lambda_gcv(s, ft, 200)
    assert bool(r["flags"] & mq.MQH_INFO_GCV_AT_EDGE) == edge
    np.testing.assert_allclose(r["curve"], vals, rtol=1e-11)
    # the GCV minimiser is fixed only to ~sqrt(eps) by rounding (flat minimum)
    assert r["lambda_"] == pytest.approx(lam, rel=1e-6)
    assert r["crit"] == pytest.approx(gv, rel=1e-10)
    say("param_choice lcurve")
    r = mq.mqh_param_choice(s, ft, mq.MQH_METHOD_HKT, mq.MQH_RULE_LCURVE, want_curve=True)
    lam, kap, edge, grid, kv = orc.choose_lambda_lcurve(s, ft, 200)
    np.testing.assert_allclose(r["curve"], kv, rtol=1e-8, atol=1e-10 * np.max(np.abs(kv)))
    assert r["lambda_"] == pytest.approx(lam, rel=1e-12)
    say("param_choice tsvd")
    r = mq.mqh_param_choice(s, ft, mq.MQH_METHOD_INE_TSVD, mq.MQH_RULE_GCV)
    assert r["k"] == orc.choose_rank(s, ft)
    r = mq.mqh_param_choice(s, ft, mq.MQH_METHOD_INE_TSVD, mq.MQH_RULE_FIXED, k_trunc=9)
    assert r["k"] == 9


def test_param_choice_gcv_closed_form(mq, orc):
    s, ft, V = orc.proj_svd(np.array([3.0]), np.array([2.0, 1.0]))
    say("param_choice l=1")
    r = mq.mqh_param_choice(s, ft, mq.MQH_METHOD_HKT, mq.MQH_RULE_GCV)
    assert r["lambda_"] == pytest.approx(math.sqrt(10.0 / 8.0), rel=1e-7)


def test_param_choice_weighted_gcv(mq, orc, proj_case):
    p, g, s, ft, V = proj_case
    for w in (0.5, 0.8, 1.0):
        say("param_choice wgcv", w)
        r = mq.mqh_param_choice(s, ft, mq.MQH_METHOD_HKT, mq.MQH_RULE_WGCV, want_curve=True, gcv_weight=w)
        lam, gv, edge, grid, vals = orc.choose_lambda_gcv(s, ft, 200, omega=w)
        np.testing.assert_allclose(r["curve"], vals, rtol=1e-11)
        assert bool(r["flags"] & mq.MQH_INFO_GCV_AT_EDGE) == edge
        assert r["lambda_"] == pytest.approx(lam, rel=1e-6)
        r = mq.mqh_param_choice(s, ft, mq.MQH_METHOD_INE_TSVD, mq.MQH_RULE_WGCV, gcv_weight=w)
        assert r["k"] == orc.choose_rank(s, ft, w)
    s1, f1, _ = orc.proj_svd(np.array([2.0]), np.array([1.3, 0.7]))
    r = mq.mqh_param_choice(s1, f1, mq.MQH_METHOD_HKT, mq.MQH_RULE_WGCV, gcv_weight=0.5)
    lam, _, _, _, _ = orc.choose_lambda_gcv(s1, f1, 200, omega=0.5)
    assert r["lambda_"] == pytest.approx(lam, rel=1e-6)


def _cond_bound(alpha, beta, orc, k):
    sk = np.linalg.svd(orc.bidiag_matrix(alpha[:k], beta[: k + 1]), compute_uv=False)
    return 64 * k * EPS * sk[0] / sk[-1]


@pytest.mark.parametrize("rule", ["gcv", "lcurve", "fixed"])
def test_lsqr_path_and_choice(mq, orc, proj_case, rule):
    p, g, s, ft, V = proj_case
    rr = {"gcv": mq.MQH_RULE_GCV, "lcurve": mq.MQH_RULE_LCURVE, "fixed": mq.MQH_RULE_FIXED}[rule]
    say("lsqr", rule, "l =", g.ell)
    r = mq.mqh_lsqr(g.alpha, g.beta, p.n, rule=rr, k_trunc=17)
    rho, eta, Y = orc.lsqr_path(g.alpha, g.beta)
    assert np.all(np.abs(r["rho"] - rho) <= 1e-13 * g.beta[0])
    for k in range(1, g.ell + 1):
        tol = _cond_bound(g.alpha, g.beta, orc, k)
        assert abs(r["eta"][k - 1] - eta[k - 1]) <= tol * eta[k - 1], k
    if rule == "gcv":
        ko = orc.choose_k_lsqr_gcv(rho, p.n)
    elif rule == "lcurve":
        ko, _, edge, _ = orc.lcurve_discrete_corner(rho, eta)
        assert bool(r["flags"] & mq.MQH_INFO_LCURVE_AT_EDGE) == edge
    else:
        ko = 17
    assert r["k"] == ko
    yo = Y[ko - 1]
    assert np.linalg.norm(r["y"] - yo) <= _cond_bound(g.alpha, g.beta, orc, ko) * np.linalg.norm(yo)
    assert np.all(r["y"][ko:] == 0.0)


def test_lsqr_small_and_degenerate(mq, orc):
    for ell in (1, 2, 3):
        rng = np.random.default_rng(40 + ell)
        a = rng.random(ell) + 0.3
        b = np.concatenate([[1.1], rng.random(ell) + 0.3])
        say("lsqr small", ell)
        for rr in (mq.MQH_RULE_GCV, mq.MQH_RULE_LCURVE):
            r = mq.mqh_lsqr(a, b, 50, rule=rr)
            rho, eta, Y = orc.lsqr_path(a, b)
            ko = orc.choose_k_lsqr_gcv(rho, 50) if rr == mq.MQH_RULE_GCV else orc.lcurve_discrete_corner(rho, eta)[0]
            assert r["k"] == ko
            np.testing.assert_allclose(r["y"], Y[ko - 1], rtol=1e-12, atol=1e-14)
    # n = ell: the Krylov GCV stops before the full space
    a, b = np.array([1.0, 0.5]), np.array([2.0, 0.3, 0.2])
    r = mq.mqh_lsqr(a, b, 2, rule=mq.MQH_RULE_GCV)
    assert r["k"] == 1


def test_proj_solution_and_lift(mq, orc, proj_case):
    p, g, s, ft, V = proj_case
    say("proj_solution")
    Vt = np.ascontiguousarray(V.T)  # row i = v~_i, the layout of the ABI (column-major V)
    y = mq.mqh_proj_solution(s, ft, Vt, mq.MQH_METHOD_HKT, lam=s[10])
    yo = orc.y_tikhonov(s, ft, V, s[10])
    assert np.linalg.norm(y - yo) <= 1e-13 * np.linalg.norm(yo)
    y = mq.mqh_proj_solution(s, ft, Vt, mq.MQH_METHOD_INE_TSVD, k=12)
    yo = orc.y_tsvd(s, ft, V, 12)
    assert np.linalg.norm(y - yo) <= 1e-13 * np.linalg.norm(yo)
    say("lift")
    Zr = np.ascontiguousarray(g.Z.T)
    c = mq.mqh_lift(Zr, yo)
    co = orc.lift(g.Z, yo)
    assert np.all(np.abs(c - co) <= 1e-13 * (np.abs(g.Z) @ np.abs(yo)))


def test_eval(mq, orc):
    p = I.sphere_scaled(700, 300, kappa=5.0, eps=2.5, ell=10)
    coef = I.random_vector(p.n, 3)
    with _problem(mq, p, "matfree_fp64") as pr:
        say("eval")
        u = pr.eval(coef, p.x_eval)
    uo = orc.eval_u(p.nodes, p.eps, coef, p.x_eval)
    B = orc.interp_matrix(p.x_eval, p.nodes, p.eps)
    assert np.all(np.abs(u - uo) <= 1e-13 * (B @ np.abs(coef)))


# ---------------------------------------------------------------------------
# whole solves
# ---------------------------------------------------------------------------

def _solve_both(mq, orc, p, mode, **kw):
    r = orc.solve(p.nodes, p.n_int, p.kappa, p.eps, p.rhs, p.ell, stored=False, **kw)
    with _problem(mq, p, mode) as pr:
        say("solve", p.name, mode, kw)
        out = pr.solve(p.f_int, p.g_bnd, p.ell, **kw)
        u = pr.eval(out.coef, p.x_eval)
    uo = orc.eval_u(p.nodes, p.eps, r.coef, p.x_eval)
    return r, out, u, uo


SOLVE_CASES = [
    ("cube_n1800", I.cube_small),
    ("cube_interior_lambda", lambda: I.cube_scaled(400, 240, kappa=3.0, eps=0.7, ell=80)),
]


@pytest.mark.parametrize("name,make", SOLVE_CASES)
@pytest.mark.parametrize("mode", ["stored_fp64", "matfree_fp64"])
def test_solve_hkt(mq, orc, name, make, mode):
    p = make()
    r, out, u, uo = _solve_both(mq, orc, p, mode)
    assert out.ell_done == r.ell
    assert np.max(np.abs(out.sv[:10] - r.s[:10]) / r.s[:10]) < 1e-12
    assert out.lam == pytest.approx(r.lam, rel=1e-6)
    assert bool(out.flags & mq.MQH_INFO_GCV_AT_EDGE) == bool(r.flags & orc.FLAG_GCV_AT_EDGE)
    # at the oracle's lambda the solutions agree to the required 1e-8 bar
    r2, out2, u2, uo2 = _solve_both(mq, orc, p, mode, rule=mq.MQH_RULE_FIXED, lambda_fixed=r.lam)
    assert np.linalg.norm(u2 - uo2) <= 1e-8 * np.linalg.norm(uo2)
    assert np.linalg.norm(out2.coef - r2.coef) <= 1e-6 * np.linalg.norm(r2.coef)
    assert out2.resid_norm == pytest.approx(r2.resid_norm, rel=1e-9)
    assert out2.sol_norm == pytest.approx(r2.sol_norm, rel=1e-8)


@pytest.mark.parametrize("name,make", SOLVE_CASES)
def test_solve_ine_tsvd(mq, orc, name, make):
    p = make()
    r, out, u, uo = _solve_both(mq, orc, p, "matfree_fp64", method=mq.MQH_METHOD_INE_TSVD)
    assert out.k == r.k
    assert np.linalg.norm(u - uo) <= 1e-8 * np.linalg.norm(uo)


def test_solve_lcurve(mq, orc):
    p = I.cube_scaled(400, 240, kappa=3.0, eps=0.7, ell=80)
    r, out, u, uo = _solve_both(mq, orc, p, "matfree_fp64", rule=mq.MQH_RULE_LCURVE)
    assert out.lam == pytest.approx(r.lam, rel=1e-10)
    assert np.linalg.norm(u - uo) <= 1e-8 * np.linalg.norm(uo)


def test_solve_fp32_entries(mq, orc):
    # FP32 entries perturb A by dA with |dA| <~ 1e-6 |A| entrywise; a Tikhonov
    # solution at lambda moves by about (s_1/lambda) |dA|/|A|, so at
    # lambda = 1e-3 s_1 the FP32 path stays within ~1e-3 of the FP64 oracle.
    p = I.cube_scaled(400, 240, kappa=3.0, eps=0.7, ell=80)
    s1 = orc.solve(p.nodes, p.n_int, p.kappa, p.eps, p.rhs, p.ell, stored=False).s[0]
    r, out, u, uo = _solve_both(mq, orc, p, "matfree_fp32", rule=mq.MQH_RULE_FIXED, lambda_fixed=1e-3 * s1)
    assert np.linalg.norm(u - uo) <= 1e-3 * np.linalg.norm(uo)
    # at the GCV choice the error against the exact solution matches the FP64 path's
    r, out, u, uo = _solve_both(mq, orc, p, "matfree_fp32")
    e32, e64 = orc.rel_l2(u, p.u_eval), orc.rel_l2(uo, p.u_eval)
    assert abs(e32 - e64) <= 0.05 * e64


@pytest.mark.parametrize("rule", ["gcv", "lcurve", "fixed"])
def test_solve_lsqr(mq, orc, rule):
    p = I.cube_scaled(400, 240, kappa=3.0, eps=0.7, ell=80)
    rr = {"gcv": mq.MQH_RULE_GCV, "lcurve": mq.MQH_RULE_LCURVE, "fixed": mq.MQH_RULE_FIXED}[rule]
    r, out, u, uo = _solve_both(mq, orc, p, "matfree_fp64", method=mq.MQH_METHOD_LSQR, rule=rr, k_trunc=25)
    assert out.k == r.k
    # rho_k depends on every Golub-Kahan scalar up to k, which the two paths round differently; the
    # HKT solve tests use the same bounds (1e-9 residual, 1e-8 solution)
    assert out.resid_norm == pytest.approx(r.resid_norm, rel=1e-9)
    tol = max(1e-8, _cond_bound(r.alpha, r.beta, orc, r.k))
    assert out.sol_norm == pytest.approx(r.sol_norm, rel=tol)
    assert np.linalg.norm(u - uo) <= tol * np.linalg.norm(uo)


def test_solve_hkt_weighted_gcv(mq, orc):
    p = I.cube_scaled(400, 240, kappa=3.0, eps=0.7, ell=80)
    kw = dict(rule=mq.MQH_RULE_WGCV, gcv_weight=0.6)
    r, out, u, uo = _solve_both(mq, orc, p, "stored_fp64", **kw)
    assert out.lam == pytest.approx(r.lam, rel=1e-6)
    # at the oracle's lambda the solutions agree to the required bar
    r2, out2, u2, uo2 = _solve_both(mq, orc, p, "stored_fp64", rule=mq.MQH_RULE_FIXED, lambda_fixed=r.lam)
    assert np.linalg.norm(u2 - uo2) <= 1e-8 * np.linalg.norm(uo2)


def test_solve_deterministic(mq):
    p = I.cube_scaled(300, 200, kappa=4.0, eps=1.0, ell=30)
    with _problem(mq, p, "matfree_fp32") as pr:
        say("determinism")
        a = pr.solve(p.f_int, p.g_bnd, p.ell)
        b = pr.solve(p.f_int, p.g_bnd, p.ell)
    assert np.array_equal(a.coef, b.coef) and a.lam == b.lam


@pytest.mark.parametrize("n_int,n_bnd", [(1, 0), (0, 1), (0, 37), (37, 0), (2, 1), (63, 2), (64, 1), (1000, 7)])
def test_edge_sizes(mq, orc, n_int, n_bnd):
    X = I.random_nodes_cube(n_int + n_bnd, 900 + n_int)
    f = I.random_vector(n_int + n_bnd, 901)
    ell = min(5, n_int + n_bnd)
    for mode in ("matfree_fp32",):
        say("edge sizes", n_int, n_bnd, mode)
        with mq.Problem(X[:n_int] if n_int else None, X[n_int:] if n_bnd else None, 2.0, 3.0, mode) as pr:
            ys = [pr.apply(f, trans=t) for t in (False, True)]
        A = orc.assemble(X, n_int, 2.0, 3.0)
        for t, y in zip((False, True), ys):
            ref = orc.apply(None, X, n_int, 2.0, 3.0, f, trans=t)
            scale = (A.T if t else A) @ np.abs(f)  # all entries are positive
            assert np.all(np.abs(y - ref) <= 4e-6 * scale)
    for mode in ("stored_fp64", "matfree_fp64"):
        say("edge sizes", n_int, n_bnd, mode)
        with mq.Problem(X[:n_int] if n_int else None, X[n_int:] if n_bnd else None, 2.0, 3.0, mode) as pr:
            y = pr.apply(f, trans=True)
            out = pr.solve(f[:n_int] if n_int else None, f[n_int:] if n_bnd else None, ell,
                           rule=mq.MQH_RULE_FIXED, lambda_fixed=1e-2)
        ref = orc.apply(None, X, n_int, 2.0, 3.0, f, trans=True)
        A = orc.assemble(X, n_int, 2.0, 3.0)
        assert np.all(np.abs(y - ref) <= 1e-13 * (np.abs(A.T) @ np.abs(f)))
        r = orc.solve(X, n_int, 2.0, 3.0, f, ell, rule=orc.RULE_FIXED, lambda_fixed=1e-2)
        assert out.ell_done == r.ell
        assert np.linalg.norm(out.coef - r.coef) <= 1e-8 * max(np.linalg.norm(r.coef), 1e-300)


# ---------------------------------------------------------------------------
# full size (unit ball, n = 100000), in the launch configuration the
# benchmark times: sampled outputs against the oracle one by one, and the
# Golub-Kahan relations on sampled rows
# ---------------------------------------------------------------------------

@pytest.fixture(scope="module")
def sphere_full():
    return I.sphere_large()


@pytest.mark.parametrize("mode", ["matfree_fp32", "matfree_fp64", "stored_fp64"])
def test_products_full_size_sampled(mq, orc, sphere_full, mode):
    p = sphere_full
    x = I.random_vector(p.n, 21)
    idx = np.unique(np.concatenate([np.arange(0, p.n, 997), [p.n_int - 1, p.n_int, p.n - 1]])).astype(np.int64)
    tol = 4e-6 if mode == "matfree_fp32" else 1e-13
    with _problem(mq, p, mode) as pr:
        for trans in (False, True):
            say("full-size apply", mode, "trans", trans)
            y = pr.apply(x, trans=trans)
            ref = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, x, idx, trans=trans)
            scale = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, np.abs(x), idx, trans=trans)
            err = np.abs(y[idx] - ref) / scale
            assert np.all(err <= tol), float(err.max())


def test_gkb_relations_full_size_fp32(mq, orc, sphere_full):
    # A Z = W C and A^T W_l = Z_l C_l^T hold for the operator the GPU applies;
    # against the FP64 oracle's A they hold to the FP32 entry error.
    p = sphere_full
    with _problem(mq, p, "matfree_fp32") as pr:
        say("full-size gkb fp32, ell", p.ell)
        r = pr.gkb(p.rhs, p.ell)
    assert r["ell_done"] == p.ell
    Wc, Zc, a, b = r["W"], r["Z"], r["alpha"], r["beta"]  # rows are basis vectors
    l = p.ell
    WtW = Wc @ Wc.T
    ZtZ = Zc @ Zc.T
    assert np.max(np.abs(WtW - np.eye(l + 1))) < 1e-12
    assert np.max(np.abs(ZtZ - np.eye(l))) < 1e-12
    assert abs(Wc[0] @ p.rhs - b[0]) <= 1e-12 * b[0]
    idx = np.arange(5, p.n, 1499).astype(np.int64)
    for j in (0, l // 2, l - 1):
        say("relation column", j)
        azj = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, Zc[j], idx)
        sc = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, np.abs(Zc[j]), idx)
        wc = a[j] * Wc[j, idx] + b[j + 1] * Wc[j + 1, idx]
        assert np.all(np.abs(azj - wc) <= 1e-5 * sc), float(np.max(np.abs(azj - wc) / sc))
        atw = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, Wc[j], idx, trans=True)
        sct = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, np.abs(Wc[j]), idx, trans=True)
        zc = a[j] * Zc[j, idx] + (b[j] * Zc[j - 1, idx] if j > 0 else 0.0)
        assert np.all(np.abs(atw - zc) <= 1e-5 * sct), float(np.max(np.abs(atw - zc) / sct))


def test_hkt_full_size_stored_fp64(mq, orc, sphere_full):
    # The benchmark's own solve (stored FP64 A, n = 100000, ell = 300,
    # HKT + GCV): the Golub-Kahan relations against the oracle's A on sampled
    # rows, then every projected step against the oracle on the GPU's alpha,
    # beta, and the coefficients against the oracle's projected solution
    # lifted with the GPU's Z.
    p = sphere_full
    l = p.ell
    with _problem(mq, p, "stored_fp64") as pr:
        say("full-size gkb stored fp64, ell", l)
        r = pr.gkb(p.rhs, l)
        say("full-size solve stored fp64, ell", l)
        out = pr.solve(p.f_int, p.g_bnd, l)
    assert r["ell_done"] == l and out.ell_done == l
    Wc, Zc, a, b = r["W"], r["Z"], r["alpha"], r["beta"]
    assert np.max(np.abs(Wc @ Wc.T - np.eye(l + 1))) < 1e-12
    assert np.max(np.abs(Zc @ Zc.T - np.eye(l))) < 1e-12
    idx = np.arange(7, p.n, 1511).astype(np.int64)
    worst = 0.0
    for j in (0, l // 2, l - 1):
        azj = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, Zc[j], idx)
        sc = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, np.abs(Zc[j]), idx)
        wc = a[j] * Wc[j, idx] + b[j + 1] * Wc[j + 1, idx]
        atw = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, Wc[j], idx, trans=True)
        sct = orc.apply_sampled(p.nodes, p.n_int, p.kappa, p.eps, np.abs(Wc[j]), idx, trans=True)
        zc = a[j] * Zc[j, idx] + (b[j] * Zc[j - 1, idx] if j > 0 else 0.0)
        worst = max(worst, float(np.max(np.abs(azj - wc) / sc)), float(np.max(np.abs(atw - zc) / sct)))
    say("relations, worst ratio", worst)
    assert worst <= 1e-12  # the FP64 product bound (1e-13) plus the reorthogonalisation rounding
    # the solve repeats the same Golub-Kahan run
    np.testing.assert_allclose(out.alpha, a, rtol=1e-12)
    np.testing.assert_allclose(out.beta, b, rtol=1e-12)
    say("projected steps against the oracle")
    s, ft, V = orc.proj_svd(a, b)
    sv, ftg, _ = mq.mqh_proj_svd(a, b)
    assert np.max(np.abs(sv[:10] - s[:10]) / s[:10]) < 1e-12
    assert np.max(np.abs(sv - s)) < 64 * l * EPS * s[0]
    assert np.max(np.abs(out.sv[:10] - s[:10]) / s[:10]) < 1e-12
    lam, gv, edge, grid, vals = orc.choose_lambda_gcv(s, ft, 200)
    assert out.lam == pytest.approx(lam, rel=1e-6)
    assert bool(out.flags & mq.MQH_INFO_GCV_AT_EDGE) == edge
    y = orc.y_tikhonov(s, ft, V, out.lam)
    coef = Zc.T @ y
    assert np.linalg.norm(out.coef - coef) <= 1e-8 * np.linalg.norm(coef)


def test_duplicate_nodes_finite(mq):
    X = I.random_nodes_cube(60, 44)
    X[7] = X[3]
    say("duplicate nodes")
    with mq.Problem(X[:30], X[30:], 3.0, 4.0, "matfree_fp64") as pr:
        out = pr.solve(np.ones(30), np.ones(30), 20)
    assert np.all(np.isfinite(out.coef))


def test_invalid_inputs(mq):
    X = I.random_nodes_cube(40, 3)
    with mq.Problem(X[:20], X[20:], 2.0, 3.0, "matfree_fp64") as pr:
        say("invalid inputs")
        bad = np.ones(20)
        bad[3] = math.nan
        with pytest.raises(mq.MQHError):
            pr.solve(bad, np.ones(20), 5)
        with pytest.raises(mq.MQHError):
            pr.solve(np.ones(20), np.ones(20), 41)  # ell > n
        with pytest.raises(mq.MQHError):
            pr.solve(np.ones(20), np.ones(20), 5, method=mq.MQH_METHOD_INE_TSVD, rule=mq.MQH_RULE_FIXED, k_trunc=0)
