"""The conjugate gradients' state on the device: iterates, counts and ends of
the loop around the few iterations that are queued at a time, against the same
recurrence in NumPy, on matrices handed over in CSR form.

Bound: the matrices are diagonally dominant (condition below 10), so after ten
iterations rounding has grown by at most a few hundred ulps: 1e-12 relative.
The tolerances of the counted runs lie half way between two residuals of the
recurrence, which differ by a factor of 2 or more.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_1811_03339_amd as F
from fpde_inputs import kuhn_cube

pytestmark = pytest.mark.gpu

ENOTSPD, ENOCONV = -7, -8
_M = {}


def problem(cells):
    """Mesh with (cells - 1)^3 unknowns; a symmetric five-band matrix of that size."""
    if cells not in _M:
        m = kuhn_cube(cells)
        gm = F.Mesh(m.xyz, m.tet)
        n = gm.n_dof
        rng = np.random.default_rng(n)
        rows, cols, vals = [np.arange(n)], [np.arange(n)], [rng.uniform(3.0, 6.0, n)]
        for off in (1, 37):
            if off >= n:
                continue
            v = rng.uniform(-0.5, 0.5, n - off)
            i = np.arange(n - off)
            rows += [i, i + off]
            cols += [i + off, i]
            vals += [v, v]
        r, c, v = (np.concatenate(a) for a in (rows, cols, vals))
        o = np.lexsort((c, r))
        r, c, v = r[o], c[o], v[o]
        rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int64)
        _M[cells] = gm, r, c.astype(np.int32), v, rp, rng.normal(size=n)
    return _M[cells]


def reference(r, c, v, b, iters):
    """Iterates and relative residuals of CG with the Jacobi preconditioner."""
    n = b.size
    mul = lambda x: np.bincount(r, v * x[c], minlength=n)  # noqa: E731
    d = v[r == c]
    u, res, z = np.zeros(n), b.copy(), b / d
    p, rz, out = z.copy(), b @ z, []
    for _ in range(iters):
        q = mul(p)
        al = rz / (p @ q)
        u, res = u + al * p, res - al * q
        z = res / d
        be, rz = (res @ z) / rz, res @ z
        p = z + be * p
        out.append((u, np.linalg.norm(res) / np.linalg.norm(b)))
    return out


def solve(gm, rp, c, v, b, tol, max_iter=0):
    dev = [torch.tensor(a, device="cuda") for a in (rp, c, v, b)]
    u = torch.full((b.size,), float("nan"), dtype=torch.float64, device="cuda")
    info = F.fpde_solve_info()
    st = F._lib().fpde_cg_solve(gm._h, ctypes.byref(F.params(1.5)), *(ctypes.c_void_p(t.data_ptr()) for t in dev),
                                ctypes.c_void_p(u.data_ptr()), float(tol), int(max_iter), ctypes.byref(info),
                                F._stream(None))
    torch.cuda.synchronize()
    return st, info, u.cpu().numpy()


@pytest.mark.parametrize("cells", [3, 8, 42])
def test_iterates_and_counts(cells):
    gm, r, c, v, rp, b = problem(cells)
    k_max = 4 if cells == 3 else 9  # 8 unknowns: the residual is rounding after 8
    ref = reference(r, c, v, b, k_max + 1)
    for k in range(1, k_max + 1):
        want, res = ref[k - 1]
        st, info, u = solve(gm, rp, c, v, b, 1e-300, k)
        assert st == ENOCONV and info.ir_iters == k
        assert np.abs(u - want).max() <= 1e-12 * np.abs(want).max()
        assert abs(info.final_rel_residual - res) <= 1e-12
        assert res <= 0.5 * (ref[k - 2][1] if k > 1 else 1.0)
        tol = np.sqrt(res * (ref[k - 2][1] if k > 1 else 1.0))
        st, info, u2 = solve(gm, rp, c, v, b, tol)
        assert st == F.FPDE_OK and info.ir_iters == k
        assert np.array_equal(u, u2)


def test_ends_without_a_solution():
    gm, r, c, v, rp, b = problem(8)
    for rhs, tol in ((0.0 * b, 1e-10), (b, 1.0), (b, 2.0)):
        st, info, u = solve(gm, rp, c, v, rhs, tol)
        assert st == F.FPDE_OK and info.ir_iters == 0 and not u.any()
    bad = v.copy()
    bad[np.flatnonzero(r == c)[5]] = -1.0
    assert solve(gm, rp, c, bad, b, 1e-10)[0] == ENOTSPD
    bad = np.where(r == c, v, 40.0 * v)  # positive diagonal, indefinite
    assert solve(gm, rp, c, bad, b, 1e-10)[0] == ENOTSPD
    nan = b.copy()
    nan[3] = np.nan
    assert solve(gm, rp, c, v, nan, 1e-10)[1].ir_iters == 0
    st, info, u = solve(gm, rp, c, v, b, 1e-10)  # the state starts afresh
    assert st == F.FPDE_OK and info.final_rel_residual <= 2e-10
