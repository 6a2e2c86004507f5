"""The conjugate gradients' loop around the matrix-free product (its own pair of
kernels: one decides whether the loop has ended, the other reads that): counts,
iterates and ends of the few iterations that are queued at a time, against the
recurrence in NumPy on the oracle's matrix.

Bound: the products agree with the oracle's to 1e-11, and nine iterations at the
condition of these matrices (below 100) let that grow to 1e-8 at most.  A counted
run's tolerance lies half way between its residual and the smallest one before,
where the two differ by a factor of 1.2 or more.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1811_03339_amd as F
from fpde_inputs import kuhn_cube
from test_gpu_cg import problem, reference
from test_gpu_cg import solve as solve_csr
from test_gpu_tubes import bar

pytestmark = pytest.mark.gpu

ENOCONV = -8
KC = (1.0, 0.5, 2.0)


def solve(gm, p, b, tol, max_iter=0):
    dev = torch.tensor(b, device="cuda")
    u = torch.full((b.size,), float("nan"), dtype=torch.float64, device="cuda")
    info = F.fpde_solve_info()
    st = F._lib().fpde_cg_solve(gm._h, ctypes.byref(p), None, None, None, ctypes.c_void_p(dev.data_ptr()),
                                ctypes.c_void_p(u.data_ptr()), float(tol), int(max_iter), ctypes.byref(info),
                                F._stream(None))
    torch.cuda.synchronize()
    return st, info, u.cpu().numpy()


@pytest.mark.parametrize("mesh", ["cube5", "bar"])
def test_iterates_and_counts(mesh):
    if mesh == "cube5":
        m = kuhn_cube(5)
        xyz, tet = m.xyz, m.tet
    else:
        xyz, tet = bar(3, 4, 17)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    A = om.assemble(4, 1.5, KC)
    A = 0.5 * (A + A.T)
    assert np.linalg.cond(A / np.sqrt(np.outer(np.diag(A), np.diag(A)))) < 100
    n = gm.n_dof
    b = np.random.default_rng(n).normal(size=n)
    r, c = (a.ravel() for a in np.indices(A.shape))
    ref = reference(r, c, A.ravel(), b, 9)
    p = F.params(1.5, KC, quad_points=4)
    least, counted = 1.0, 0
    for k in range(1, 10):
        want, res = ref[k - 1]
        st, info, u = solve(gm, p, b, 1e-300, k)
        assert st == ENOCONV and info.ir_iters == k
        assert np.abs(u - want).max() <= 1e-8 * np.abs(want).max()
        assert abs(info.final_rel_residual - res) <= 1e-8
        if res < least / 1.2:
            st, info, u2 = solve(gm, p, b, np.sqrt(res * least))
            assert st == F.FPDE_OK and info.ir_iters == k
            assert np.array_equal(u, u2)
            counted += 1
        least = min(least, res)
    assert counted >= 5


def test_ends_without_a_solution():
    m = kuhn_cube(5)
    gm = F.Mesh(m.xyz, m.tet)
    b = np.random.default_rng(3).normal(size=gm.n_dof)
    p = F.params(1.5, KC, quad_points=4)
    for rhs, tol in ((0.0 * b, 1e-10), (b, 1.0), (b, 2.0)):
        st, info, u = solve(gm, p, rhs, tol)
        assert st == F.FPDE_OK and info.ir_iters == 0 and not u.any()
    st, info, u = solve(gm, p, b, 1e-10)  # the state starts afresh
    assert st == F.FPDE_OK and info.final_rel_residual <= 2e-10


@pytest.mark.parametrize("csr", [False, True])
def test_right_hand_side_that_is_not_a_number(csr):
    """The norm of the right-hand side compares as not positive, which counts as a
    right-hand side of zero: no iteration, status OK, u = 0, and a residual that is
    not a number."""
    if csr:
        gm, r, c, v, rp, b = problem(8)
    else:
        m = kuhn_cube(5)
        gm = F.Mesh(m.xyz, m.tet)
        b = np.ones(gm.n_dof)
    b = b.copy()
    b[3] = np.nan
    st, info, u = solve_csr(gm, rp, c, v, b, 1e-10) if csr else solve(gm, F.params(1.5, KC), b, 1e-10)
    assert st == F.FPDE_OK and info.ir_iters == 0 and not u.any() and np.isnan(info.final_rel_residual)
