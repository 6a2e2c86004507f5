"""LU without row exchanges at the sizes where its tiles and groups end, on a
three-dimensional handle of k^3 unknowns padded by the leading dimension:
inside one diagonal block, one block, inside a group of eight 64-column
panels, exactly one group (512), one group and a ragged trailing square (729,
1000), several groups (1728, 2744); and a pivot that is zero or not finite in
every 16-column panel of a block.

Bound: the matrices are diagonally dominant by columns with multipliers below
1 / 2, so no entry grows by more than 2 and the factor's rounding error stays
below n eps times a small constant: 1e-12 covers 2 744 eps twice over.
"""
import numpy as np
import pytest
import torch

import paper_1811_03339_amd as F
from fpde_inputs import kuhn_cube

pytestmark = pytest.mark.gpu
_MESHES = {}


def mesh(k):
    if k not in _MESHES:
        m = kuhn_cube(k)
        _MESHES[k] = F.Mesh(m.xyz, m.tet)
    return _MESHES[k]


def dominant(n, seed):
    rng = np.random.default_rng(seed)
    A = rng.uniform(-1, 1, size=(n, n))
    return A + np.diag(2.0 * np.abs(A).sum(0) + 1.0)


def lu_reference(A):
    """Elimination without row exchanges, 32 columns at a time."""
    A = A.copy()
    n = len(A)
    for k in range(0, n, 32):
        e = min(k + 32, n)
        for j in range(k, e):
            A[j + 1:, j] /= A[j, j]
            A[j + 1:, j + 1:e] -= np.outer(A[j + 1:, j], A[j, j + 1:e])
        if e < n:
            unit = np.tril(A[k:e, k:e], -1) + np.eye(e - k)
            A[k:e, e:] = np.linalg.solve(unit, A[k:e, e:])
            A[e:, e:] -= A[e:, k:e] @ A[k:e, e:]
    return A


@pytest.mark.parametrize("k", [2, 3, 4, 5, 6, 7, 9, 10, 11, 13, 15])
@pytest.mark.parametrize("pad", [0, 5])
def test_factor_and_solve(k, pad):
    gm = mesh(k)
    n = gm.n_dof
    print(f"[case] lu n={n} pad={pad}", flush=True)
    S = dominant(n, n)
    buf = torch.full((n, n + pad), 7.0, dtype=torch.float64, device="cuda")
    A = buf[:, :n]
    A.copy_(torch.tensor(S))
    assert gm.lu_factor(A) == -1
    torch.cuda.synchronize()
    want = lu_reference(S)
    assert np.abs(A.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    assert pad == 0 or bool((buf[:, n:] == 7.0).all())
    rhs = np.random.default_rng(1).normal(size=n)
    u = torch.empty(n, dtype=torch.float64, device="cuda")
    gm.lu_solve(A, torch.tensor(rhs, device="cuda"), u)
    torch.cuda.synchronize()
    ref = np.linalg.solve(S, rhs)
    assert np.abs(u.cpu().numpy() - ref).max() <= 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("at", [0, 15, 16, 33, 63, 64, 100, 124])
@pytest.mark.parametrize("bad", [0.0, float("inf"), float("nan")])
def test_bad_pivot_is_reported_with_its_block(at, bad):
    gm = mesh(6)  # 125 unknowns
    S = np.diag(np.linspace(1.0, 2.0, 125))
    S[at, at] = bad
    with pytest.raises(F.FpdeError) as e:
        gm.lu_factor(torch.tensor(S, device="cuda"))
    assert e.value.status == -12 and e.value.failed_pivot == 64 * (at // 64)
