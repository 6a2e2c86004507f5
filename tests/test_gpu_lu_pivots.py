"""The LU factorization of blocks whose neighbouring unknowns nearly coincide (the
symmetric part stays definite, the pivots get small): L U against the matrix.

Bound (u = 2^-53): an entry is a sum of at most n products with n roundings, the
pivot's reciprocal and the products with it add 3 u: (n + 8) u of the largest entry
of |L| |U|, for matrices of one 64 x 64 block (no inverse enters).  Scaled by powers
of two on both sides the factor is the same but for the scaling.
"""
import numpy as np
import pytest
import torch

from test_gpu_diag_block import spd
from test_gpu_lu_block import mesh

pytestmark = pytest.mark.gpu


def near_pairs(n, first, delta):
    """G C G^T with C = I + a skew part; rows (first, first + 1), .. of G differ by delta."""
    G = np.linalg.cholesky(spd(n, n + 7)[0]).astype(np.longdouble)
    for k in range(first, n - 1, 2):
        G[k + 1] = G[k] + np.longdouble(delta) * G[k + 1]
    W = np.random.default_rng(n).normal(size=(n, n)) / np.sqrt(n)
    return (G @ (np.eye(n) + 0.5 * (W - W.T)) @ G.T).astype(np.float64)


def factor(k, A):
    X = torch.tensor(A, device="cuda")
    mesh(k).lu_factor(X)
    torch.cuda.synchronize()
    return X.cpu().numpy()


@pytest.mark.parametrize("delta", [1e-1, 1e-2, 1e-3, 1e-4, 1e-5])
@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("k", [3, 4, 5])
def test_nearly_dependent_pairs(k, first, delta):
    n = (k - 1) ** 3
    A = near_pairs(n, first, delta)
    X = factor(k, A).astype(np.longdouble)
    L, U = np.tril(X, -1) + np.eye(n), np.triu(X)
    assert float(np.abs(L @ U - A).max()) <= (n + 8) * 2.0 ** -53 * float((np.abs(L) @ np.abs(U)).max())


@pytest.mark.parametrize("e", [-480, 480])
@pytest.mark.parametrize("k", [3, 4, 5])
def test_scaled_by_powers_of_two(k, e):
    n = (k - 1) ** 3
    A = near_pairs(n, 0, 0.3)
    rng = np.random.default_rng(n)
    r, c = (np.ldexp(1.0, rng.integers(-20, 20, n) + e) for _ in range(2))
    X, Y = factor(k, A), factor(k, A * r[:, None] * c[None, :])
    low = np.tril(np.ones((n, n), dtype=bool), -1)
    assert np.array_equal(np.where(low, Y / r[:, None] * r[None, :], Y / r[:, None] / c[None, :]), X)
