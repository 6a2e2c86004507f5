"""Pivots of the Cholesky's diagonal blocks that depend on each other or lie far
apart: neighbouring unknowns that nearly coincide, diagonals that differ by
2^2000, and unknowns pinned to zero by an infinite diagonal entry.

Bounds (u = 2^-53).  L L^T: the entry (i, j) is a sum of at most n products with
n roundings, the reciprocal root of the pivot and its products add 3 u in each
factor, and sum_k |L_ik L_jk| <= sqrt(S_ii S_jj) (Cauchy-Schwarz): (n + 8) u of the
largest diagonal entry, for blocks of at most 64 rows (no inverse enters).
Scaled and pinned matrices: the bounds of the other test of the blocks (condition
below 10 up to a scaling by powers of two that is carried through exactly).
"""
import numpy as np
import pytest
import torch  # noqa: F401

from test_gpu_diag_block import factor, spd, strip

pytestmark = pytest.mark.gpu


def near_pairs(n, first, delta):
    """SPD; unknowns (first, first + 1), (first + 2, first + 3), .. differ by delta."""
    F = np.linalg.cholesky(spd(n, n + 7)[0]).astype(np.longdouble)
    for k in range(first, n - 1, 2):
        F[k + 1] = F[k] + np.longdouble(delta) * F[k + 1]
    return (F @ F.T).astype(np.float64)


@pytest.mark.parametrize("delta", [1e-1, 1e-2, 1e-3, 1e-4, 1e-5])
@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("n", [4, 16, 17, 33, 48, 64])
def test_nearly_dependent_pairs(n, first, delta):
    S = near_pairs(n, first, delta)
    L, _ = factor(strip(n), S, np.ones(n))
    L = L.astype(np.longdouble)
    assert float(np.abs(L @ L.T - S).max()) <= (n + 8) * 2.0 ** -53 * S.max()


@pytest.mark.parametrize("n", [2, 3, 16, 63, 64, 65, 129])
@pytest.mark.parametrize("order", ["down", "up", "random"])
def test_diagonals_far_apart(n, order):
    S, rhs = spd(n, n)
    e = np.where((np.arange(n) & 1) == (order == "up"), 500, -500)
    if order == "random":
        e = np.round(np.random.default_rng(n).uniform(-500, 500, n)).astype(int)
    d = np.ldexp(1.0, e)
    L, u = factor(strip(n), S * d[:, None] * d[None, :], rhs * d)
    assert np.abs(L / d[:, None] - np.linalg.cholesky(S)).max() <= 1e-12
    assert np.abs(u * d - np.linalg.solve(S, rhs)).max() <= 1e-11


@pytest.mark.parametrize("n,at", [(2, 0), (2, 1), (64, 5), (64, 62), (64, 63), (129, 0), (129, 70), (129, 128)])
def test_infinite_diagonal_pins_its_unknown(n, at):
    S, rhs = spd(n, n)
    S[at, at] = np.inf
    keep = np.arange(n) != at
    want = np.zeros(n)
    want[keep] = np.linalg.solve(S[np.ix_(keep, keep)], rhs[keep])
    L, u = factor(strip(n), S, rhs)
    assert u[at] == 0.0 and np.abs(u - want).max() <= 1e-11
    L[at, at] = 0.0
    assert np.isfinite(L).all()
