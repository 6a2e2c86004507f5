"""The 64 x 64 diagonal blocks of the Cholesky factorization, through the
dense solve of a two-dimensional handle (a strip of 2 x (n + 1) squares has
exactly n unknowns): sizes around the 16-column panels and the block, rows
graded over 2^240, matrices near both ends of the exponent range, and a
pivot that is not positive at even and odd positions of every panel.

Bound: the matrices have condition numbers below 10 up to their power-of-two
scaling (which every step of the factorization carries through exactly), so
a backward error of n eps per entry leaves the factor within 10 n eps < 3e-13
of LAPACK's at n <= 129; 1e-12 leaves a factor three.
"""
import numpy as np
import pytest
import torch

import paper_1811_03339_amd as F

pytestmark = pytest.mark.gpu


def strip(n):
    """Handle with n unknowns."""
    xs, ys = np.linspace(0.0, 1.0, n + 2), np.array([0.0, 0.5, 1.0])
    xy = np.stack(np.meshgrid(xs, ys, indexing="ij"), -1).reshape(-1, 2)
    tri = []
    for i in range(n + 1):
        for j in range(2):
            a, b = 3 * i + j, 3 * (i + 1) + j
            tri += [(a, b, b + 1), (a, b + 1, a + 1)]
    m = F.Mesh2D(xy, np.array(tri, dtype=np.int32))
    assert m.n_dof == n
    return m


def spd(n, seed):
    rng = np.random.default_rng(seed)
    M = rng.normal(size=(n, n))
    return M @ M.T / n + np.eye(n), rng.normal(size=n)


def factor(m, S, rhs):
    A, b = torch.tensor(S, device="cuda"), torch.tensor(rhs, device="cuda")
    u = torch.empty_like(b)
    m.solve(A, b, u)
    torch.cuda.synchronize()
    return np.tril(A.cpu().numpy()), u.cpu().numpy()


@pytest.mark.parametrize("n", [1, 2, 3, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 80, 127, 129])
@pytest.mark.parametrize("scale", ["one", "graded", "small", "large"])
def test_factor_matches_lapack(n, scale):
    S, rhs = spd(n, n)
    ref = np.linalg.cholesky(S)
    e = {"one": np.zeros(n), "small": np.full(n, -480), "large": np.full(n, 480),
         "graded": np.round(np.random.default_rng(n + 1).uniform(-120, 120, n))}[scale]
    d = np.ldexp(1.0, e.astype(int))
    L, u = factor(strip(n), S * d[:, None] * d[None, :], rhs * d)
    assert np.abs(L / d[:, None] - ref).max() <= 1e-12
    assert np.abs(u * d - np.linalg.solve(S, rhs)).max() <= 1e-11


@pytest.mark.parametrize("at", [0, 1, 2, 14, 15, 16, 17, 31, 46, 47, 48, 63, 64, 77, 95])
@pytest.mark.parametrize("bad", [-1.0, 0.0, float("nan")])
def test_bad_pivot_is_reported_with_its_block(at, bad):
    m = strip(96)
    S = np.diag(np.linspace(1.0, 2.0, 96))
    S[at, at] = bad
    with pytest.raises(F.FpdeError) as e:
        factor(m, S, np.ones(96))
    assert e.value.status == -7
    # the handle is usable afterwards
    S, rhs = spd(96, 5)
    L, _ = factor(m, S, rhs)
    assert np.abs(L - np.linalg.cholesky(S)).max() <= 1e-12
