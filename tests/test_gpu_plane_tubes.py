"""The two-dimensional accumulation on both of its ways, on squares and strips of
cells whose tubes have from a few to several hundred nodes: the row gather (at
most 128 unknowns, and long chords of few rows), tube blocks as a square, as a
packed triangle and in bands of it; values over several steps of a half-ray.
Against the oracle's matrix, at the bar of the other two-dimensional tests
(1e-10, max-norm relative).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_03339_amd as F

pytestmark = pytest.mark.gpu


def grid(nx, ny):
    """nx x ny squares of edge 1/8 cut into two triangles each; interior vertices moved."""
    m = np.array([nx, ny]) + 1
    g = np.stack(np.meshgrid(*[np.arange(k) for k in m], indexing="ij"), -1).reshape(-1, 2)
    inner = ((g > 0) & (g < m - 1)).all(1)
    xy = 0.125 * (g + np.where(inner[:, None], np.random.default_rng(nx).uniform(-0.2, 0.2, g.shape), 0.0))
    a = (np.arange(nx)[:, None] * m[1] + np.arange(ny)).ravel()
    b = a + m[1]
    return xy, np.concatenate([np.stack([a, b, b + 1], 1), np.stack([a, b + 1, a + 1], 1)]).astype(np.int32)


def rel(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


# unknowns 1, 121, 144, 1 521, 447, 1 796, 1 299
SHAPES = [(2, 2), (12, 12), (13, 13), (40, 40), (150, 4)]


@pytest.mark.parametrize("shape,quad", [(s, q) for s in SHAPES for q in (3, 7)] + [((450, 5), 3), ((1300, 2), 3)])
def test_matrix_matches_oracle(shape, quad):
    xy, tri = grid(*shape)
    gm, om = F.Mesh2D(xy, tri), oracle.OracleMesh2D(xy, tri)
    n = gm.n_dof
    for alpha, K in ((1.37, (1.0, 0.5)), (1.9, (2.0, 3.0)))[: 2 if shape in SHAPES else 1]:
        want = om.assemble(quad, alpha, K)
        A = torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
        gm.assemble(F.params2d(alpha, K, quad_points=quad), A)
        torch.cuda.synchronize()
        assert rel(A.cpu().numpy(), want) <= 1e-10


def test_strided_matrix_and_second_rule():
    """lda beyond the unknowns, the columns past them left alone; both rules of one mesh."""
    xy, tri = grid(30, 20)
    gm, om = F.Mesh2D(xy, tri), oracle.OracleMesh2D(xy, tri)
    n = gm.n_dof
    for quad in (3, 7, 3):
        A = torch.full((n, n + 5), -7.0, dtype=torch.float64, device="cuda")
        gm.assemble(F.params2d(1.6, (1.0, 1.0), quad_points=quad), A)
        torch.cuda.synchronize()
        assert rel(A[:, :n].cpu().numpy(), om.assemble(quad, 1.6, (1.0, 1.0))) <= 1e-10
        assert bool((A[:, n:] == -7.0).all())
