"""Chords with more nodes than a tube may have (4 096).  In three dimensions the
plan is refused, and soon, also where the nodes outnumber the plan's hash table
(8 192 slots); in two dimensions the matrix is accumulated row by row.

The two-dimensional matrix of a strip of equal cells depends on the distance of
two unknowns along the strip only, so its first and last columns of cells are
compared with the oracle's matrix of a short strip, at the bar of the other
two-dimensional tests (1e-10).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_03339_amd as F
from test_gpu_tubes import bar

pytestmark = pytest.mark.gpu


def strip(nx, ny):
    m = np.array([nx, ny]) + 1
    g = np.stack(np.meshgrid(*[np.arange(k) for k in m], indexing="ij"), -1).reshape(-1, 2)
    a = (np.arange(nx)[:, None] * m[1] + np.arange(ny)).ravel()
    b = a + m[1]
    return 0.125 * g, np.concatenate([np.stack([a, b, b + 1], 1), np.stack([a, b + 1, a + 1], 1)]).astype(np.int32)


@pytest.mark.parametrize("cells", [100, 150])
def test_plan_of_a_tube_with_too_many_nodes_is_refused(cells):
    """Eight thin rows of cells beside a wide one in both directions across the
    chords: a cell of the mean size takes in 8 x 8 rows of interior nodes."""
    xyz, tet = bar(cells, 9, 9)
    t = np.round(4.0 * xyz[:, 1:])
    xyz[:, 1:] = 0.25 * np.where(t <= 8.0, 1e-3 * t, 8e-3 + 9.0 * (t - 8.0))
    gm = F.Mesh(xyz, tet)
    with pytest.raises(F.FpdeError) as e:
        gm.plan(4)
    assert e.value.status == -11
    with pytest.raises(F.FpdeError) as e:
        gm.assemble(F.params(1.5), F.new_matrix(gm))
    assert e.value.status == -11
    assert len(gm.paths(4, 1, 0, 8)[0]) == 8  # the handle is usable


def test_strip_with_long_chords_matches_oracle():
    """Two interior rows of 2 099 nodes: 4 198 a chord along the strip."""
    nx, ncmp = 2100, 40
    gm, om = F.Mesh2D(*strip(nx, 3)), oracle.OracleMesh2D(*strip(ncmp, 3))
    n, k = gm.n_dof, 2 * (ncmp - 1)
    assert n == 2 * (nx - 1)
    A = torch.full((n, n), float("nan"), dtype=torch.float64, device="cuda")
    gm.assemble(F.params2d(1.37, (1.0, 0.5), quad_points=3, max_steps=3 * nx), A)
    torch.cuda.synchronize()
    want = om.assemble(3, 1.37, (1.0, 0.5))
    for part in (A[:k, :k], A[-k:, -k:]):
        assert np.abs(part.cpu().numpy() - want).max() <= 1e-10 * np.abs(want).max()
    assert float((A - A.T).abs().max()) <= 1e-10 * np.abs(want).max()
