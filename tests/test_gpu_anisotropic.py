"""Meshes whose elements are longer along one axis: the tubes follow the elements'
shape, so that stretching a mesh along an axis leaves the sizes of its tubes alone,
and matrix, product and general form match the oracle's (1e-11 max-norm relative,
the bar of the other assembly tests)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_03339_amd as F
from test_gpu_plane_tubes import grid
from test_gpu_tubes import bar, rel

pytestmark = pytest.mark.gpu

K = (1.0, 0.5, 2.0)


@pytest.mark.parametrize("stretch", [(1.0, 0.02, 0.02), (1.0, 1.0, 50.0), (0.1, 1.0, 10.0)])
def test_tubes_follow_the_elements(stretch):
    xyz, tet = bar(20, 6, 6)
    wide = F.Mesh(xyz, tet).plan_info(4)["max_tube_nodes"]
    xyz = xyz * np.array(stretch)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    assert abs(gm.plan_info(4)["max_tube_nodes"] - wide) <= 0.1 * wide
    want = om.assemble(4, 1.37, K)
    A = F.new_matrix(gm)
    gm.assemble(F.params(1.37, K), A)
    x = torch.tensor(np.random.default_rng(1).normal(size=gm.n_dof), device="cuda")
    y = torch.empty_like(x)
    gm.apply(F.params(1.37, K), x, y)
    torch.cuda.synchronize()
    assert rel(A.cpu().numpy(), want) <= 1e-11
    assert rel(y.cpu().numpy(), want @ x.cpu().numpy()) <= 1e-11
    a, b, c = (0.3, 0.8, 0.55), (0.9, 0.4, 0.7), np.random.default_rng(2).uniform(-1.0, 2.0, (6, 4 * len(tet)))
    gm.form_assemble(F.form_params(a, b, quad_points=4, coef=F.FPDE_COEF_USER), A, torch.tensor(c, device="cuda"))
    torch.cuda.synchronize()
    assert rel(A.cpu().numpy(), om.assemble_form(4, a, b, c)) <= 1e-11


@pytest.mark.parametrize("stretch", [0.02, 50.0])
def test_plane(stretch):
    xy, tri = grid(40, 12)
    xy = xy * np.array([1.0, stretch])
    gm, om = F.Mesh2D(xy, tri), oracle.OracleMesh2D(xy, tri)
    A = torch.empty((gm.n_dof, gm.n_dof), dtype=torch.float64, device="cuda")
    gm.assemble(F.params2d(1.37, (1.0, 0.5), quad_points=7), A)
    torch.cuda.synchronize()
    assert rel(A.cpu().numpy(), om.assemble(7, 1.37, (1.0, 0.5))) <= 1e-10
