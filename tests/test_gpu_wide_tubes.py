"""Tubes of many nodes: blocks in several bands of the triangle and in bands of
full rows, few heavy tubes split between workgroups, and the product's and the
diagonal's LDS near its limit (tubes of 2 560 to 4 096 nodes).

The oracle's matrix where it is quick (the bar of 150 cells); the kernels against
each other beyond: the product and the diagonal (their own sums) against the
assembled matrix, the general form with both orders alpha / 2 and both
coefficients K c_alpha, which is the Riesz matrix, against the same.

Bound: 1e-11 (max-norm relative), the bar of the other assembly tests.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_1811_03339_amd as F
from test_gpu_tubes import bar, rel

pytestmark = pytest.mark.gpu

K = (1.0, 0.5, 2.0)
ALPHA = 1.37
# least and largest number of nodes that the widest tube is to have
MESHES = {"bar150": (201, 1024), "bar400": (1025, 2559), "bar800": (2560, 4096), "cube28": (201, 283),
          "block52": (284, 512), "slab": (201, 1024)}


def mesh(name):
    if name.startswith("bar"):
        return bar(int(name[3:]), 3, 3)
    if name == "slab":
        return bar(8, 30, 30)
    return bar(52, 24, 24) if name == "block52" else bar(28, 28, 28)


def close(a, b):
    return float((a - b).abs().max() / b.abs().max()) <= 1e-11


@pytest.mark.parametrize("name", MESHES)
def test_kernels_agree(name):
    xyz, tet = mesh(name)
    gm = F.Mesh(xyz, tet)
    n, quad, G = gm.n_dof, 4, 4 * len(tet)
    lo, hi = MESHES[name]
    assert lo <= gm.plan_info(quad)["max_tube_nodes"] <= hi
    p = F.params(ALPHA, K, quad_points=quad)
    A = F.new_matrix(gm)
    A.fill_(float("nan"))
    gm.assemble(p, A)
    torch.cuda.synchronize()
    if name == "bar150":
        assert rel(A.cpu().numpy(), oracle.OracleMesh(xyz, tet).assemble(quad, ALPHA, K)) <= 1e-11
    # the product, twice the same bits
    x = torch.tensor(np.random.default_rng(n).normal(size=n), device="cuda")
    y = [torch.full_like(x, float("nan")) for _ in range(2)]
    for v in y:
        gm.apply(p, x, v)
    torch.cuda.synchronize()
    assert close(y[0], A @ x) and torch.equal(y[0], y[1])
    # the diagonal, through the first iterate of the conjugate gradients
    u = torch.empty_like(x)
    with pytest.raises(F.FpdeError) as e:
        gm.cg_solve(p, x, u, tol=1e-300, max_iter=1)
    assert e.value.status == -8
    z = x / A.diagonal()
    assert close(u, z * ((x @ z) / (z @ (A @ z))))
    # the general form with the same operators
    c = tuple(k / (2.0 * math.cos(0.5 * math.pi * ALPHA)) for k in K)
    g = (0.5 * ALPHA,) * 3
    coef = torch.tensor(np.repeat(np.array(c + c)[:, None], G, 1), device="cuda")
    B = torch.empty_like(A)
    for kind in (F.FPDE_COEF_CONST, F.FPDE_COEF_USER):
        B.fill_(float("nan"))
        gm.form_assemble(F.form_params(g, g, c, c, quad, kind), B, coef if kind == F.FPDE_COEF_USER else None)
        torch.cuda.synchronize()
        assert close(B, A)
    if n < 2000:  # the fixed order of additions
        first = None
        for _ in range(2):
            gm.assemble(F.params(ALPHA, K, quad_points=quad, deterministic=True), B)
            torch.cuda.synchronize()
            assert close(B, A) and (first is None or torch.equal(first, B))
            first = B.clone()


@pytest.mark.parametrize("user", [False, True])
def test_form_of_a_long_bar_matches_oracle(user):
    """Different trial and test orders, coefficients that vary from point to point."""
    xyz, tet = bar(120, 3, 3)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    quad, a, b = 4, (0.3, 0.8, 0.55), (0.9, 0.4, 0.7)
    cl, cr = (1.0, 0.5, 2.0), (0.7, 1.5, 0.25)
    coef = np.repeat(np.array(cl + cr)[:, None], len(tet) * quad, 1)
    if user:
        coef = np.random.default_rng(3).uniform(-1.0, 2.0, coef.shape)
    A = F.new_matrix(gm)
    A.fill_(float("nan"))
    p = F.form_params(a, b, cl, cr, quad, F.FPDE_COEF_USER if user else F.FPDE_COEF_CONST)
    gm.form_assemble(p, A, torch.tensor(coef, device="cuda") if user else None)
    torch.cuda.synchronize()
    assert rel(A.cpu().numpy(), om.assemble_form(quad, a, b, coef)) <= 1e-11
