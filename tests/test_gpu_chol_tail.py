"""Dense Cholesky solves around the size from which the last columns are taken
as one group, and trailing updates whose tile rows do and do not fill the last
super-block, through the dense solve of a two-dimensional handle; and the FP32
factor of a size whose trailing updates run in slices beside the next group.

Bound: Cholesky's normwise backward error is below n eps; its solve with that
factor stays below 3 n eps |A| |u| in the residual.
"""
import numpy as np
import pytest
import torch

import paper_1811_03339_amd as P
from fpde_inputs import kuhn_cube
from test_gpu_diag_block import strip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2113, 2176, 2177, 2177 + 128, 2176 + 896, 2177 + 1024, 6145, 9000])
def test_residual(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    M = torch.randn((n, 2000), dtype=torch.float64, device="cuda", generator=g)
    A = M @ M.T / 2000 + torch.eye(n, dtype=torch.float64, device="cuda")
    b = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    F, u = A.clone(), torch.full_like(b, float("nan"))
    strip(n).solve(F, b, u)
    torch.cuda.synchronize()
    res = float((A @ u - b).norm() / (torch.linalg.matrix_norm(A) * u.norm()))
    assert res <= 3 * n * np.finfo(float).eps
    L = torch.tril(F)
    x = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    err = float((L @ (L.T @ x) - A @ x).norm() / (torch.linalg.matrix_norm(A) * x.norm()))
    assert err <= n * np.finfo(float).eps


def test_sliced_updates():
    """17 576 unknowns, mixed precision: the FP32 factor reproduces the matrix to
    n 2^-24 (normwise, on random vectors), and refinement ends within 5 steps."""
    m = kuhn_cube(27)
    gm = P.Mesh(m.xyz, m.tet)
    n = gm.n_dof
    p = P.params(1.5, (1.0, 0.5, 2.0), quad_points=4, precision=P.FPDE_MIXED)
    A = P.new_matrix(gm, P.FPDE_MIXED)
    b = torch.empty(n, dtype=torch.float64, device="cuda")
    u = torch.empty_like(b)
    gm.assemble(p, A, b)
    A0 = torch.tril(A)
    info = gm.solve(p, A, b, u)
    torch.cuda.synchronize()
    assert info.final_rel_residual <= 1e-8 and info.ir_iters <= 5
    x = torch.randn((n, 2), dtype=torch.float32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    x = x.double()
    L = torch.tril(A)
    got = torch.cat([L[i:i + 2048].double() @ (L.double().T @ x) for i in range(0, n, 2048)])
    D = torch.diagonal(A0).double()[:, None] * x
    want = torch.cat([A0[i:i + 2048].double() @ x for i in range(0, n, 2048)]) + A0.double().T @ x - D
    assert float((got - want).norm() / want.norm()) <= n * 2.0 ** -24
