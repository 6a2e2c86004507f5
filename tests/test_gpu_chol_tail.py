"""Dense Cholesky solves around the size from which the last columns are taken
as one group, and trailing updates whose tile rows do and do not fill the last
super-block, through the dense solve of a two-dimensional handle.

Bound: Cholesky's normwise backward error is below n eps; its solve with that
factor stays below 3 n eps |A| |u| in the residual.
"""
import numpy as np
import pytest
import torch

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
