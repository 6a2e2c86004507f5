"""Triangular solves whose entries are published over a NaN with all bits set:
right-hand sides that hold that very value, other NaNs and infinities end like
any other, for one block, a partial last block and many blocks; and the solve
may overwrite its right-hand side.
"""
import numpy as np
import pytest
import torch

from test_gpu_diag_block import spd, strip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 1000])
def test_unset_bits_in_the_right_hand_side(n):
    M, b = spd(n, n)
    gm = strip(n)
    ref = torch.tensor(np.linalg.solve(M, b))
    k = n // 2
    for bits in (-1, 0x7FF8000000000000, 0x7FF0000000000000):
        A = torch.tensor(M, device="cuda")
        rhs = torch.tensor(b, device="cuda")
        rhs.view(torch.int64)[k] = bits
        u = torch.empty_like(rhs)
        gm.solve(A, rhs, u)
        torch.cuda.synchronize()
        assert not torch.isfinite(u[k:]).any()
    A, u = torch.tensor(M, device="cuda"), torch.tensor(b, device="cuda")
    gm.solve(A, u, u)
    torch.cuda.synchronize()
    # condition below 10: n eps on the factor, three solves' worth
    assert float((u.cpu() - ref).abs().max()) <= 1e-12 * float(ref.abs().max())
