"""An infinity or NaN in the vector of a matrix-free product reaches the rows
that some pair of half-rays couples to its node, and no other row.

The other rows have the same bits as with a zero in its place: the same
products are added in the same order.
"""
import numpy as np
import pytest
import torch

import paper_1811_03339_amd as F
from test_gpu_tubes import bar

pytestmark = pytest.mark.gpu


def couplings(gm, G, quad):
    """C[j, k]: nodes j and k are entries of opposite half-rays of some Gauss point and axis."""
    n = gm.n_dof
    C = np.zeros((n, n), dtype=bool)
    for axis in range(3):
        side = []
        for d in (2 * axis, 2 * axis + 1):
            off, dof, _ = gm.ray_values(quad, 1.37, d, 0, G)
            M = np.zeros((G, n), dtype=np.float32)
            M[np.repeat(np.arange(G), np.diff(off)), dof] = 1.0
            side.append(M)
        C |= (side[0].T @ side[1]) > 0.0
    return C | C.T


@pytest.mark.parametrize("quad", [4, 11])
@pytest.mark.parametrize("shape", [(3, 4, 17), (6, 6, 6), (3, 3, 75)])
def test_nonfinite_entry_stays_in_its_column(shape, quad):
    xyz, tet = bar(*shape)
    gm = F.Mesh(xyz, tet)
    n = gm.n_dof
    C = couplings(gm, len(tet) * quad, quad)
    p = F.params(1.37, (1.0, 0.5, 2.0), quad_points=quad)
    x = np.random.default_rng(n).normal(size=n)

    def product(node, v):
        x1 = x.copy()
        x1[node] = v
        y = torch.full((n,), -3.0, dtype=torch.float64, device="cuda")
        gm.apply(p, torch.tensor(x1, device="cuda"), y)
        torch.cuda.synchronize()
        return y.cpu().numpy()

    for node in (0, 1, n // 2, n - 1):
        zero, coupled = product(node, 0.0), C[:, node]
        assert shape == (3, 3, 75) or not coupled.all()
        for v in (np.inf, -np.inf, np.nan):
            y = product(node, v)
            assert not np.isfinite(y[coupled]).any()
            assert np.array_equal(y[~coupled], zero[~coupled])
