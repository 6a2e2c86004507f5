"""Half-ray vectors and adjoint sums computed from the plan's segments, 64 at a
time in strips of 16 half-rays: rays shorter than a step, rays over several
steps (vertices that stay in the window across a step's end), a last strip of
a direction that is not full, and directions of one launch with their own
orders.  Against the oracle's walk.

Bounds: 1e-10 of the ray's largest value, the bar of the other vector tests;
the adjoint sums are sums of at most 1e6 products of dots of a few hundred
terms, 1e-10 relative as in the other gradient tests.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_03339_amd as F
from test_gpu_tubes import bar

pytestmark = pytest.mark.gpu

BARS = [(2, 2, 2), (2, 2, 9), (3, 3, 26), (3, 3, 75)]


def merged(ids, vals):
    out = {}
    for k, v in zip(ids.tolist(), vals.tolist()):
        out[k] = out.get(k, 0.0) + v
    return out


@pytest.mark.parametrize("quad", [4, 11])
@pytest.mark.parametrize("shape", BARS)
def test_vectors(shape, quad):
    xyz, tet = bar(*shape)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    G = quad * len(tet)
    for alpha, d in ((1.3, 0), (1.3, 5), (1.9, 4), (1.9, 3)):
        for g0 in (0, G // 2, G - 20):
            off, dof, val = gm.ray_values(quad, alpha, d, g0, 20)
            for k in range(20):
                got = merged(dof[off[k]:off[k + 1]], val[off[k]:off[k + 1]])
                want = merged(*om.ray_values(quad, g0 + k, d // 2, d % 2, alpha))
                assert set(got) == set(want)
                scale = max(abs(v) for v in want.values()) if want else 1.0
                assert max((abs(got[q] - want[q]) for q in want), default=0.0) <= 1e-10 * scale


@pytest.mark.parametrize("quad", [4, 11])
@pytest.mark.parametrize("shape", BARS)
def test_adjoint(shape, quad):
    xyz, tet = bar(*shape)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    alpha, K = 1.4, np.array([1.0, 0.5, 2.0])
    rng = np.random.default_rng(11)
    u, lam = rng.uniform(0.5, 1.5, (2, gm.n_dof))
    S, T = om.adjoint_sums(quad, alpha, u, lam)
    ca, dca = oracle.c_alpha(alpha), oracle.dc_alpha(alpha)
    p = F.params(alpha, tuple(K), quad_points=quad)
    ga, gk = gm.adjoint(p, torch.tensor(u, device="cuda"), torch.tensor(lam, device="cuda"))
    want = -float(np.sum(K * (dca * S + ca * T)))
    assert np.abs(gk + ca * S).max() <= 1e-10 * np.abs(ca * S).max()
    assert abs(ga - want) <= 1e-10 * np.sum(K * (abs(dca * S) + abs(ca * T)))
