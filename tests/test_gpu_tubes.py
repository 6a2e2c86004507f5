"""The tube accumulation on bars of a x b x c Kuhn cells, whose chords along
the bar have from a few to several hundred entries and whose tubes have from
a few to several hundred nodes: steps of 64 entries exactly filled, exceeded
and nearly empty, blocks that fit the LDS as a square, as a packed triangle
and only in bands of it.  The Riesz matrix (plain and with the fixed order of
additions), its CSR form, the general form (constant coefficients and one per
Gauss point) and the matrix-free product against the oracle.

Bound: every entry is a sum of at most a few thousand products; 1e-11
(max-norm relative) is the bar of the other assembly tests, whose sums are
longer.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1811_03339_amd as F

pytestmark = pytest.mark.gpu


def bar(a, b, c):
    """a x b x c cubes of edge 1/4 cut into six tetrahedra each; interior vertices moved."""
    m = np.array([a, b, c]) + 1
    g = np.stack(np.meshgrid(*[np.arange(k) for k in m], indexing="ij"), -1).reshape(-1, 3)
    inner = ((g > 0) & (g < m - 1)).all(1)
    xyz = 0.25 * (g + np.where(inner[:, None], np.random.default_rng(c).uniform(-0.1, 0.1, g.shape), 0.0))
    vid = lambda p: (p[0] * m[1] + p[1]) * m[2] + p[2]  # noqa: E731
    tets = []
    for i in np.ndindex(a, b, c):
        for perm in [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]:
            p = list(i)
            t = [vid(p)]
            for ax in perm:
                p[ax] += 1
                t.append(vid(p))
            tets.append(t)
    return xyz, np.array(tets, dtype=np.int32)


def rel(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


BARS = [(2, 2, 2), (2, 2, 9), (3, 3, 17), (3, 3, 26), (4, 3, 40), (3, 3, 75)]


@pytest.mark.parametrize("quad", [4, 11])
@pytest.mark.parametrize("shape", BARS)
def test_matrix_matches_oracle(shape, quad):
    xyz, tet = bar(*shape)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    info = gm.plan_info(quad)
    print(f"[case] {shape} {quad} n={gm.n_dof} longest {info['max_entries']} nodes {info['max_tube_nodes']}", flush=True)
    K = (1.0, 0.5, 2.0)
    want = om.assemble(quad, 1.37, K)
    A = F.new_matrix(gm)
    for det in (False, True):
        A.fill_(float("nan"))
        gm.assemble(F.params(1.37, K, quad_points=quad, deterministic=det), A)
        torch.cuda.synchronize()
        assert rel(A.cpu().numpy(), want) <= 1e-11
    first = A.clone()
    gm.assemble(F.params(1.6, K, quad_points=quad, deterministic=True), A)
    gm.assemble(F.params(1.37, K, quad_points=quad, deterministic=True), A)
    torch.cuda.synchronize()
    assert torch.equal(first, A)
    rp, col = gm.template_csr()
    val = torch.empty(col.numel(), dtype=torch.float64, device="cuda")
    gm.assemble_csr(F.params(1.37, K, quad_points=quad), rp, col, val)
    torch.cuda.synchronize()
    rows = np.repeat(np.arange(gm.n_dof), np.diff(rp.cpu().numpy()))
    assert np.abs(val.cpu().numpy() - want[rows, col.cpu().numpy()]).max() <= 1e-11 * np.abs(want).max()


@pytest.mark.parametrize("quad", [4, 11])
@pytest.mark.parametrize("shape", BARS)
def test_product_and_cg_match_oracle(shape, quad):
    """K x and (through the preconditioner) the diagonal, matrix-free; the
    product twice gives the same bits."""
    xyz, tet = bar(*shape)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    K, n = (1.0, 0.5, 2.0), gm.n_dof
    want = om.assemble(quad, 1.37, K)
    x = np.random.default_rng(n).normal(size=n)
    p = F.params(1.37, K, quad_points=quad)
    y = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2)]
    for v in y:
        gm.apply(p, torch.tensor(x, device="cuda"), v)
    torch.cuda.synchronize()
    assert rel(y[0].cpu().numpy(), want @ x) <= 1e-11
    assert torch.equal(y[0], y[1])
    u = torch.empty_like(y[0])
    info = gm.cg_solve(p, torch.tensor(x, device="cuda"), u, tol=1e-12)
    torch.cuda.synchronize()
    assert info.final_rel_residual <= 1e-10 and 1 <= info.ir_iters <= n + 50
    assert rel(u.cpu().numpy(), np.linalg.solve(want, x)) <= 1e-8


def test_bars_reach_every_band():
    """The shapes above have the half-rays and tubes that they are chosen for."""
    sizes = [F.Mesh(*bar(*s)).plan_info(4) for s in BARS]
    longest, nodes = [s["max_entries"] for s in sizes], [s["max_tube_nodes"] for s in sizes]
    assert min(longest) <= 16 and any(16 < v <= 64 for v in longest) and max(longest) > 128
    assert min(nodes) <= 141 and any(141 < v <= 200 for v in nodes) and max(nodes) > 200


@pytest.mark.parametrize("user", [False, True])
@pytest.mark.parametrize("shape", BARS[:1] + BARS[2:5])
def test_form_matches_oracle(shape, user):
    xyz, tet = bar(*shape)
    gm, om = F.Mesh(xyz, tet), oracle.OracleMesh(xyz, tet)
    quad, a, b = 4, (0.3, 0.8, 0.55), (0.9, 0.4, 0.7)
    cl, cr = (1.0, 0.5, 2.0), (0.7, 1.5, 0.25)
    coef = np.repeat(np.array(cl + cr)[:, None], len(tet) * quad, 1)
    if user:
        coef = np.random.default_rng(3).uniform(-1.0, 2.0, coef.shape)
    A = F.new_matrix(gm)
    p = F.form_params(a, b, cl, cr, quad, F.FPDE_COEF_USER if user else F.FPDE_COEF_CONST)
    gm.form_assemble(p, A, torch.tensor(coef, device="cuda") if user else None)
    torch.cuda.synchronize()
    assert rel(A.cpu().numpy(), om.assemble_form(quad, a, b, coef)) <= 1e-11
