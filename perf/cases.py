"""Performance cases of the library: what its users have it do, through the
Python entry points, from the smallest call to the largest.

A case names an operation (``op``), a mesh recipe and the options of the
call.  The meshes follow the recipes of ``fpde_inputs`` (one quality round
instead of twelve, so that they are made quickly); the seed turns hull meshes
by a random rotation (for sparse storage: permutes and stretches the axes) and
moves the interior nodes of cubes, which changes the integration paths, and draws the orders, coefficients and sources.

Values of the plan are kept per order by the library, so every pass sweeps
two orders (or several, as a batch): no pass finds the previous one's values.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1811_03339_amd as F
from fpde_inputs import (circle_points, ellipsoid_points, fibonacci_sphere, hull_mesh, kuhn_cube, polygon_mesh,
                         sphere_points)


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: 27 unknowns, the manufactured solution on the unit cube; launches and host round trips
        dict(name="riesz_cube384", op="riesz", mesh="cube", n=4, quad=4, mixed=False, source="mms"),
        # an ordinary FP64 pass: 3 072 unknowns, fine rule, a source given at the Gauss points
        dict(name="riesz_sphere20k", op="riesz", mesh="sphere", hull=400, h=0.104, quad=11, mixed=False,
             source="user"),
        # a large FP64 pass below the factorization's look-ahead size, on the flat ellipsoid's long and short chords
        dict(name="riesz_ellipsoid85k", op="riesz", mesh="ellipsoid", hull=2000, h=0.041, quad=4, mixed=False,
             source="one"),
        # the largest: 25 000 unknowns, 1.7 million Gauss points, FP32 matrix and factor with FP64 refinement
        dict(name="riesz_sphere150k_mixed", op="riesz", mesh="sphere", hull=400, h=0.053, quad=11, mixed=True,
             source="one"),
        # a parameter study: both rules at three orders, assembled and solved as one batch
        dict(name="batch_sphere20k", op="batch", mesh="sphere", hull=400, h=0.104, count=6),
        # the two-sided divergence-form problem on the ball: non-symmetric assembly, LU, solve
        dict(name="sec3_ball_h076", op="div", mesh="ball", hull=1628, h=0.0384, quad=4, coef="sec3", source="ball"),
        # the general form with constant coefficients (every value set anew in each assembly)
        dict(name="form_sphere20k", op="form", mesh="sphere", hull=400, h=0.104, quad=4, coef="const"),
        # the general form with a coefficient at every Gauss point, on a coarse ball with the fine rule
        dict(name="form_user_ball_h139", op="form", mesh="ball", hull=469, h=0.07152, quad=11, coef="user"),
        # two dimensions: assembly and dense solve on the disk
        dict(name="plane_disk4k", op="plane", mesh="disk", hull=160, h=0.028, quad=7),
        # sparse storage on the template: assembly into CSR and conjugate gradients
        dict(name="csr_cg_sphere20k", op="csr", mesh="sphere", hull=400, h=0.104, quad=4),
        # no matrix at all: matrix-free conjugate gradients
        dict(name="matfree_cg_ball40k", op="matfree", mesh="sphere", hull=800, h=0.082, quad=4),
        # two steps of parameter estimation: forward solve and gradient in alpha and K
        dict(name="gradient_ball40k", op="grad", mesh="sphere", hull=800, h=0.082, quad=4, mixed=False),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_mesh(rng, n_lo, n_hi):
    """A solid of about n_lo .. n_hi interior nodes."""
    n = _log(rng, n_lo, n_hi)
    kind = rng.choice(["cube", "sphere", "sphere", "ball", "ellipsoid"])
    if kind == "cube":
        return dict(mesh="cube", n=max(2, round(n ** (1.0 / 3.0)) + 1))
    vol, hull = {"sphere": (4.19, (60, 800)), "ball": (0.52, (60, 1200)), "ellipsoid": (1.0, (200, 2000))}[kind]
    return dict(mesh=kind, hull=rng.randint(*hull), h=round((0.8 * vol / n) ** (1.0 / 3.0), 5))


def draw(rng):
    op = rng.choice(["riesz", "riesz", "riesz", "batch", "div", "form", "plane", "csr", "matfree", "grad"])
    if op == "riesz":
        mixed = rng.random() < 0.4
        c = _draw_mesh(rng, 30, 20000 if mixed else 11000)
        src = rng.choice(["one", "user", "mms"] if c["mesh"] == "cube" else ["one", "user"])
        return dict(op=op, **c, quad=rng.choice([4, 11]), mixed=mixed, source=src)
    if op == "batch":
        return dict(op=op, **_draw_mesh(rng, 30, 3000), count=rng.randint(2, 8))
    if op == "div":
        coef = rng.choice(["sec3", "user"])
        return dict(op=op, mesh="ball", hull=rng.randint(60, 1500), h=round(_log(rng, 0.04, 0.16), 5),
                    quad=rng.choice([4, 11]), coef=coef, source=rng.choice(["one", "user", "ball"]))
    if op == "form":
        return dict(op=op, **_draw_mesh(rng, 30, 3500), quad=rng.choice([4, 11]), coef=rng.choice(["const", "user"]))
    if op == "plane":
        return dict(op=op, mesh="disk", hull=rng.randint(16, 240), h=round(_log(rng, 0.028, 0.25), 5),
                    quad=rng.choice([3, 7]))
    if op == "grad":
        return dict(op=op, **_draw_mesh(rng, 30, 6000), quad=rng.choice([4, 11]), mixed=rng.random() < 0.3)
    return dict(op=op, **_draw_mesh(rng, 100, 9000), quad=rng.choice([4, 11]))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
@functools.lru_cache(maxsize=32)
def _base_mesh(kind, n, h):
    if kind == "cube":
        m = kuhn_cube(n, morton=True)
    elif kind == "disk":
        m = polygon_mesh(circle_points(n), h, 31)
    else:
        pts = {"sphere": lambda: sphere_points(n, 2), "ball": lambda: fibonacci_sphere(n, 0.5),
               "ellipsoid": lambda: ellipsoid_points(n, (1.0, 0.7, 0.4), 5)}[kind]()
        m = hull_mesh(pts, h, 7, max_rounds=1)
    return np.ascontiguousarray(m.xyz, dtype=np.float64), np.ascontiguousarray(m.tet, dtype=np.int32)


def _dof_map(cells, n_vert):
    """Unknown of every vertex (-1 on the boundary): vertices on no boundary face, by increasing id."""
    k = cells.shape[1]
    faces = np.concatenate([np.delete(cells, j, axis=1) for j in range(k)])
    faces.sort(axis=1)
    uniq, count = np.unique(faces, axis=0, return_counts=True)
    inner = np.zeros(n_vert, dtype=bool)
    inner[cells.ravel()] = True
    inner[uniq[count == 1].ravel()] = False
    return np.where(inner, np.cumsum(inner) - 1, -1).astype(np.int64)


def _mesh(case, rng):
    xyz, cells = _base_mesh(case["mesh"], case["n"] if case["mesh"] == "cube" else case["hull"], case.get("h"))
    if case["mesh"] == "cube":
        inner = _dof_map(cells, len(xyz)) >= 0
        xyz = xyz + np.where(inner[:, None], rng.uniform(-0.1, 0.1, xyz.shape) / case["n"], 0.0)
    elif case["op"] == "csr":
        # the sparse pattern follows the axes: a change that keeps its size
        xyz = np.ascontiguousarray(xyz[:, rng.permutation(3)] * rng.uniform(0.8, 1.25, 3))
    else:
        q, r = np.linalg.qr(rng.normal(size=(xyz.shape[1],) * 2))
        xyz = np.ascontiguousarray(xyz @ (q * np.sign(np.diag(r))).T)
    return xyz, cells


def _orders(rng, lo, hi):
    """Two different orders, both in (lo, hi)."""
    mid, d = 0.5 * (lo + hi), 0.5 * (hi - lo)
    return [mid - d * rng.uniform(0.05, 0.95), mid + d * rng.uniform(0.05, 0.95)]


def _inputs(case, seed):
    """Everything a call needs, on the host."""
    rng = np.random.default_rng([int(seed), 77])
    xyz, cells = _mesh(case, rng)
    dim, op = xyz.shape[1], case["op"]
    d = dict(xyz=xyz, cells=cells, K=rng.uniform(0.5, 2.0, dim))
    gauss = len(cells) * case.get("quad", 4)
    if op == "div":
        d["beta"] = [rng.uniform(0.55, 0.9, 3), rng.uniform(0.55, 0.9, 3)]
        if case["coef"] == "user":
            # the transport split of the problem: positive on both sides, summing to one
            p = rng.uniform(0.6, 1.0, 3 * gauss)
            d["coef"] = np.concatenate([p, 1.0 - p])
    elif op == "form":
        d["trial"], d["test"] = rng.uniform(0.1, 1.0, 3), rng.uniform(0.1, 1.0, 3)
        d["cl"], d["cr"] = rng.uniform(0.5, 2.0, 3), rng.uniform(0.5, 2.0, 3)
        if case["coef"] == "user":
            d["coef"] = rng.uniform(0.5, 2.0, 6 * gauss)
    elif op == "batch":
        a = np.sort(rng.uniform(1.15, 1.9, (case["count"] + 1) // 2))
        d["alpha"], d["quads"] = [float(a[z // 2]) for z in range(case["count"])], [(4, 11)[z % 2] for z in
                                                                                     range(case["count"])]
    else:
        d["alpha"] = _orders(rng, 1.15, 1.9)
    if case.get("source") == "user":
        d["f"] = rng.uniform(0.5, 1.5, gauss)
    if op == "grad":
        d["gbar"] = rng.uniform(-1.0, 1.0, int((_dof_map(cells, len(xyz)) >= 0).sum()))
    return d


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _vec(n):
    return torch.empty(max(n, 1), dtype=torch.float64, device="cuda")


def prepare(case, seed):
    d, op, quad = _inputs(case, seed), case["op"], case.get("quad")
    mesh = F.Mesh2D(d["xyz"], d["cells"]) if op == "plane" else F.Mesh(d["xyz"], d["cells"])
    s = dict(op=op, mesh=mesh, f=_dev(d["f"]) if "f" in d else None, coef=_dev(d["coef"]) if "coef" in d else None)
    n = mesh.n_dof
    prec = F.FPDE_MIXED if case.get("mixed") else F.FPDE_FP64
    source = {"mms": F.FPDE_SRC_CUBE_MMS, "user": F.FPDE_SRC_USER, "ball": F.FPDE_SRC_BALL_MMS}.get(
        case.get("source"), F.FPDE_SRC_ONE)
    if op == "batch":
        s["p"] = [F.params(a, d["K"], quad_points=q) for a, q in zip(d["alpha"], d["quads"])]
        count = case["count"]
        s["A"] = torch.empty((count, n, n), dtype=torch.float64, device="cuda")
        s["b"], s["u"] = (torch.empty((count, n), dtype=torch.float64, device="cuda") for _ in range(2))
        for q in sorted(set(d["quads"])):
            mesh.plan(q)
        return s
    if op == "plane":
        s["p"] = [F.params2d(a, d["K"], quad_points=quad) for a in d["alpha"]]
        s["A"] = torch.empty((n, n), dtype=torch.float64, device="cuda")
    else:
        mesh.plan(quad)
        if op == "div":
            s["p"] = [F.div_params(b, quad, F.FPDE_COEF_USER if case["coef"] == "user" else F.FPDE_COEF_SEC3,
                                   source, 0.5) for b in d["beta"]]
        elif op == "form":
            kind = F.FPDE_COEF_USER if case["coef"] == "user" else F.FPDE_COEF_CONST
            s["p"] = [F.form_params(a, b, d["cl"], d["cr"], quad, kind)
                      for a, b in ((d["trial"], d["test"]), (d["test"], d["trial"]))]
        elif op == "grad":
            s["gbar"], s["quad"], s["prec"] = _dev(d["gbar"]), quad, prec
            s["alpha"], s["K"] = d["alpha"], d["K"]
        else:
            s["p"] = [F.params(a, d["K"], quad_points=quad, precision=prec, source=source) for a in d["alpha"]]
        if op == "csr":
            s["rp"], s["col"] = mesh.template_csr()
            s["val"] = torch.empty(s["col"].numel(), dtype=torch.float64, device="cuda")
        if op in ("riesz", "div"):
            s["A"] = F.new_matrix(mesh, prec)
        if op == "form":
            s["A"] = [F.new_matrix(mesh), F.new_matrix(mesh)]
    s["b"], s["u"] = _vec(n), [_vec(n), _vec(n)]
    if op == "matfree":
        s["b"].copy_(_dev(np.random.default_rng([int(seed), 78]).uniform(0.5, 1.5, n)))
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    m, op = s["mesh"], s["op"]
    if op == "riesz":
        for p, u in zip(s["p"], s["u"]):
            m.assemble(p, s["A"], s["b"], s["f"])
            m.solve(p, s["A"], s["b"], u)
        return dict(u=s["u"], b=s["b"], A=s["A"])
    if op == "batch":
        m.assemble_batch(s["p"], s["A"], s["b"])
        m.solve_batch(s["A"], s["b"], s["u"])
        return dict(u=s["u"], b=s["b"], A=s["A"])
    if op == "div":
        for p, u in zip(s["p"], s["u"]):
            m.div_assemble(p, s["A"], s["b"], s["coef"], s["f"])
            m.lu_factor(s["A"])
            m.lu_solve(s["A"], s["b"], u)
        return dict(u=s["u"], b=s["b"], A=s["A"])
    if op == "form":
        for p, A in zip(s["p"], s["A"]):
            m.form_assemble(p, A, s["coef"])
        return dict(A=s["A"])
    if op == "plane":
        for p, u in zip(s["p"], s["u"]):
            m.assemble(p, s["A"], s["b"])
            m.solve(s["A"], s["b"], u)
        return dict(u=s["u"], b=s["b"], A=s["A"])
    if op == "csr":
        for p, u in zip(s["p"], s["u"]):
            m.assemble_csr(p, s["rp"], s["col"], s["val"], s["b"])
            m.cg_solve(p, s["b"], u, (s["rp"], s["col"], s["val"]))
        return dict(u=s["u"], b=s["b"], val=s["val"])
    if op == "matfree":
        for p, u in zip(s["p"], s["u"]):
            m.cg_solve(p, s["b"], u)
        return dict(u=s["u"])
    # grad: one step of an optimizer each, on new parameters
    out = []
    for a in s["alpha"]:
        alpha = torch.tensor(a, dtype=torch.float64, requires_grad=True)
        K = torch.tensor(s["K"], dtype=torch.float64, requires_grad=True)
        u = F.FracSolve.apply(alpha, K, m, s["quad"], s["prec"])
        (u * s["gbar"]).sum().backward()
        out.append(dict(u=u.detach(), dalpha=alpha.grad, dK=K.grad))
    return out


# --------------------------------------------------------------------------
# the work of one pass
# --------------------------------------------------------------------------
def work(case):
    xyz, cells = _base_mesh(case["mesh"], case["n"] if case["mesh"] == "cube" else case["hull"], case.get("h"))
    n, t, dim = int((_dof_map(cells, len(xyz)) >= 0).sum()), len(cells), xyz.shape[1]
    # a half-ray meets about t^(1/dim) elements and as many nodes; every pair of half-rays multiplies its entries
    seg = t ** (1.0 / dim)

    def assembly(quad, products=4.0):
        return dim * t * quad * (2 * 30 * seg + products * 0.8 * seg ** 2)

    op, elem = case["op"], 4 if case.get("mixed") else 8
    mesh_bytes = xyz.nbytes + cells.nbytes
    if op == "batch":
        flops = sum(assembly((4, 11)[z % 2]) + n ** 3 / 3 + 2 * n ** 2 for z in range(case["count"]))
        return dict(bytes=mesh_bytes + case["count"] * (8 * n * n + 16 * n), flops=flops)
    quad = case["quad"]
    if op in ("riesz", "plane"):
        one = dict(bytes=elem * n * n + 16 * n, flops=assembly(quad) + n ** 3 / 3 + 2 * n ** 2)
    elif op == "div":
        one = dict(bytes=8 * n * n + 16 * n, flops=assembly(quad, 0.0) + dim * t * quad * 16 * seg + 2 * n ** 3 / 3)
    elif op == "form":
        one = dict(bytes=8 * n * n + (48 * t * quad if case["coef"] == "user" else 0), flops=assembly(quad, 4.0))
    elif op == "csr":
        nnz = min(n * n, 12.0 * n ** (4.0 / 3.0) + 27 * n)
        one = dict(bytes=12 * nnz + 24 * n, flops=assembly(quad) + 45 * 2 * nnz)
    elif op == "matfree":
        one = dict(bytes=24 * n, flops=dim * t * quad * 2 * (30 * seg + 45 * 4 * seg))
    else:
        one = dict(bytes=elem * n * n + 24 * n, flops=assembly(quad) + dim * t * quad * 60 * seg + n ** 3 / 3)
    return dict(bytes=mesh_bytes + 2 * one["bytes"], flops=2 * one["flops"])


# --------------------------------------------------------------------------
# the same in 64 bits from the definitions: every line against every element
# --------------------------------------------------------------------------
def _rule(nq):
    """Barycentric points and weights (summing to one)."""
    pts, w = [], []
    if nq == 4:
        a, b = (5 + 3 * math.sqrt(5)) / 20, (5 - math.sqrt(5)) / 20
        pts, w = [[a if j == q else b for j in range(4)] for q in range(4)], [0.25] * 4
    elif nq == 11:
        pts, w = [[0.25] * 4], [-148 / 1875]
        pts += [[11 / 14 if j == v else 1 / 14 for j in range(4)] for v in range(4)]
        w += [343 / 7500] * 4
        a, b = (1 + math.sqrt(5 / 14)) / 4, (1 - math.sqrt(5 / 14)) / 4
        pts += [[a if j in (v, k) else b for j in range(4)] for v in range(4) for k in range(v + 1, 4)]
        w += [56 / 375] * 6
    elif nq == 3:
        pts, w = [[2 / 3 if j == q else 1 / 6 for j in range(3)] for q in range(3)], [1 / 3] * 3
    else:
        r = math.sqrt(15)
        pts, w = [[1 / 3] * 3], [9 / 40]
        for a, wa in (((6 - r) / 21, (155 - r) / 1200), ((6 + r) / 21, (155 + r) / 1200)):
            pts += [[1 - 2 * a if j == v else a for j in range(3)] for v in range(3)]
            w += [wa] * 3
    return np.array(pts), np.array(w)


class _Lines:
    """Order-gamma derivatives of the basis functions at the Gauss points, by
    cutting each axis-parallel line with every element."""

    def __init__(self, xyz, cells, nq):
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        t64 = functools.partial(torch.tensor, dtype=torch.float64, device=self.dev)
        bary, w = _rule(nq)
        v = t64(xyz[cells])                                   # T, k, dim
        self.dim, self.T, self.nq = v.shape[2], len(cells), nq
        edges = v[:, 1:] - v[:, :1]                           # rows e_1 .. e_dim
        inv = torch.linalg.inv(edges.cpu()).to(self.dev)      # columns: gradients of the coordinates 1 .. dim
        self.grad = torch.cat([-inv.sum(2, keepdim=True), inv], 2).transpose(1, 2).contiguous()  # T, k, dim
        self.c0 = -(self.grad * v[:, :1]).sum(2)
        self.c0[:, 0] += 1.0
        vol = torch.linalg.det(edges.cpu()).abs().to(self.dev) / math.factorial(self.dim)
        self.x = torch.einsum("qk,tkd->tqd", t64(bary), v).reshape(-1, self.dim)
        self.w = (vol[:, None] * t64(w)[None]).reshape(-1)
        self.bary = t64(bary)
        dof = _dof_map(cells, len(xyz))
        self.n = int((dof >= 0).sum())
        self.dof = torch.tensor(dof[cells], device=self.dev)
        self.G = len(self.x)
        self.chunk = max(1, min(self.G, int(1.2e8) // max(self.T, self.n)))

    def chunks(self):
        return [slice(a, min(a + self.chunk, self.G)) for a in range(0, self.G, self.chunk)]

    def cut(self, sl, i):
        """(point in the chunk, element, lo, hi) of the pieces of the lines along e_i."""
        x = self.x[sl]
        lo = torch.full((len(x), self.T), -math.inf, dtype=torch.float64, device=self.dev)
        hi = -lo
        for j in range(self.dim + 1):
            d = self.grad[:, j, i]
            d = torch.where(d.abs() < 1e-13 * self.grad[:, j].abs().amax(1), torch.full_like(d, -1e-200), d)
            b = x @ self.grad[:, j].T + self.c0[:, j]
            r = b.mul_((-1.0 / d)[None])
            inf = torch.full_like(d, math.inf)
            lo = torch.maximum(lo, r + torch.where(d > 0, 0.0, -inf)[None], out=lo)
            hi = torch.minimum(hi, r + torch.where(d < 0, 0.0, inf)[None], out=hi)
        g, t = torch.nonzero(hi - lo > 1e-14, as_tuple=True)
        return g, t, lo[g, t], hi[g, t]

    def values(self, piece, i, gamma):
        """Left and right values (two lists over the local vertices) of the pieces; gamma may need a gradient."""
        g, t, lo, hi = piece
        gamma = torch.as_tensor(gamma, dtype=torch.float64, device=self.dev)
        scale = torch.exp(-torch.lgamma(2.0 - gamma))

        def power(r):
            r = r.clamp(min=0.0)
            return torch.where(r > 0, torch.exp((1.0 - gamma) * torch.log(torch.where(r > 0, r, 1.0))), 0.0)

        right, left = scale * (power(hi) - power(lo)), scale * (power(-lo) - power(-hi))
        slope = self.grad[t, :, i]
        return left[:, None] * slope, -right[:, None] * slope

    def dense(self, piece, val, rows):
        out = torch.zeros(rows * (self.n + 1), dtype=torch.float64, device=self.dev)
        d = self.dof[piece[1]]
        d = torch.where(d < 0, self.n, d)
        out.index_add_(0, (piece[0][:, None] * (self.n + 1) + d).reshape(-1), val.reshape(-1))
        return out.view(rows, self.n + 1)[:, :self.n]

    def own(self, sl, i):
        """Slopes along e_i of the basis functions at the Gauss points."""
        g = torch.arange(self.G, device=self.dev)[sl]
        t = g // self.nq
        return self.dense((g - g[0], t), self.grad[t, :, i], len(g))

    def load(self, f):
        g = torch.arange(self.G, device=self.dev)
        t = g // self.nq
        v = (self.w * f)[:, None] * self.bary[g % self.nq]
        d = self.dof[t]
        out = torch.zeros(self.n + 1, dtype=torch.float64, device=self.dev)
        out.index_add_(0, torch.where(d < 0, self.n, d).reshape(-1), v.reshape(-1))
        return out[:self.n]

    def riesz(self, alphas, K):
        """The stiffness matrices at several orders."""
        out = [torch.zeros((self.n, self.n), dtype=torch.float64, device=self.dev) for _ in alphas]
        for sl in self.chunks():
            w = self.w[sl]
            for i in range(self.dim):
                piece = self.cut(sl, i)
                for a, M in zip(alphas, out):
                    L, R = (self.dense(piece, v, len(w)) for v in self.values(piece, i, 0.5 * a))
                    M += K[i] / (2 * math.cos(math.pi * a / 2)) * (L.T @ (w[:, None] * R))
        return [M + M.T for M in out]


def _factored(M):
    L = torch.linalg.cholesky(M)
    return torch.tril(L) + torch.triu(M, 1), L


def _spd_solve(L, b):
    return torch.cholesky_solve(b[:, None], L)[:, 0]


def _lu(A):
    """L U without row exchanges, in place, 64 columns at a time."""
    n = len(A)
    for k in range(0, n, 64):
        e = min(k + 64, n)
        for j in range(k, e):
            A[j + 1:, j] /= A[j, j]
            A[j + 1:, j + 1:e] -= torch.outer(A[j + 1:, j], A[j, j + 1:e])
        if e < n:
            unit = torch.tril(A[k:e, k:e], -1) + torch.eye(e - k, dtype=A.dtype, device=A.device)
            A[k:e, e:] = torch.linalg.solve_triangular(unit, A[k:e, e:], upper=False, unitriangular=True)
            A[e:, e:] -= A[e:, k:e] @ A[k:e, e:]
    return A


def _cube_source(x, alpha, K):
    phi = x ** 2 * (1 - x) ** 2

    def Phi(s):
        return sum(c * s ** (k - alpha) / math.gamma(k + 1 - alpha) for k, c in ((2, 2.0), (3, -12.0), (4, 24.0)))

    c = 1 / (2 * math.cos(math.pi * alpha / 2))
    f = 0.0
    for i in range(3):
        f = f + K[i] * c * (Phi(x[:, i]) + Phi(1 - x[:, i])) * phi[:, (i + 1) % 3] * phi[:, (i + 2) % 3]
    return f


def _ball_source(x, beta, r):
    f, n2 = 0.0, (x ** 2).sum(1)
    for i in range(3):
        b, xi = beta[i], x[:, i]
        c = (r * r - n2 + xi ** 2).clamp(min=0.0).sqrt()

        def chord(s, up):
            # u = s^4 - 4 c s^3 + 4 c^2 s^2 along the chord; its derivative of order b (+ 1)
            s = s.clamp(min=0.0)
            return sum(a * s ** (k - b - up) / math.gamma(k + 1 - b - up)
                       for k, a in ((2, 8 * c * c), (3, -24 * c), (4, 24.0)))

        sn, cs = torch.sin(xi), torch.cos(xi)
        f = f - sn * chord(xi + c, 0) + cs * chord(xi + c, 1) - sn * chord(c - xi, 0) + (1 - cs) * chord(c - xi, 1)
    return f


def _template(xyz, cells, dev):
    """Pairs of unknowns whose patch boxes overlap in two coordinates at least."""
    lo, hi = np.full(xyz.shape, np.inf), np.full(xyz.shape, -np.inf)
    for j in range(4):
        np.minimum.at(lo, cells[:, j], xyz[cells].min(1))
        np.maximum.at(hi, cells[:, j], xyz[cells].max(1))
    dof = _dof_map(cells, len(xyz))
    lo, hi = (torch.tensor(v[dof >= 0], device=dev) for v in (lo, hi))
    meet = (lo[:, None] <= hi[None]) & (lo[None] <= hi[:, None])
    return meet.sum(2) >= 2


def exact(case, seed):
    op, quad = case["op"], case.get("quad", 11)
    xyz, cells = _base_mesh(case["mesh"], case["n"] if case["mesh"] == "cube" else case["hull"], case.get("h"))
    n = int((_dof_map(cells, len(xyz)) >= 0).sum())
    # lines times elements, and the products over the Gauss points: more would take too long
    if len(cells) ** 2 * quad > 2.4e10 or n > 9000 or len(cells) * quad * n ** 2.0 > 4e13:
        return None
    d = _inputs(case, seed)
    ln = _Lines(d["xyz"], d["cells"], quad)
    x, w = ln.x, ln.w
    if op in ("riesz", "plane", "csr", "matfree"):
        Ms = ln.riesz(d["alpha"], d["K"])
        out = dict(u=[])
        for a, M in zip(d["alpha"], Ms):
            if op == "matfree":
                b = torch.tensor(np.random.default_rng([int(seed), 78]).uniform(0.5, 1.5, n), device=ln.dev)
            elif case.get("source") == "mms":
                b = ln.load(_cube_source(x, a, d["K"]))
            elif case.get("source") == "user":
                b = ln.load(torch.tensor(d["f"], device=ln.dev))
            else:
                b = ln.load(torch.ones_like(w))
            A, L = _factored(M)
            out["u"].append(_spd_solve(L, b))
        if op != "matfree":
            out["b"] = b
        if op in ("riesz", "plane"):
            # the factor, and K above its diagonal
            out["A"] = A
        if op == "csr":
            out["val"] = M[_template(d["xyz"], d["cells"], ln.dev)]
        return out
    if op == "batch":
        out = dict(u=[], b=[], A=[])
        both = {q: _Lines(d["xyz"], d["cells"], q) for q in set(d["quads"])}
        mats = {q: ln_.riesz(sorted({a for a, k in zip(d["alpha"], d["quads"]) if k == q}), d["K"])
                for q, ln_ in both.items()}
        for a, q in zip(d["alpha"], d["quads"]):
            M = mats[q][sorted({v for v, k in zip(d["alpha"], d["quads"]) if k == q}).index(a)]
            A, L = _factored(M)
            b = both[q].load(torch.ones_like(both[q].w))
            out["A"].append(A)
            out["b"].append(b)
            out["u"].append(_spd_solve(L, b))
        return {k: torch.stack(v) for k, v in out.items()}
    if op == "div":
        out = dict(u=[])
        if case["coef"] == "user":
            pq = torch.tensor(d["coef"], device=ln.dev).view(2, 3, -1)
        else:
            pq = torch.stack([torch.cos(x).T, 1 - torch.cos(x).T])
        Ms = [torch.zeros((n, n), dtype=torch.float64, device=ln.dev) for _ in d["beta"]]
        for sl in ln.chunks():
            for i in range(3):
                piece, test = ln.cut(sl, i), ln.own(sl, i)
                for beta, M in zip(d["beta"], Ms):
                    L, R = (ln.dense(piece, v, len(test)) for v in ln.values(piece, i, beta[i]))
                    flux = (w * pq[0, i])[sl, None] * L - (w * pq[1, i])[sl, None] * R
                    M -= test.T @ flux
        for beta, M in zip(d["beta"], Ms):
            f = _ball_source(x, beta, 0.5) if case["source"] == "ball" else (
                torch.tensor(d["f"], device=ln.dev) if case["source"] == "user" else torch.ones_like(w))
            b = ln.load(f)
            A = _lu(M)
            y = torch.linalg.solve_triangular(A, b[:, None], upper=False, unitriangular=True)
            out["u"].append(torch.linalg.solve_triangular(torch.triu(A), y, upper=True)[:, 0])
        out["b"], out["A"] = b, A
        return out
    if op == "form":
        if case["coef"] == "user":
            c = torch.tensor(d["coef"], device=ln.dev).view(2, 3, -1)
        else:
            c = torch.tensor(np.stack([d["cl"], d["cr"]]), device=ln.dev)[:, :, None].expand(2, 3, ln.G)
        out = [torch.zeros((n, n), dtype=torch.float64, device=ln.dev) for _ in range(2)]
        for sl in ln.chunks():
            for i in range(3):
                piece, rows = ln.cut(sl, i), len(w[sl])
                sides = [[ln.dense(piece, v, rows) for v in ln.values(piece, i, o[i])]
                         for o in (d["trial"], d["test"])]
                for k in range(2):
                    (La, Ra), (Lb, Rb) = sides[k], sides[1 - k]
                    out[k] += Rb.T @ ((w * c[0, i])[sl, None] * La) + Lb.T @ ((w * c[1, i])[sl, None] * Ra)
        return dict(A=out)
    # grad: dJ/dp = -lam^T (dK/dp) u with J = gbar . u
    gbar = torch.tensor(d["gbar"], device=ln.dev)
    out, b = [], ln.load(torch.ones_like(w))
    for a, M in zip(d["alpha"], ln.riesz(d["alpha"], d["K"])):
        L = torch.linalg.cholesky(M)
        u, lam = _spd_solve(L, b), _spd_solve(L, gbar)
        alpha = torch.tensor(a, dtype=torch.float64, requires_grad=True)
        K = torch.tensor(d["K"], dtype=torch.float64, requires_grad=True)
        ext = torch.cat([torch.stack([u, lam]), torch.zeros(2, 1, dtype=torch.float64, device=ln.dev)], 1)
        for sl in ln.chunks():
            for i in range(3):
                piece = ln.cut(sl, i)
                dof = ln.dof[piece[1]]
                both = ext[:, torch.where(dof < 0, n, dof)]       # 2, pieces, vertices
                dots = []
                for v in ln.values(piece, i, 0.5 * alpha.to(ln.dev)):
                    rows = torch.zeros((2, len(w[sl])), dtype=torch.float64, device=ln.dev)
                    dots.append(rows.index_add(1, piece[0], (v[None] * both).sum(2)))
                (Lu, Ll), (Ru, Rl) = dots
                S = (w[sl] * (Rl * Lu + Ll * Ru)).sum().cpu()
                (-K[i] / (2 * torch.cos(math.pi * alpha / 2)) * S).backward()
        out.append(dict(u=u, dalpha=alpha.grad, dK=K.grad))
    return out
