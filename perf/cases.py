"""Workloads by which the library's speed is followed.

Each case is one call (or the short sequence of calls) that a program using
the library makes again and again, on a mesh it has set up before: operator
applies (constant, variable-coefficient, blended, P2), the smoother, the
residual with its norm, the grid transfers, one multigrid solve and a batch of
solves.  Sizes are those of the benchmark and the serving workload (2D levels
up to 14, 3D up to 8, strips of 1 to 64 macros under seeded affine maps) and
the smaller and uneven ones in between; `draw` spreads further cases over the
same ranges.

A case holds: "kind"; "dim"; "k" (macros of a strip: a triangle for k = 1 and
the unit cube's six tets for k = 6); "level"; "dtype"; "affine" (seed of the
map that stretches the strip, 0: none); "order" (seed that permutes each
cell's vertices, 0: canonical); solves also "mode", "rtol".

Input vectors are seeded values on the strip's integer lattice (before the
map), so the copies of a DoF shared by several macros are equal.
"""
from __future__ import annotations

import itertools
import random
import time
from math import comb

import numpy as np
import torch

import paper_2305_15116_amd as P
from paper_2305_15116_amd import workloads as W

DEV = "cuda"
TYPES = {"f64": torch.float64, "f32": torch.float32}


# ---------------------------------------------------------------- the cases
def listed():
    def case(name, kind, dim, k, level, dtype="f64", affine=0, order=0, **more):
        return dict(name=name, kind=kind, dim=dim, k=k, level=level, dtype=dtype, affine=affine, order=order, **more)

    return [
        # the smallest call: one triangle that fits a cache, one launch; what a program pays per call
        case("apply2d_l8_f64", "apply", 2, 1, 8),
        # the headline benchmark: one stretched triangle of 134 million DoFs
        case("apply2d_l14_f64", "apply", 2, 1, 14, affine=2),
        # the 3D benchmark mesh: six tets of a cube, 17 million DoFs
        case("apply3d_cube_l8_f64", "apply", 3, 6, 8),
        # an uneven strip of a coarse level in FP32, vertices in any order: a multigrid level, or a small request
        case("apply3d_strip11_l5_f32", "apply", 3, 11, 5, "f32", affine=5, order=7),
        # a coefficient that varies in space: weights formed on the fly, 3D
        case("varcoef3d_cube_l8_f64", "varcoef", 3, 6, 8),
        # quadratic elements on a strip of five triangles
        case("p2_strip5_l11_f64", "p2", 2, 5, 11, affine=3),
        # curved macros: every element matrix formed on the fly
        case("blended_strip7_l11_f64", "blended", 2, 7, 11, affine=4),
        # the smoother as the mixed-precision cycle runs it on its finest level
        case("smooth3d_cube_l8_f32", "smooth", 3, 6, 8, "f32"),
        # a residual and its norm (the stopping test): a mid-size strip, an odd number of tets
        case("residual3d_strip13_l7_f64", "residual", 3, 13, 7, affine=8, order=3),
        # both transfers between the two finest levels of the mixed-precision cycle
        case("transfer3d_cube_l8_f32", "transfer", 3, 6, 8, "f32"),
        # a whole solve: conjugate gradients around the mixed-precision cycle on the cube
        case("solve3d_cube_l8_mode3", "solve", 3, 6, 8, mode=3, rtol=1e-10),
        # serving: twelve requests of both dimensions and mixed sizes advanced together
        dict(name="batch12_mode3", kind="batch", n=12, mix=1, mode=3, rtol=1e-8, top2=9, top3=6),
    ]


def points(dim, level):
    """Lattice points of one macro."""
    return comb((1 << level) + dim, dim)


def draw(rng):
    kind = rng.choice(["apply", "apply", "apply", "varcoef", "varcoef", "p2", "blended", "smooth", "smooth", "residual",
                       "residual", "transfer", "solve", "solve", "batch"])
    if kind == "batch":
        return dict(kind="batch", n=rng.randint(3, 24), mix=rng.randint(1, 1 << 20), mode=rng.choice([1, 2, 3, 3]),
                    rtol=1e-8, top2=rng.randint(7, 9), top3=rng.randint(5, 6))
    dim = 2 if kind in ("p2", "blended") else rng.choice([2, 3, 3])
    if kind == "solve":
        level, most = (rng.randint(5, 11) if dim == 2 else rng.randint(4, 8)), 4e6 if dim == 2 else 2e7
    else:
        level, most = (rng.randint(5, 14) if dim == 2 else rng.randint(3, 8)), 1.35e8 if kind == "apply" else 4e7
        while points(dim, level) > most:
            level -= 1
    kmax = max(1, min(64, int(most // points(dim, level))))
    k = max(1, min(kmax, int(round(2 ** rng.uniform(0, np.log2(kmax) if kmax > 1 else 0)))))
    c = dict(kind=kind, dim=dim, k=k, level=level, dtype="f64" if kind in ("blended", "solve") else rng.choice(["f64", "f32"]),
             affine=rng.choice([0, rng.randint(1, 1 << 20)]), order=0 if kind == "solve" else rng.choice([0, rng.randint(1, 1 << 20)]))
    if kind == "p2":
        c["level"] -= 1  # its vectors live on the next level
    if kind == "solve":
        c["mode"], c["rtol"] = rng.choice([0, 1, 2, 3, 3, 4, 5]), 1e-8
    return c


def requests_of(case):
    """The meshes of a batch, drawn as the serving workload draws them (levels from 5 up, smaller strips)."""
    r = random.Random(case["mix"])
    out = []
    for _ in range(case["n"]):
        dim = r.randint(2, 3)
        level = r.randint(5, case["top2"] if dim == 2 else case["top3"])
        out.append(dict(kind="solve", dim=dim, k=r.randint(1, 24 if dim == 2 else 9), level=level, dtype="f64",
                        affine=r.randint(1, 1 << 30), order=0, mode=case["mode"], rtol=case["rtol"]))
    return out


# ---------------------------------------------------------------- meshes and inputs
def strip(case):
    """(integer vertex positions, cells, J, mapped vertex coordinates) of the case's mesh."""
    ref, cells = (W.strip_2d if case["dim"] == 2 else W.strip_3d)(case["k"])
    if case["order"]:
        cells = W.shuffle_cell_orders(cells, case["order"])
    J, t = W.random_affine(case["dim"], case["affine"]) if case["affine"] else (np.eye(case["dim"]), np.zeros(case["dim"]))
    return np.rint(ref).astype(np.int64), cells, J, W.apply_affine(ref, J, t)


def lattice(dim, N):
    """Coordinates [x, y(, z)] of a macro's lattice points in storage order (x fastest)."""
    ax = torch.arange(N + 1, device=DEV)
    g = torch.meshgrid(*([ax] * dim), indexing="ij")
    keep = sum(g) <= N
    return [a[keep] for a in reversed(g)]


def shape_of(ref, N):
    """Points of the integer lattice that holds the strip, per axis."""
    return [int(m) * N + 1 for m in ref.max(axis=0)]


def global_ids(ref, cells, N):
    """Index of every storage point in the strip's integer lattice (row-major)."""
    dim = ref.shape[1]
    xi, shape, out = lattice(dim, N), shape_of(ref, N), []
    w = [N - sum(xi)] + xi
    for cell in cells:
        g = torch.zeros_like(xi[0])
        for d in range(dim):
            g = g * shape[d] + sum(w[j] * int(ref[v, d]) for j, v in enumerate(cell))
        out.append(g)
    return torch.cat(out)


def values(seed, ids, n, lo=-1.0, hi=1.0):
    """Seeded uniform values by lattice index."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 62))
    v = torch.rand(n, dtype=torch.float64, device=DEV, generator=gen) * (hi - lo) + lo
    return v[ids]


def on_boundary(cells, dim, N):
    """Storage points on facets that belong to one cell only."""
    facets = {}
    for c, cell in enumerate(cells):
        for j in range(dim + 1):
            facets.setdefault(tuple(sorted(np.delete(cell, j))), []).append((c, j))
    xi = lattice(dim, N)
    w = [N - sum(xi)] + xi
    outer = [set(f) for f, own in facets.items() if len(own) == 1]
    verts = {frozenset(s) for f in outer for n in range(1, dim + 1) for s in itertools.combinations(sorted(f), n)}
    got = []
    for cell in cells:
        support = sum((w[j] != 0).to(torch.int64) << j for j in range(dim + 1))
        table = torch.zeros(1 << (dim + 1), dtype=torch.bool)
        for m in range(1, 1 << (dim + 1)):
            table[m] = frozenset(int(cell[j]) for j in range(dim + 1) if m >> j & 1) in verts
        got.append(table.to(DEV)[support])
    return torch.cat(got)


def inputs(case, seed):
    """The vectors a case's call reads, by name, in storage layout."""
    ref, cells, J, _ = strip(case)
    kind, dim, lv = case["kind"], case["dim"], case["level"] + (case["kind"] == "p2")
    N, t = 1 << lv, TYPES[case["dtype"]]
    ids, n = global_ids(ref, cells, N), int(np.prod(shape_of(ref, N)))
    out = {}
    if kind == "solve":
        out["b"] = values(seed, ids, n).masked_fill_(on_boundary(cells, dim, N), 0.0)
        return out
    out["x"] = values(seed, ids, n).to(t)
    if kind in ("smooth", "residual"):
        out["b"] = values(seed + 1000003, ids, n).to(t)
    if kind == "varcoef":
        out["k"] = values(seed + 1000003, ids, n, 0.5, 2.5).to(t)
    if kind == "blended":  # bubbles that keep the mapped triangles valid
        u = values(seed + 1000003, torch.arange(2 * case["k"], device=DEV), 2 * case["k"], -0.4, 0.4).reshape(-1, 2)
        out["bubble"] = (u @ torch.as_tensor(J.T.copy(), device=DEV)).contiguous()
    if kind == "transfer":
        cids = global_ids(ref, cells, N // 2)
        out["e"] = values(seed + 1000003, cids, int(np.prod(shape_of(ref, N // 2)))).to(t)
    return out


def prepare(case, seed):
    if case["kind"] == "batch":
        subs = requests_of(case)
        members = [prepare(c, seed + 7919 * i) for i, c in enumerate(subs)]
        return dict(case=case, members=members, batch=P.batch_create(len(subs), mode=case["mode"], max_iter=200))
    _, cells, _, coords = strip(case)
    lv = case["level"] + (case["kind"] == "p2")
    s = dict(case=case, mesh=P.create_macro_mesh(coords, cells, lv), **inputs(case, seed))
    if case["kind"] == "solve":
        s["x"] = torch.zeros_like(s["b"])
        s["work"] = torch.empty(P.mesh_workspace_bytes(s["mesh"], lv, case["mode"]), dtype=torch.uint8, device=DEV)
    elif case["kind"] == "smooth":
        s["tmp"] = torch.empty_like(s["x"])
    elif case["kind"] == "transfer":
        s["xf"], s["bc"] = s["x"].clone(), torch.empty_like(s["e"])
    else:
        s["y"] = torch.empty_like(s["x"])
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        for i, m in enumerate(s["members"]):
            m["x"].zero_()
            P.batch_add(s["batch"], m["mesh"], m["case"]["level"], m["b"], m["x"], m["work"], m["case"]["rtol"], i)
        left = len(s["members"])
        while left:
            left -= len(P.batch_step(s["batch"]))
        return [m["x"] for m in s["members"]]
    mesh, level = s["mesh"], case["level"]
    if kind == "apply":
        P.apply_stencil(mesh, level, s["x"], s["y"])
    elif kind == "varcoef":
        P.apply_varcoef(mesh, level, s["k"], s["x"], s["y"])
    elif kind == "p2":
        P.apply_p2(mesh, level, s["x"], s["y"])
    elif kind == "blended":
        P.apply_blended(mesh, level, s["bubble"], s["x"], s["y"])
    elif kind == "smooth":  # two sweeps, in place
        P.smooth(mesh, level, 2.0 / 3.0, 2, s["b"], s["x"], s["tmp"])
        return s["x"]
    elif kind == "residual":
        return s["y"], P.residual(mesh, level, s["b"], s["x"], s["y"], norm=True)
    elif kind == "transfer":  # down, and the correction up onto an iterate
        P.restrict_residual(mesh, level, s["x"], s["bc"])
        P.prolong_add(mesh, level, s["e"], s["xf"])
        return s["bc"], s["xf"]
    else:
        s["x"].zero_()
        P.vcycle_solve(mesh, level, s["b"], s["x"], s["work"], mode=case["mode"], max_iter=200, rtol=case["rtol"])
        return s["x"]
    return s["y"]


def work(case):
    if case["kind"] == "batch":
        all_ = [work(c) for c in requests_of(case)]
        return {k: sum(w[k] for w in all_) for k in ("bytes", "flops")}
    kind, dim, e = case["kind"], case["dim"], 8 if case["dtype"] == "f64" else 4
    lv = case["level"] + (kind == "p2")
    n = case["k"] * points(dim, lv)
    stencil = 13 if dim == 2 else 29
    if kind == "apply":
        return {"bytes": 2 * e * n, "flops": stencil * n}
    if kind == "varcoef":  # per point and element: mean of the coefficient, its row, their product
        return {"bytes": 3 * e * n, "flops": (6 * 10 if dim == 2 else 24 * 12) * n}
    if kind == "p2":  # 19 and three times 9 entries per four points
        return {"bytes": 2 * e * n, "flops": 2 * 46 / 4 * n}
    if kind == "blended":
        return {"bytes": 2 * e * n, "flops": 60 * n}
    if kind == "smooth":
        return {"bytes": 3 * e * n, "flops": 2 * (stencil + 3) * n}
    if kind == "residual":
        return {"bytes": 3 * e * n, "flops": (stencil + 3) * n}
    if kind == "transfer":
        c = case["k"] * points(dim, lv - 1)
        return {"bytes": e * (3 * n + 2 * c), "flops": 11 * n}
    # a solve of 16 iterations: per iteration the cycle's four sweeps, residual
    # and transfers on each level (the first sweep, from zero, inside the
    # second) and the outer vectors
    v = 4 if case["mode"] & 1 else 8
    levels = sum(points(dim, l) for l in range(3, lv + 1)) * case["k"]
    return {"bytes": 16 * (14 * v * levels + 80 * n), "flops": 16 * (5 * stencil * levels + (stencil + 12) * n)}


# ---------------------------------------------------------------- 64-bit values
# Micro-elements of one lattice cell: vertex offsets, and how much the anchor
# must stay below N (Bey's refinement; the octahedron is cut along the
# (0,1,0)-(1,0,1) diagonal).
ELEMENTS = {
    2: [([(0, 0), (1, 0), (0, 1)], 1), ([(1, 0), (1, 1), (0, 1)], 2)],
    3: [([(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)], 1), ([(0, 1, 0), (1, 0, 1), (1, 0, 0), (1, 1, 0)], 2),
        ([(0, 1, 0), (1, 0, 1), (1, 1, 0), (0, 1, 1)], 2), ([(0, 1, 0), (1, 0, 1), (0, 1, 1), (0, 0, 1)], 2),
        ([(0, 1, 0), (1, 0, 1), (0, 0, 1), (1, 0, 0)], 2), ([(1, 1, 0), (1, 0, 1), (0, 1, 1), (1, 1, 1)], 3)],
}


def gradients(offs, J, N):
    """(gradients of the P1 basis, volume) of a micro-element of a macro with Jacobian J."""
    dim = len(offs[0])
    E = J @ (np.array(offs[1:], dtype=np.float64) - np.array(offs[0], dtype=np.float64)).T / N
    G = np.linalg.inv(E)
    return np.vstack([-G.sum(axis=0), G]), abs(np.linalg.det(E)) / (2.0 if dim == 2 else 6.0)


def p1_matrix(offs, J, N):
    G, vol = gradients(offs, J, N)
    return vol * G @ G.T


def p2_matrix(offs, J, N):
    """P2 element matrix on a triangle: vertices, then the midpoints of (0,1), (1,2), (0,2)."""
    G, vol = gradients(offs, J, N)
    K = np.zeros((6, 6))
    for lam in ([0.5, 0.5, 0.0], [0.0, 0.5, 0.5], [0.5, 0.0, 0.5]):
        D = [(4 * lam[i] - 1) * G[i] for i in range(3)] + [4 * (lam[i] * G[j] + lam[j] * G[i]) for i, j in ((0, 1), (1, 2), (0, 2))]
        K += vol / 3 * np.array(D) @ np.array(D).T
    return K


class Exact:
    """Plain 64-bit evaluation of a case: elements summed macro by macro on dense lattices."""

    def __init__(self, case, level):
        self.dim, self.N = case["dim"], 1 << level
        self.ref, self.cells, _, self.coords = strip(case)
        self.xi = lattice(self.dim, self.N)
        self.n = self.xi[0].numel()
        self.ids = global_ids(self.ref, self.cells, self.N)
        self.size = int(np.prod(shape_of(self.ref, self.N)))
        self.dirichlet = on_boundary(self.cells, self.dim, self.N)
        self.copies = torch.bincount(self.ids, minlength=self.size)[self.ids].double()
        self.place = tuple(reversed(self.xi))

    def jacobian(self, c):
        return (self.coords[self.cells[c][1:]] - self.coords[self.cells[c][0]]).T

    def dense(self, v, c):
        a = torch.zeros([self.N + 1] * self.dim, dtype=torch.float64, device=DEV)
        a[self.place] = v[c * self.n:(c + 1) * self.n]
        return a

    def joined(self, v):
        """Sums over the copies of each DoF, on every copy."""
        return torch.zeros(self.size, dtype=torch.float64, device=DEV).index_add_(0, self.ids, v)[self.ids]

    def elements(self, matrix, x, weight=None, k=None, diagonal=False, step=1, nodes=None):
        """sum_T K_T x_T over all micro-elements: matrix(macro, type) or weight(macro, type) -> list of per-element entries."""
        n, out = self.N // step, []
        for c in range(len(self.cells)):
            xd, kd = self.dense(x, c), None if k is None else self.dense(k, c)
            yd = torch.zeros_like(xd)
            ax = torch.arange(n, device=DEV)
            total = sum(torch.meshgrid(*([ax] * self.dim), indexing="ij"))
            for t, (offs, slack) in enumerate(ELEMENTS[self.dim]):
                at = nodes(offs) if nodes else offs
                cut = [tuple(slice(o, o + (n - 1) * step + 1, step) for o in reversed(p)) for p in at]
                keep = (total <= n - slack).double()
                if k is not None:
                    keep = keep * sum(kd[s] for s in cut) / len(cut)
                K = matrix(c, t)
                xs = [xd[s] for s in cut]
                for v in range(len(cut)):
                    row = K[v][v] if diagonal else sum(K[v][u] * xs[u] for u in range(len(cut)))
                    yd[cut[v]] += keep * row
            out.append(yd[self.place])
        return self.joined(torch.cat(out))

    def p1(self, x, k=None, diagonal=False):
        mats = {}

        def matrix(c, t):
            if (c, t) not in mats:
                mats[c, t] = p1_matrix(ELEMENTS[self.dim][t][0], self.jacobian(c), self.N).tolist()
            return mats[c, t]
        return self.elements(matrix, x, k=k, diagonal=diagonal)

    def apply(self, x, k=None):
        return torch.where(self.dirichlet, x, self.p1(x, k))

    def p2(self, x):
        def nodes(offs):
            v = [tuple(2 * a for a in p) for p in offs]
            return v + [tuple((a + b) // 2 for a, b in zip(v[i], v[j])) for i, j in ((0, 1), (1, 2), (0, 2))]

        def matrix(c, t):
            return p2_matrix(ELEMENTS[2][t][0], self.jacobian(c), self.N // 2).tolist()
        return torch.where(self.dirichlet, x, self.elements(matrix, x, step=2, nodes=nodes))

    def blended(self, x, bubble):
        N = self.N
        ay, ax = torch.meshgrid(*([torch.arange(N + 1, device=DEV).double() / N] * 2), indexing="ij")
        hat = (1 - ax - ay) * ax * ay

        def matrix(c, t):
            J, offs = self.jacobian(c), ELEMENTS[2][t][0]
            cut = [tuple(slice(o, o + N) for o in reversed(p)) for p in offs]
            pos = []  # vertex positions relative to the first vertex: affine part exact, bubble differences
            for p, s in zip(offs, cut):
                d = J @ (np.array(p, float) - np.array(offs[0], float)) / N
                h = hat[s] - hat[cut[0]]
                pos.append((d[0] + float(bubble[c, 0]) * h, d[1] + float(bubble[c, 1]) * h))
            e = [(pos[(i + 2) % 3][0] - pos[(i + 1) % 3][0], pos[(i + 2) % 3][1] - pos[(i + 1) % 3][1]) for i in range(3)]
            det = (e[1][0] * e[2][1] - e[1][1] * e[2][0]).abs()
            det = torch.where(det > 0, det, torch.ones_like(det))
            return [[(e[i][0] * e[j][0] + e[i][1] * e[j][1]) / (2 * det) for j in range(3)] for i in range(3)]
        return torch.where(self.dirichlet, x, self.elements(matrix, x))

    def restricted(self, r, coarse):
        """P^T r on the coarse lattice: each fine DoF counted once, Dirichlet DoFs left out."""
        r = torch.where(self.dirichlet, 0.0, r / self.copies)
        out = []
        for c in range(len(self.cells)):
            a = torch.nn.functional.pad(self.dense(r, c), [1, 1] * self.dim)
            even = lambda d: a[tuple(slice(1 + o, 2 + o + self.N, 2) for o in reversed(d))]  # noqa: E731
            s = even((0,) * self.dim) + 0.5 * sum(even(d) for d in neighbours(self.dim))
            out.append(s[coarse.place])
        return torch.where(coarse.dirichlet, 0.0, coarse.joined(torch.cat(out)))

    def prolonged(self, e, coarse):
        """P e: coarse values at even points, means of the two ends of a coarse micro-edge at the others."""
        out = []
        for c in range(len(self.cells)):
            a, f = coarse.dense(e, c), torch.zeros([self.N + 1] * self.dim, dtype=torch.float64, device=DEV)
            f[(slice(0, None, 2),) * self.dim] = a
            n = self.N // 2
            for d in neighbours(self.dim):
                if d < tuple([0] * self.dim):
                    continue  # one of each pair +-d
                lo = [max(0, -o) for o in d]  # coarse anchors p with p and p + d on the lattice
                size = [n + 1 - abs(o) for o in d]
                u = a[tuple(slice(l, l + s) for l, s in reversed(list(zip(lo, size))))]
                v = a[tuple(slice(l + o, l + o + s) for l, s, o in reversed(list(zip(lo, size, d))))]
                f[tuple(slice(2 * l + o, 2 * (l + s - 1) + o + 1, 2) for l, s, o in reversed(list(zip(lo, size, d))))] = 0.5 * (u + v)
            out.append(f[self.place])
        return torch.where(self.dirichlet, 0.0, torch.cat(out))

    def solved(self, b, seconds=9.0):
        """The solution for a canonical strip, whose refinement is one grid with one stencil: plain conjugate
        gradients on that grid; None if that takes too long."""
        shape = shape_of(self.ref, self.N)
        step = (self.ref[self.cells[0][1:]] - self.ref[self.cells[0][0]])  # grid step of each lattice direction
        stencil = {}
        for t, (offs, _) in enumerate(ELEMENTS[self.dim]):
            K = p1_matrix(offs, self.jacobian(0), self.N)
            for v, u in itertools.product(range(len(offs)), repeat=2):
                d = tuple(int(q) for q in (np.array(offs[u]) - np.array(offs[v])) @ step)
                stencil[d] = stencil.get(d, 0.0) + K[v, u]
        scale = max(abs(w) for w in stencil.values())
        stencil = {d: w for d, w in stencil.items() if abs(w) > 1e-14 * scale}
        free = torch.zeros(self.size, dtype=torch.float64, device=DEV)
        free[self.ids[~self.dirichlet]] = 1.0
        free = free.reshape(shape)
        rhs = torch.zeros(self.size, dtype=torch.float64, device=DEV)
        rhs[self.ids] = b
        rhs = rhs.reshape(shape) * free
        inner = tuple(slice(1, 1 + n) for n in shape)
        p = torch.zeros([n + 2 for n in shape], dtype=torch.float64, device=DEV)
        x, r = torch.zeros_like(rhs), rhs.clone()
        p[inner] = r
        rr = float((r * r).sum())
        stop, began = rr * 1e-28, time.monotonic()
        while rr > stop:
            q = sum(w * p[tuple(slice(1 + o, 1 + o + n) for o, n in zip(d, shape))] for d, w in stencil.items()) * free
            a = rr / float((p[inner] * q).sum())
            x.add_(p[inner], alpha=a)
            r.sub_(q, alpha=a)
            new = float((r * r).sum())
            p[inner] = r + (new / rr) * p[inner]
            rr = new
            if time.monotonic() - began > seconds:
                return None
        return x.reshape(-1)[self.ids]


def neighbours(dim):
    """Lattice directions of the micro-edges."""
    got = set()
    for offs, _ in ELEMENTS[dim]:
        got |= {tuple(b - a for a, b in zip(p, q)) for p in offs for q in offs if p != q}
    return sorted(got)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":  # the first members that are quick to solve by plain means
        subs, began, out = requests_of(case), time.monotonic(), []
        for i, c in enumerate(subs):
            out.append(exact(c, seed + 7919 * i) if time.monotonic() - began < 6 else None)
        return out
    if kind == "solve" and (case["affine"] and case["level"] > (8 if case["dim"] == 2 else 6)):
        return None  # a stretched fine grid takes plain conjugate gradients minutes
    v = {k: t.double() for k, t in inputs(case, seed).items()}
    E = Exact(case, case["level"] + (kind == "p2"))
    if kind == "apply":
        return E.apply(v["x"])
    if kind == "varcoef":
        return E.apply(v["x"], v["k"])
    if kind == "p2":
        return E.p2(v["x"])
    if kind == "blended":
        return E.blended(v["x"], v["bubble"])
    if kind == "smooth":
        x, d = v["x"], E.p1(v["x"], diagonal=True)
        for _ in range(2):
            x = torch.where(E.dirichlet, x, x + (2.0 / 3.0) * (v["b"] - E.p1(x)) / d)
        return x
    if kind == "residual":
        r = v["b"] - E.apply(v["x"])
        return r, float((r.square() / E.copies).sum().sqrt())
    if kind == "transfer":
        C = Exact(case, case["level"] - 1)
        return E.restricted(v["x"], C), v["x"] + E.prolonged(v["e"], C)
    return E.solved(v["b"])
