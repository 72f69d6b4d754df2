"""Restriction against the transposed interpolation at every storage point: the
smallest levels, row ends, macros in shuffled vertex orders, points with more
than 64 copies, with and without Dirichlet rows.

FP64 within 1e-14 and FP32 within 1e-6 of the largest entry times the number
of copies' terms a DoF can sum (15 per copy, each a rounding of values up to 1).
"""
import numpy as np
import pytest

import harness
import paper_2305_15116_amd as P
from oracle.oracle import OracleMesh
from paper_2305_15116_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(name):
    dim = int(name[0])
    n = int(name[4:])
    if name[1:4] == "fan":  # n cells around a point (2D) or an edge (3D)
        ring = [[np.cos(2 * np.pi * i / n), np.sin(2 * np.pi * i / n), 0.5] for i in range(n)]
        if dim == 2:
            co = np.array([[0.0, 0.0]] + [r[:2] for r in ring])
            ce = np.array([[0, 1 + i, 1 + (i + 1) % n] for i in range(n)])
        else:
            co = np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 1.0]] + ring)
            ce = np.array([[0, 1, 2 + i, 2 + (i + 1) % n] for i in range(n)])
        return co, W.shuffle_cell_orders(ce, 2)
    co, ce = (W.strip_2d if dim == 2 else W.strip_3d)(n)
    return co, W.shuffle_cell_orders(ce, 4)


CASES = [("2row1", L) for L in (1, 2, 3, 7)] + [("2row5", 5), ("2row9", 2), ("2fan70", 1), ("2fan64", 3), ("2fan7", 6)] + \
        [("3row1", L) for L in (1, 2, 3, 5, 6)] + [("3row6", 3), ("3row7", 5), ("3row2", 6), ("3fan70", 2), ("3fan64", 3),
                                                  ("3fan70", 1)]


def _lattice(dim, N):
    """Lattice points of a macro (x, y, z) in storage order: x fastest, z slowest."""
    if dim == 2:
        return np.array([(x, y, 0) for y in range(N + 1) for x in range(N + 1 - y)])
    return np.array([(x, y, z) for z in range(N + 1) for y in range(N + 1 - z) for x in range(N + 1 - z - y)])


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("name,L", CASES)
def test_every_dof(name, L, dirichlet, dtype):
    co, ce = _mesh(name)
    dim, k = co.shape[1], len(ce)
    m = P.create_macro_mesh(co, ce, L, P.MF_FLAG_DIRICHLET if dirichlet else 0)
    om, oc = OracleMesh(co, ce, L), OracleMesh(co, ce, L - 1)
    s2u = harness.storage_to_unique(P.mesh_dof_keys(m, L), om.keys())
    c2u = harness.storage_to_unique(P.mesh_dof_keys(m, L - 1), oc.keys())
    r = torch.empty(len(s2u), dtype=dtype, device="cuda")
    P.mesh_fill_random(m, L, 6, r)
    b = torch.full((len(c2u),), float("nan"), dtype=dtype, device="cuda")
    P.restrict_residual(m, L, r, b)
    got = b.cpu().numpy()
    assert np.isfinite(got).all() and harness.copies_consistent(got, c2u)
    ru = np.zeros(om.n)
    ru[s2u] = r.cpu().numpy()
    if dirichlet:
        ru[om.boundary()] = 0.0
    # each unique fine DoF gives half of itself to either end of the coarse micro-edge it bisects
    N = 1 << L
    pts, cpts = _lattice(dim, N), _lattice(dim, N // 2)
    index = np.zeros((N // 2 + 1,) * 3, dtype=np.int64)
    index[cpts[:, 0], cpts[:, 1], cpts[:, 2]] = np.arange(len(cpts))
    px, py, pz = (pts & 1).T
    s = np.stack([px, np.where((px & py) == 1, -1, py), np.where((pz & (px ^ py)) == 1, -1, pz)], axis=1)
    u, v = index[tuple(((pts - s) >> 1).T)], index[tuple(((pts + s) >> 1).T)]
    want, done = np.zeros(oc.n), np.zeros(om.n, dtype=bool)
    for q in range(k):
        fine, coarse = s2u[q * len(pts):(q + 1) * len(pts)], c2u[q * len(cpts):(q + 1) * len(cpts)]
        new = ~done[fine]
        np.add.at(want, coarse[u[new]], 0.5 * ru[fine[new]])
        np.add.at(want, coarse[v[new]], 0.5 * ru[fine[new]])
        done[fine] = True
    if dirichlet:
        want[oc.boundary()] = 0.0
    assert np.abs(got - want[c2u]).max() <= (1e-14 if dtype == torch.float64 else 1e-6) * 15 * k
