"""Prolongation against the interpolation formula at every storage point: a
coarse point's cell writes fine points in pairs, so the smallest levels, row
ends, the last point of a macro, slices of 64 points and more, and Dirichlet
faces in every position are where it can go wrong.

x + (u + v) / 2 with u + v rounded once, the half exact and the sum rounded
once: results are equal bit for bit.
"""
import numpy as np
import pytest

import paper_2305_15116_amd as P
from paper_2305_15116_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [(2, 1, L) for L in (1, 2, 3, 6, 7, 8)] + [(2, 5, 5), (2, 9, 3)] + \
        [(3, 1, L) for L in (1, 2, 3, 4, 5, 6)] + [(3, 6, 3), (3, 7, 4), (3, 2, 6)]


def _lattice(dim, N):
    """Lattice points of a macro (x, y, z) in storage order: x fastest, z slowest."""
    if dim == 2:
        return np.array([(x, y, 0) for y in range(N + 1) for x in range(N + 1 - y)])
    return np.array([(x, y, z) for z in range(N + 1) for y in range(N + 1 - z) for x in range(N + 1 - z - y)])


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("dim,k,L", CASES)
def test_every_point(dim, k, L, dirichlet, dtype):
    co, ce = (W.strip_2d if dim == 2 else W.strip_3d)(k)
    ce = W.shuffle_cell_orders(ce, 4)
    m = P.create_macro_mesh(co, ce, L, P.MF_FLAG_DIRICHLET if dirichlet else 0)
    c = torch.empty(P.mesh_num_dofs(m, L - 1)[0], dtype=dtype, device="cuda")
    x = torch.empty(P.mesh_num_dofs(m, L)[0], dtype=dtype, device="cuda")
    P.mesh_fill_random(m, L - 1, 5, c)
    P.mesh_fill_random(m, L, 6, x)
    # Dirichlet points: those a sweep leaves alone
    one, fixed = torch.ones_like(x), torch.zeros_like(x)
    P.smooth(m, L, 0.5, 1, one, fixed, torch.empty_like(x))
    fixed = (fixed == 0).cpu().numpy() if dirichlet else np.zeros(len(x), dtype=bool)
    cn, want = c.cpu().numpy(), x.cpu().numpy().copy()
    P.prolong_add(m, L, c, x)
    N = 1 << L
    pts, cpts = _lattice(dim, N), _lattice(dim, N // 2)
    index = np.zeros((N // 2 + 1,) * 3, dtype=np.int64)
    index[cpts[:, 0], cpts[:, 1], cpts[:, 2]] = np.arange(len(cpts))
    px, py, pz = (pts & 1).T
    s = np.stack([px, np.where((px & py) == 1, -1, py), np.where((pz & (px ^ py)) == 1, -1, pz)], axis=1)
    u, v = index[tuple(((pts - s) >> 1).T)], index[tuple(((pts + s) >> 1).T)]
    for q in range(k):
        cq = cn[q * len(cpts):(q + 1) * len(cpts)]
        add = cq.dtype.type(0.5) * (cq[u] + cq[v])
        part = want[q * len(pts):(q + 1) * len(pts)]
        part += np.where(fixed[q * len(pts):(q + 1) * len(pts)], cq.dtype.type(0), add)
    assert np.array_equal(x.cpu().numpy(), want)
