"""The 3D walk's FP32 rows are no further from 64 bits than a plain FP32 sum.

Interior rows of every macro in FP32, against the exact sums of the same FP64
stencil and input, beside a sum of fused products in the stencil's order (each
step rounded to FP32): the walk's order may not make the error larger.
"""
import numpy as np
import pytest

import paper_2305_15116_amd as P
from paper_2305_15116_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

OFF3 = [(0, 0, -1), (1, 0, -1), (0, 1, -1), (-1, 1, -1), (0, -1, 0), (1, -1, 0), (-1, 0, 0), (0, 0, 0),
        (1, 0, 0), (-1, 1, 0), (0, 1, 0), (0, -1, 1), (1, -1, 1), (-1, 0, 1), (0, 0, 1)]


def _mesh(name):
    if name == "cube":
        return W.kuhn_cube()
    co, ce = W.strip_3d(int(name[5:]))
    return W.apply_affine(co, *W.random_affine(3, 5)), W.shuffle_cell_orders(ce, 7)


@pytest.mark.parametrize("name,L", [("cube", 4), ("cube", 6), ("strip11", 5), ("strip3", 6)])
def test_rows(name, L):
    co, ce = _mesh(name)
    m = P.create_macro_mesh(co, ce, L)
    s, _ = P.mesh_num_dofs(m, L)
    x = torch.empty(s, dtype=torch.float32, device="cuda")
    P.mesh_fill_random(m, L, 17, x)
    y = torch.empty_like(x)
    P.apply_stencil(m, L, x, y)
    xs, ys = x.cpu().numpy(), y.cpu().numpy()
    N = 1 << L
    z, yy, xx = np.meshgrid(*[np.arange(N + 1)] * 3, indexing="ij")
    keep = xx + yy + z <= N
    pts = np.stack([xx[keep], yy[keep], z[keep]], 1)  # storage order
    index = np.zeros((N + 1,) * 3, dtype=np.int64)
    index[pts[:, 0], pts[:, 1], pts[:, 2]] = np.arange(len(pts))
    inner = pts[(pts.min(1) >= 1) & (pts.sum(1) < N)]
    walk = plain = 0.0
    for c in range(len(ce)):
        base = c * len(pts)
        w = P.mesh_stencil(m, L, c)
        exact, acc = np.zeros(len(inner)), np.zeros(len(inner))
        for wo, d in zip(w, OFF3):
            v = xs[base + index[tuple((inner + d).T)]].astype(np.float64)
            exact += wo * v
            acc = (acc + np.float64(np.float32(wo)) * v).astype(np.float32).astype(np.float64)
        got = ys[base + index[tuple(inner.T)]].astype(np.float64)
        walk += ((got - exact) ** 2).sum()
        plain += ((acc - exact) ** 2).sum()
    assert 0.0 < walk <= plain, (walk / plain) ** 0.5
