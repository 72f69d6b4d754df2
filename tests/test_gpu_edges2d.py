"""2D stencil launches against the oracle where macros share DoFs, which tiles
of their own finish in the same launch: the smallest levels (vertices alone),
strips in shuffled vertex orders, up to the first level of every tile height,
fans whose centre has up to 70 copies (one tile takes 64 per step), with and
without Dirichlet rows.

FP64 within 1e-12 of the largest entry; FP32 applies within 16 u32 (|A| |x|)_i
per row (7 fused products with rounded weights and inputs per copy, and the
copies' sum), residuals and sweeps within 1e-5 and 2e-5 of the largest entry.
"""
import numpy as np
import pytest

import harness
import paper_2305_15116_amd as P
from oracle.oracle import OracleMesh
from paper_2305_15116_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U32 = 2.0 ** -24


def _mesh(name):
    if name.startswith("fan"):  # n triangles around a point
        n = int(name[3:])
        co = np.array([[0.0, 0.0]] + [[np.cos(2 * np.pi * i / n), np.sin(2 * np.pi * i / n)] for i in range(n)])
        return co, W.shuffle_cell_orders(np.array([[0, 1 + i, 1 + (i + 1) % n] for i in range(n)]), 2)
    co, ce = W.strip_2d(int(name[5:]))
    return W.apply_affine(co, *W.random_affine(2, 9)), W.shuffle_cell_orders(ce, 6)


CASES = [("strip2", L) for L in (0, 1, 2, 3, 4, 6, 7, 9, 10)] + [("strip7", 5), ("strip22", 6), ("strip64", 3), ("strip22", 8), ("strip44", 8), ("fan6", 5),
         ("fan64", 0), ("fan64", 2), ("fan70", 0), ("fan70", 1), ("fan70", 5)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("name,L", CASES)
def test_rows_match_oracle(name, L, dirichlet, dtype):
    co, ce = _mesh(name)
    m = P.create_macro_mesh(co, ce, L, P.MF_FLAG_DIRICHLET if dirichlet else 0)
    om = OracleMesh(co, ce, L)
    s2u = harness.storage_to_unique(P.mesh_dof_keys(m, L), om.keys())
    s, _ = P.mesh_num_dofs(m, L)
    x = torch.empty(s, dtype=dtype, device="cuda")
    b = torch.empty_like(x)
    P.mesh_fill_random(m, L, 31, x)
    P.mesh_fill_random(m, L, 32, b)
    y, r, t = (torch.full_like(x, float("nan")) for _ in range(3))
    P.apply_stencil(m, L, x, y)
    nrm = P.residual(m, L, b, x, r, norm=True)
    xs = x.clone()
    P.smooth(m, L, 0.6, 1, b, xs, t)
    torch.cuda.synchronize()
    A = om.csr(dirichlet=dirichlet)
    f64 = dtype == torch.float64
    xu, bu = np.zeros(om.n), np.zeros(om.n)
    xu[s2u], bu[s2u] = x.cpu().numpy(), b.cpu().numpy()
    ax = A @ xu
    fixed = om.boundary() if dirichlet else np.zeros(om.n, dtype=bool)
    got = [v.cpu().numpy() for v in (y, r, xs)]
    for v in got:
        assert np.isfinite(v).all() and harness.copies_consistent(v, s2u)
    if f64:
        assert harness.rel_err_max(got[0], ax[s2u]) <= 1e-12
    else:
        assert (np.abs(got[0] - ax[s2u]) <= (16 * U32 * (abs(A) @ np.abs(xu)))[s2u] + 1e-30).all()
    assert harness.rel_err_max(got[1].astype(np.float64), (bu - ax)[s2u]) <= (1e-12 if f64 else 1e-5)
    assert abs(nrm - np.linalg.norm(bu - ax)) <= (1e-12 if f64 else 1e-5) * np.linalg.norm(bu - ax)
    sweep = np.where(fixed, xu, xu + 0.6 / A.diagonal() * (bu - ax))
    assert harness.rel_err_max(got[2].astype(np.float64), sweep[s2u]) <= (1e-12 if f64 else 2e-5)
