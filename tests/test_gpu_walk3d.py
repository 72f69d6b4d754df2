"""3D stencil launches against the oracle at the edges of their tile shapes:
the smallest levels (no interior point, then one), the first level of every
band height, meshes whose vertices and edges have more than 64 copies, faces
in every local position, with and without Dirichlet rows.

FP64 within 1e-12 of the largest entry; FP32 applies within 16 u32 (|A| |x|)_i
per row (15 fused products with rounded weights and inputs, and the copies'
sum), residuals and sweeps within 1e-5 and 2e-5 of the largest entry.
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


def _fan(n):
    """n tets around one edge: its points, and both its vertices, have n copies."""
    ring = [[np.cos(2 * np.pi * i / n), np.sin(2 * np.pi * i / n), 0.5] for i in range(n)]
    return (np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 1.0]] + ring),
            np.array([[0, 1, 2 + i, 2 + (i + 1) % n] for i in range(n)], dtype=np.int64))


def _mesh(name):
    if name == "tet":
        return W.unit_tet()
    if name == "cube":
        return W.kuhn_cube()
    if name.startswith("fan"):
        co, ce = _fan(int(name[3:]))
        return co, W.shuffle_cell_orders(ce, 2)
    co, ce = W.strip_3d(int(name[5:]))
    return W.apply_affine(co, *W.random_affine(3, 9)), W.shuffle_cell_orders(ce, 6)


CASES = [("tet", L) for L in (0, 1, 2, 3, 4, 5, 6, 7)] + [("cube", 5), ("strip7", 2), ("strip7", 3), ("strip7", 4),
         ("strip11", 5), ("strip3", 6), ("strip2", 7), ("fan70", 0), ("fan70", 2), ("fan64", 3), ("fan70", 4)]


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
    y = torch.full_like(x, float("nan"))
    r = torch.full_like(x, float("nan"))
    t = torch.full_like(x, float("nan"))
    P.apply_stencil(m, L, x, y)
    nrm = P.residual(m, L, b, x, r, norm=True)
    xs = x.clone()
    P.smooth(m, L, 0.6, 1, b, xs, t)
    torch.cuda.synchronize()
    A = om.csr(dirichlet=dirichlet)
    f64 = dtype == torch.float64
    xo, bo = x.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)
    xu, bu = np.zeros(om.n), np.zeros(om.n)
    xu[s2u], bu[s2u] = xo, bo
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


def test_non_finite_values_stay_with_their_neighbours():
    """A NaN and an infinity in x reach exactly the rows whose stencils hold them."""
    co, ce = _mesh("strip2")
    L = 4
    m = P.create_macro_mesh(co, ce, L)
    om = OracleMesh(co, ce, L)
    s2u = harness.storage_to_unique(P.mesh_dof_keys(m, L), om.keys())
    rng = np.random.default_rng(3)
    A = om.csr(dirichlet=True)
    hit = rng.choice(om.n, 12, replace=False)
    xu = rng.uniform(-1, 1, om.n)
    xu[hit[:6]], xu[hit[6:]] = np.nan, np.inf
    y = torch.empty(len(s2u), dtype=torch.float64, device="cuda")
    P.apply_stencil(m, L, torch.as_tensor(xu[s2u], device="cuda"), y)
    torch.cuda.synchronize()
    bad = (~np.isfinite(xu)).astype(np.float64)
    held = A.copy()  # the stored entries, zeros among them
    held.data[:] = 1.0
    got = np.isfinite(y.cpu().numpy())
    assert got[((held @ bad) == 0)[s2u]].all()
    assert not got[(((A != 0).astype(np.float64) @ bad) > 0)[s2u]].any()
