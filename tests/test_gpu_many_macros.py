"""Grids of many macros against the oracle: most points lie on macro boundaries,
shared DoFs have many copies, and tiles of shared DoFs fill many workgroups.

FP64 within 1e-12 of the largest entry, FP32 within 1e-5 (sums of at most 24
macros' parts of at most 30 products each, u32 = 6e-8).
"""
import numpy as np
import pytest

import harness
import paper_2305_15116_amd as P
from oracle.oracle import OracleMesh, prolongation
from paper_2305_15116_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def grid2(k):
    """k x k squares of two triangles."""
    co = np.array([[i, j] for j in range(k + 1) for i in range(k + 1)], dtype=np.float64)
    v = np.array([[j * (k + 1) + i for i in range(k)] for j in range(k)]).ravel()
    ce = np.stack([np.stack([v, v + 1, v + k + 1], 1), np.stack([v + k + 2, v + k + 1, v + 1], 1)], 1).reshape(-1, 3)
    return W.apply_affine(co, *W.random_affine(2, 9)), W.shuffle_cell_orders(ce, 4)


def grid3(k):
    """k x k x k cubes of six tets."""
    co1, ce1 = W.kuhn_cube()
    vid = lambda p: int(p[0] + (k + 1) * (p[1] + (k + 1) * p[2]))  # noqa: E731
    co = np.array([[x, y, z] for z in range(k + 1) for y in range(k + 1) for x in range(k + 1)], dtype=np.float64)
    ce = np.array([[vid(co1[v] + o) for v in cell] for o in np.ndindex(k, k, k) for cell in ce1])
    return W.apply_affine(co, *W.random_affine(3, 9)), W.shuffle_cell_orders(ce, 4)


MESHES = [(2, 13, 0), (2, 13, 3), (2, 16, 5), (3, 2, 1), (3, 3, 2), (3, 3, 3), (3, 2, 4)]


def _case(dim, k, L, dirichlet, dtype):
    co, ce = (grid2 if dim == 2 else grid3)(k)
    m = P.create_macro_mesh(co, ce, L, P.MF_FLAG_DIRICHLET if dirichlet else 0)
    om = OracleMesh(co, ce, L)
    s2u = harness.storage_to_unique(P.mesh_dof_keys(m, L), om.keys())
    s, _ = P.mesh_num_dofs(m, L)
    x, b = (torch.empty(s, dtype=dtype, device="cuda") for _ in range(2))
    P.mesh_fill_random(m, L, 31, x)
    P.mesh_fill_random(m, L, 32, b)
    return m, om, s2u, x, b


def _unique(om, s2u, v):
    u = np.zeros(om.n)
    u[s2u] = v.cpu().numpy()
    return u


def _check(got, want, s2u, tol):
    got = got.cpu().numpy()
    assert np.isfinite(got).all() and harness.copies_consistent(got, s2u)
    assert harness.rel_err_max(got.astype(np.float64), want[s2u]) <= tol


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("dim,k,L", MESHES)
def test_rows(dim, k, L, dirichlet, dtype):
    m, om, s2u, x, b = _case(dim, k, L, dirichlet, dtype)
    tol = 1e-12 if dtype == torch.float64 else 1e-5
    y, r, t, v = (torch.full_like(x, float("nan")) for _ in range(4))
    P.apply_stencil(m, L, x, y)
    P.residual(m, L, b, x, r, norm=True)
    xs = x.clone()
    P.smooth(m, L, 0.6, 1, b, xs, t)
    kc = b * 0.75 + 1.5
    P.apply_varcoef(m, L, kc, x, v)
    torch.cuda.synchronize()
    xu, bu, ku = (_unique(om, s2u, q) for q in (x, b, kc))
    A = om.csr(dirichlet=dirichlet)
    ax = A @ xu
    fixed = om.boundary() if dirichlet else np.zeros(om.n, dtype=bool)
    _check(y, ax, s2u, tol)
    _check(r, bu - ax, s2u, tol)
    _check(xs, np.where(fixed, xu, xu + 0.6 / A.diagonal() * (bu - ax)), s2u, 2 * tol)
    _check(v, om.csr_varcoef(ku, dirichlet=dirichlet) @ xu, s2u, tol)


# coarse levels with fewer and with more copies of shared DoFs than one launch takes (2^18 in 2D; 2^19 and 5 2^17 in 3D)
@pytest.mark.parametrize("dim,k,L", [(2, 40, 4), (2, 120, 3), (3, 6, 3), (3, 16, 3)])
def test_restriction(dim, k, L):
    co, ce = (grid2 if dim == 2 else grid3)(k)
    om, oc = OracleMesh(co, ce, L), OracleMesh(co, ce, L - 1)
    Pm = prolongation(om, oc)
    s2u = c2u = None
    for dirichlet in (True, False):
        m = P.create_macro_mesh(co, ce, L, P.MF_FLAG_DIRICHLET if dirichlet else 0)
        if s2u is None:
            s2u = harness.storage_to_unique(P.mesh_dof_keys(m, L), om.keys())
            c2u = harness.storage_to_unique(P.mesh_dof_keys(m, L - 1), oc.keys())
        for dtype in (torch.float64, torch.float32):
            r = torch.empty(len(s2u), dtype=dtype, device="cuda")
            P.mesh_fill_random(m, L, 6, r)
            b = torch.full((len(c2u),), float("nan"), dtype=dtype, device="cuda")
            P.restrict_residual(m, L, r, b)
            ru = _unique(om, s2u, r)
            if dirichlet:
                ru[om.boundary()] = 0.0
            want = Pm.T @ ru
            if dirichlet:
                want[oc.boundary()] = 0.0
            _check(b, want, c2u, 1e-13 if dtype == torch.float64 else 1e-5)
