"""Rows that macros share in the P2, variable-coefficient and blended applies, a
lane per copy in the same launch: fans whose centre has up to 70 copies (64 per
step), strips in shuffled vertex orders, the smallest levels, with and without
Dirichlet rows, against the oracle's matrices within 1e-12 (FP64) and 1e-5
(FP32) of the largest entry; every copy equal.
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
    if name.startswith("fan"):  # n triangles around a point
        n = int(name[3:])
        co = np.array([[0.0, 0.0]] + [[np.cos(2 * np.pi * i / n), np.sin(2 * np.pi * i / n)] for i in range(n)])
        return co, W.shuffle_cell_orders(np.array([[0, 1 + i, 1 + (i + 1) % n] for i in range(n)]), 2)
    co, ce = W.strip_2d(int(name[5:]))
    return W.apply_affine(co, *W.random_affine(2, 9)), W.shuffle_cell_orders(ce, 6)


@pytest.mark.parametrize("kind,dtype", [("p2", torch.float64), ("p2", torch.float32), ("varcoef", torch.float64),
                                        ("varcoef", torch.float32), ("blended", torch.float64)])
@pytest.mark.parametrize("dirichlet", [True, False])
@pytest.mark.parametrize("name,L", [("strip2", 1), ("strip3", 2), ("strip2", 7), ("strip7", 6), ("fan6", 4), ("fan64", 1),
                                    ("fan70", 0), ("fan70", 1), ("fan70", 3)])
def test_shared_rows_match_oracle(name, L, dirichlet, kind, dtype):
    co, ce = _mesh(name)
    lattice = L + 1 if kind == "p2" else L
    m = P.create_macro_mesh(co, ce, lattice, P.MF_FLAG_DIRICHLET if dirichlet else 0)
    om = OracleMesh(co, ce, lattice)
    s2u = harness.storage_to_unique(P.mesh_dof_keys(m, lattice), om.keys())
    x = torch.empty(len(s2u), dtype=dtype, device="cuda")
    P.mesh_fill_random(m, lattice, 31, x)
    xu = np.zeros(om.n)
    xu[s2u] = x.cpu().numpy()
    y = torch.full_like(x, float("nan"))
    if kind == "p2":
        P.apply_p2(m, L, x, y)
        A = om.csr_p2(dirichlet=dirichlet)
    elif kind == "varcoef":
        k = torch.empty_like(x)
        P.mesh_fill_random(m, L, 32, k)
        k += 1.5
        P.apply_varcoef(m, L, k, x, y)
        ku = np.zeros(om.n)
        ku[s2u] = k.cpu().numpy()
        A = om.csr_varcoef(ku, dirichlet=dirichlet)
    else:
        d = np.random.default_rng(L).uniform(-0.02, 0.02, (len(ce), 2))
        P.apply_blended(m, L, torch.as_tensor(d, device="cuda"), x, y)
        A = om.csr_blended(d, dirichlet=dirichlet)
    got, want = y.cpu().numpy(), (A @ xu)[s2u]
    assert np.isfinite(got).all() and harness.copies_consistent(got, s2u)
    assert harness.rel_err_max(got.astype(np.float64), want) <= (1e-12 if dtype == torch.float64 else 1e-5)
