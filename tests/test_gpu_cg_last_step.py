"""CG adds a step to x in the next iteration's direction pass, so a solve or a
batch member that ends without one (max_iter) must still have its last step:
the residual of the returned x is the recurrence's, which agrees with the
oracle's within 1e-8 of |b| after a few iterations (FP64 vectors; rounding of
a few dozen operations on values up to 1e3 |b|)."""
import numpy as np
import pytest

import harness
import paper_2305_15116_amd as P
from oracle.oracle import OracleMesh
from paper_2305_15116_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("mode", [2, 3])
@pytest.mark.parametrize("dim,L,max_iter", [(2, 6, 1), (2, 6, 4), (3, 4, 1), (3, 4, 3)])
def test_x_has_every_step(dim, L, max_iter, mode, batched):
    co, ce = (W.strip_2d if dim == 2 else W.strip_3d)(3)
    m = P.create_macro_mesh(co, ce, L)
    om = OracleMesh(co, ce, L)
    s2u = harness.storage_to_unique(P.mesh_dof_keys(m, L), om.keys())
    b = torch.empty(len(s2u), dtype=torch.float64, device="cuda")
    P.mesh_fill_random(m, L, 33, b)
    x = torch.zeros_like(b)
    ws = torch.empty(P.mesh_workspace_bytes(m, L, mode), dtype=torch.uint8, device="cuda")
    if batched:
        B = P.batch_create(1, mode=mode, max_iter=max_iter)
        P.batch_add(B, m, L, b, x, ws, 0.0, 7)
        done = []
        while not done:
            done = P.batch_step(B)
        assert done[0][1] == P.MF_NOT_CONVERGED and done[0][2] == max_iter
        rel = done[0][3]
    else:
        rc, it, rel, _ = P.vcycle_solve(m, L, b, x, ws, mode=mode, rtol=0.0, max_iter=max_iter)
        assert rc == P.MF_NOT_CONVERGED and it == max_iter
    torch.cuda.synchronize()
    bu, xu = np.zeros(om.n), np.zeros(om.n)
    bu[s2u], xu[s2u] = b.cpu().numpy(), x.cpu().numpy()
    assert harness.copies_consistent(x.cpu().numpy(), s2u)
    res = np.linalg.norm(bu - om.spmv(xu)) / np.linalg.norm(bu)
    assert abs(res - rel) <= 1e-8, (res, rel)
