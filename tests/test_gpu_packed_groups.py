"""Kernels with several elements per workgroup (orders 2..6 and 8) on element
counts around their packing, against the oracle: FP64 to 1e-12, FP32 to 5e-6 (the
bounds of the operator and preconditioner tests)."""
import numpy as np
import pytest

import meshgen
from oracle.problem import Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("k", [(1, 1, 1), (3, 1, 1), (2, 2, 2), (5, 3, 1), (3, 3, 3)])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 6, 8])
def test_packed_workgroups(N, k):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[packed] N={N} k={k}", flush=True)
    m = meshgen.cube_mesh(k, perturb=0.1, seed=N)
    m, _ = meshgen.rotate_elements(m, seed=2)
    M, P = sem.Mesh(m.vtx, m.hex, N), Problem(m.vtx, m.hex, N)
    rng = np.random.default_rng(5)
    u = rng.uniform(-1.0, 1.0, M.n_global)
    r = u * (P.dirichlet == 0)
    Au, Pr = P.A(u), P.precond()(r)
    for dtype, code, tol in ((torch.float64, sem.SEM_F64, 1e-12), (torch.float32, sem.SEM_F32, 5e-6)):
        for tile in (sem.TILE_LINE_GEO, sem.TILE_LINE):
            M.set_tile(tile, code)
            y = M.apply_A(torch.tensor(u, device="cuda:0", dtype=dtype)).double().cpu().numpy()
            assert rel(y, Au) <= tol if np.any(Au) else not np.any(y)
        z = M.precond(torch.tensor(r, device="cuda:0", dtype=dtype)).double().cpu().numpy()
        assert rel(z, Pr) <= tol if np.any(Pr) else not np.any(z)
    M.close()
