"""sem_pcg_solve_noalloc where the partial sums are many against the nodes (single
elements and rows of them at N = 2, free vertices everywhere), with either coarse
solver: the same solutions, bit for bit, as sem_pcg_solve."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode", ["SOLVE_FP64", "SOLVE_FP32_REFINED"])
@pytest.mark.parametrize("amg", [False, True])
@pytest.mark.parametrize("k", [(1, 1, 1), (3, 1, 1), (9, 1, 1), (17, 1, 1), (7, 6, 5)])
def test_noalloc_small(k, amg, mode):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[noalloc small] k={k} amg={amg} mode={mode}", flush=True)
    m = meshgen.cube_mesh(k, perturb=0.1, seed=sum(k))
    M = sem.Mesh(m.vtx, m.hex, 2)
    M.set_coefficients(1.0, 2.0)
    M.set_dirichlet(np.zeros(M.n_global))
    if amg:
        M.set_coarse_solver(sem.COARSE_AMG)
    b = torch.tensor(np.random.default_rng(len(m.hex)).uniform(-1.0, 1.0, M.n_global), device="cuda:0")
    kw = dict(mode=getattr(sem, mode), rtol=1e-10)
    for rep in range(2):
        x, info = M.solve(b, noalloc=True, **kw)
        ref, one = M.solve(b, **kw)
        assert info["iterations"] == one["iterations"] and info["rel_residual"] <= 1e-10
        assert torch.equal(x, ref)
    M.close()
