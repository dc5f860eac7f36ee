"""Every order applies the operator without the autotuner, in both precisions,
against the oracle (FP64 1e-12, FP32 5e-6: the bounds of the operator tests)."""
import numpy as np
import pytest

import meshgen
from oracle.problem import Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N", range(2, 16))
def test_default_tile(N):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = meshgen.cube_mesh((3, 2, 1) if N > 8 else (3, 2, 2), perturb=0.1, seed=N)
    M, P = sem.Mesh(m.vtx, m.hex, N, autotune=False), Problem(m.vtx, m.hex, N)
    u = np.random.default_rng(N).uniform(-1.0, 1.0, M.n_global)
    want = P.A(u)
    for dtype, tol in ((torch.float64, 1e-12), (torch.float32, 5e-6)):
        y = M.apply_A(torch.tensor(u, device="cuda:0", dtype=dtype)).double().cpu().numpy()
        assert np.linalg.norm(y - want) <= tol * np.linalg.norm(want)
    M.close()
