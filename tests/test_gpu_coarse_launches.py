"""The exact coarse solve on meshes that between them take every instance of the
sweep kernels that the dispatch can choose (test_launch_shapes.py holds the list
to that): rows of up to 128 entries by 1, 2, 4 and 8 per wave and longer ones by 1, 2
and 4, forward and backward, over two to four heights, against known solutions of
systems with the oracle's coarse matrix."""
import numpy as np
import pytest

import meshgen
from oracle.coarse import coarse_matrix

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MESHES = [(2, 2, 4000), (3, 3, 1200), (3, 100, 100), (2, 150, 150), (10, 10, 125), (24, 24, 24), (32, 32, 32)]


def mesh_of(k):
    return meshgen.cube_mesh(k, lengths=tuple(float(v) for v in k), perturb=0.1, seed=sum(k))


@pytest.mark.parametrize("k", MESHES)
def test_coarse_solve_launches(k):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[coarse launches] k={k}", flush=True)
    m = mesh_of(k)
    M = sem.Mesh(m.vtx, m.hex, 2, autotune=False)
    free = np.nonzero(M.boundary_mask()[:M.n_vertices] == 0)[0]
    A = coarse_matrix(m.vtx, m.hex, M.n_vertices)[free][:, free]
    rng = np.random.default_rng(sum(k))
    for rep in range(2):  # a second right-hand side on the same handle
        ref, R = np.zeros((2, M.n_vertices))
        ref[free] = rng.uniform(-1.0, 1.0, len(free))
        R[free] = A @ ref[free]
        Z = M.coarse_solve(torch.tensor(R, device="cuda:0")).cpu().numpy()
        # backward stable, and R is A ref to rounding: about eps cond(A), below 2e-16 * 1e4 on these boxes
        assert np.linalg.norm(Z - ref) <= 1e-11 * np.linalg.norm(ref)
        assert not Z[np.setdiff1d(np.arange(M.n_vertices), free)].any()
    M.close()
