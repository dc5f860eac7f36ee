"""The exact coarse solve on meshes whose dissection forest is merged in
different ways (one dense front, several heights, rows of fewer and of more than
128 entries, odd row lengths, more than one staging chunk, several rows per
wave), against a sparse direct factorisation of the oracle's coarse matrix."""
import numpy as np
import pytest
import scipy.sparse.linalg

import meshgen
from oracle.coarse import coarse_matrix

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [(2, 2, 2), (3, 2, 2), (4, 4, 4), (6, 6, 6), (6, 6, 7), (9, 8, 7), (12, 12, 12),
                               (17, 16, 15), (20, 19, 22), (5, 6, 70)])
def test_coarse_solve_merged_heights(k):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = meshgen.cube_mesh(k, lengths=tuple(float(v) for v in k), perturb=0.1, seed=sum(k))
    m, _ = meshgen.permute_elements(m, seed=1 + sum(k))
    M = sem.Mesh(m.vtx, m.hex, 2, autotune=False)
    free = np.nonzero(M.boundary_mask()[:M.n_vertices] == 0)[0]
    A = coarse_matrix(m.vtx, m.hex, M.n_vertices)[free][:, free].tocsc()
    lu = scipy.sparse.linalg.splu(A)
    rng = np.random.default_rng(sum(k))
    for rep in range(2):  # a second right-hand side on the same handle
        R = rng.uniform(-1.0, 1.0, M.n_vertices)
        ref = np.zeros(M.n_vertices)
        ref[free] = lu.solve(R[free])
        Z = M.coarse_solve(torch.tensor(R, device="cuda:0")).cpu().numpy()
        # both sides are backward stable: about eps cond(A), below 2e-16 * 1e4 on these boxes
        assert np.linalg.norm(Z - ref) <= 1e-11 * np.linalg.norm(ref)
        assert (Z[np.setdiff1d(np.arange(M.n_vertices), free)] == 0.0).all()
