"""Batched solves with one order (no parallel branches), two and four orders, and
instance sizes around the reduction chunk, against single solves of the same
handles' meshes: both meet 1e-10 in the true residual, so the solutions differ by
at most about 2e-10 times the condition number's share, 1e-8 here."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# (k, N): (4 * 4 + 1)^3 = 4913 nodes, (3 * 5 + 1)^3 = 4096, one free vertex at k = 2
@pytest.mark.parametrize("mode", ["SOLVE_FP64", "SOLVE_FP32_REFINED"])
@pytest.mark.parametrize("sizes", [[(3, 5)], [(4, 4), (2, 4), (5, 4)], [(2, 2), (6, 3)], [(3, 3), (2, 9), (4, 5), (3, 3), (2, 7)]])
def test_batch_orders(sizes, mode):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    mode = getattr(sem, mode)
    print(f"[batch orders] {sizes} mode {mode}", flush=True)
    meshes = [meshgen.cube_mesh(k, perturb=0.1, seed=40 + i) for i, (k, _) in enumerate(sizes)]
    B = sem.Batch([(m.vtx, m.hex, N) for m, (_, N) in zip(meshes, sizes)])
    rng = np.random.default_rng(17)
    bs = [torch.tensor(rng.uniform(-1.0, 1.0, n), device="cuda:0") for n in B.n_global]
    for rep in range(3):  # the captured iteration replayed, other right-hand sides each time
        bs = [b.flip(0).contiguous() for b in bs]
        xs, infos, _ = B.solve(bs, mode=mode, rtol=1e-10)
        for m, (_, N), b, x, info in zip(meshes, sizes, bs, xs, infos):
            M = sem.Mesh(m.vtx, m.hex, N)
            ref, single = M.solve(b, mode=mode, rtol=1e-10)
            assert info["rel_residual"] <= 1e-10
            assert abs(info["iterations"] - single["iterations"]) <= (1 if mode == sem.SOLVE_FP64 else 8)
            assert float(torch.linalg.norm(x - ref)) <= 1e-8 * float(torch.linalg.norm(ref))
            M.close()
    B.close()
