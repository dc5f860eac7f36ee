"""PCG under very large and very small kappa, whose iterates u and unscaled
products A_1 u multiply to numbers outside the FP64 range: the solution is that of
kappa = 1 over kappa.  Both meet 1e-10 in the true residual and their steps differ by
rounding alone, so they agree to 1e-10 times the condition number, < 1e4 here."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("pc", [0, 1, 3])
@pytest.mark.parametrize("kappa", [1e200, 1e-200])
@pytest.mark.parametrize("k,N", [((3, 3, 2), 5), ((2, 2, 2), 15)])  # line-phase and, by set_tile, every other operator
def test_pcg_kappa_scale(k, N, kappa, pc):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[pcg scale] k={k} N={N} kappa={kappa} pc={pc}", flush=True)
    m = meshgen.cube_mesh(k, perturb=0.1, seed=N)
    M = sem.Mesh(m.vtx, m.hex, N, autotune=False)
    rng = np.random.default_rng(N)
    b = torch.tensor(rng.uniform(-1.0, 1.0, M.n_global) * M.lumped_mass(), device="cuda:0")
    ref, one = M.solve(b, pc=pc, rtol=1e-10, max_iter=3000)
    M.set_coefficients(kappa, 0.0)
    for tile in (sem.TILE_LINE_GEO, sem.TILE_LINE, 1) + ((sem.TILE_MFMA,) if N == 15 else ()):
        M.set_tile(tile)
        x, info = M.solve(b, pc=pc, rtol=1e-10, max_iter=3000)
        assert abs(info["iterations"] - one["iterations"]) <= 2 + one["iterations"] // 50
        assert float(torch.linalg.norm(x * kappa - ref)) <= 1e-6 * float(torch.linalg.norm(ref))
    M.close()


@pytest.mark.parametrize("pc", [1, 3])
@pytest.mark.parametrize("length,scale", [(1e-20, 1e-140), (1e20, 1e140), (1e-12, 1e-140)])
@pytest.mark.parametrize("k,N", [((4, 3, 3), 3), ((3, 3, 2), 7)])
def test_pcg_box_and_load_scale(k, N, length, scale, pc):
    """Very small and very large boxes under very small and very large loads: A grows with the
    length, so the solution is the unit box's times scale / length.  Same bounds as above."""
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[pcg scale] k={k} N={N} length={length} scale={scale} pc={pc}", flush=True)
    b, ref, one = None, None, None
    for lx, f in ((1.0, 1.0), (length, scale)):
        m = meshgen.cube_mesh(k, lengths=(lx, lx, lx), perturb=0.1, seed=N)
        M = sem.Mesh(m.vtx, m.hex, N, autotune=False)
        if b is None:
            b = np.random.default_rng(N).uniform(-1.0, 1.0, M.n_global) * (M.boundary_mask() == 0)
        x, info = M.solve(torch.tensor(b * f, device="cuda:0"), pc=pc, rtol=1e-10)
        M.close()
        if ref is None:
            ref, one = x, info
            continue
        assert abs(info["iterations"] - one["iterations"]) <= 2
        assert float(torch.linalg.norm(x * (length / scale) - ref)) <= 1e-6 * float(torch.linalg.norm(ref))
