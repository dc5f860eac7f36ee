"""PCG's fused steps (scalar products from the operator's, the patch solves' and
the coarse solve's own kernels, gathers inside the updates) at the sizes where
their dispatch changes: up to and beyond 512 partial sums (summed by the
consuming kernels, or by a launch of their own), several elements per workgroup,
every preconditioner part, constant and per-element coefficients, checks every
few iterations, and solves cut off by the iteration cap; against the oracle's
PCG, which takes the same steps with assembled vectors."""
import numpy as np
import pytest

import meshgen
from oracle.problem import Problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("pc", [0, 1, 2, 3])
@pytest.mark.parametrize("k,N,coef", [((2, 3, 2), 4, None), ((4, 3, 3), 3, "const"), ((9, 8, 8), 2, None),
                                      ((9, 9, 8), 3, "element")])
def test_pcg_steps(k, N, coef, pc):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[pcg steps] k={k} N={N} coef={coef} pc={pc}", flush=True)
    m = meshgen.cube_mesh(k, perturb=0.1, seed=sum(k) + N)
    m, _ = meshgen.rotate_elements(m, seed=3)
    M = sem.Mesh(m.vtx, m.hex, N)
    rng = np.random.default_rng(N)
    kw = {}
    if coef == "const":
        kw = dict(kappa=0.3, c=7.0)
        M.set_coefficients(**kw)
    elif coef == "element":
        kw = dict(kappa=rng.uniform(0.5, 2.0, m.n_elem), c=rng.uniform(0.0, 3.0, m.n_elem))
        M.set_element_coefficients(**kw)
    P = Problem(m.vtx, m.hex, N, **kw)
    b = rng.uniform(-1.0, 1.0, M.n_global) * (P.dirichlet == 0)
    bt = torch.tensor(b, device="cuda:0")
    fine, coarse = bool(pc & 1), bool(pc & 2)
    if pc == 2:
        # the coarse space alone is singular as a preconditioner: a few steps of the recurrence, not a solve
        x, info = M.solve(bt, pc=pc, rtol=1e-12, max_iter=4, raise_on_noconv=False)
        ref, it, _, _ = P.solve(b, rtol=1e-12, max_iter=4, fine=fine, coarse=coarse)
        assert info["iterations"] == it == 4
        assert rel(x.cpu().numpy(), ref) <= 1e-10
        return
    ref, it, _, _ = P.solve(b, rtol=1e-10, fine=fine, coarse=coarse)
    for check_every in (1, 3):
        x, info = M.solve(bt, pc=pc, rtol=1e-10, check_every=check_every)
        # rounding may move the stop by one iteration; a check every 3 looks up to 2 later
        assert it - 1 <= info["iterations"] <= it + check_every
        # both residuals are below 1e-10 |b|: the solutions differ by that times the condition number, < 1e4 here
        assert rel(x.cpu().numpy(), ref) <= 1e-6
        assert info["rel_residual"] <= 1e-10
    cut = max(2, it // 2)
    ref, _, _, _ = P.solve(b, rtol=1e-10, max_iter=cut, fine=fine, coarse=coarse)
    x, info = M.solve(bt, pc=pc, rtol=1e-10, max_iter=cut, raise_on_noconv=False)
    assert info["status"] == sem.SEM_ENOCONV and info["iterations"] == cut
    assert rel(x.cpu().numpy(), ref) <= 1e-8  # the same iterate, rounding amplified over the steps
    M.close()
