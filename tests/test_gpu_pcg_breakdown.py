"""A breakdown inside the fused PCG iteration: r . z beyond the FP64 range, so
that beta is not finite behind a finite alpha.  Patch solves alone on a smooth
load let r . z grow over the first steps; the load is scaled so that it passes
the largest FP64 number at a chosen step.  The solve reports the breakdown and x
is, bit for bit, what the steps before it left."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# up to and beyond 512 partial sums of r . z (beta from the kernel that uses it, or from a launch of its
# own), workgroups of several waves (N = 5, 6, 8: 252, 245 and 243 lanes)
@pytest.mark.parametrize("check_every", [1, 2])
@pytest.mark.parametrize("k,N,step", [((4, 4, 4), 5, 1), ((3, 3, 3), 6, 1), ((4, 4, 3), 8, 1), ((9, 8, 7), 9, 2),
                                      ((9, 9, 8), 5, 1), ((9, 9, 8), 8, 1)])
def test_beta_beyond_fp64(k, N, step, check_every):
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[breakdown] k={k} N={N} step={step} check_every={check_every}", flush=True)
    m = meshgen.cube_mesh(k, perturb=0.1, seed=3)
    M = sem.Mesh(m.vtx, m.hex, N)
    dev = torch.device("cuda:0")
    s = np.prod(np.sin(np.pi * M.node_coords()), axis=1)
    b = torch.tensor(s * M.lumped_mass() * (M.boundary_mask() == 0), device=dev)
    b /= torch.linalg.norm(b)
    # r . z and p . A p of the first steps, unscaled
    r, z = b.clone(), M.precond(b, pc=sem.PC_FINE)
    p, rz, pAp = z.clone(), [float(torch.dot(b, z))], []
    for _ in range(step):
        w = M.apply_A(p)
        pAp.append(float(torch.dot(p, w)))
        r = r - rz[-1] / pAp[-1] * w
        z = M.precond(r, pc=sem.PC_FINE)
        rz.append(float(torch.dot(r, z)))
        p = z + rz[-1] / rz[-2] * p
    top = np.finfo(np.float64).max
    before = max(rz[:-1] + pAp)
    assert rz[-1] > 1.3 * before  # room for the scale
    f = np.sqrt(top / np.sqrt(rz[-1] * before))
    b = b * f
    x0 = torch.tensor(np.random.default_rng(N).uniform(-1e-40, 1e-40, M.n_global), device=dev) * f
    x0 = x0 * torch.tensor(M.boundary_mask() == 0, device=dev)
    ref = x0.clone()
    if step > 1:
        _, info = M.solve(b, x=ref, use_x0=True, pc=sem.PC_FINE, rtol=1e-10, max_iter=step - 1, raise_on_noconv=False)
        assert info["iterations"] == step - 1 and not torch.equal(ref, x0)
    x = x0.clone()
    with pytest.raises(sem.SemError) as e:
        M.solve(b, x=x, use_x0=True, pc=sem.PC_FINE, rtol=1e-10, check_every=check_every)
    assert e.value.status == sem.SEM_EBREAKDOWN
    assert torch.equal(x, ref)
    M.close()
