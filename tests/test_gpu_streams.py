"""The calls under stream capture, and handles used at the same time by several
threads on streams of their own: the same results, bit for bit, as one after
another on the default stream."""
import threading

import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def handle(k, N, seed, **kw):
    from paper_1506_05996_amd import sem
    m = meshgen.cube_mesh(k, lengths=tuple(float(v) for v in k), perturb=0.1, seed=seed)
    return sem.Mesh(m.vtx, m.hex, N, autotune=False, **kw)


def residual(M, seed, dtype=torch.float64):
    v = np.random.default_rng(seed).uniform(-1.0, 1.0, M.n_global) * (M.boundary_mask() == 0)
    return torch.tensor(v, device="cuda:0", dtype=dtype)


# one coarse front, several heights; patch tables and patch records
@pytest.mark.parametrize("dtype", ["float64", "float32"])
@pytest.mark.parametrize("k,N", [((5, 4, 3), 4), ((5, 4, 3), 7), ((17, 16, 15), 2)])
def test_captured_calls(k, N, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[capture] k={k} N={N} {dtype}", flush=True)
    M = handle(k, N, 3)
    r = residual(M, 1, getattr(torch, dtype))
    R = torch.rand(M.n_vertices, device="cuda:0", dtype=torch.float64)
    y, z, Z = torch.empty_like(r), torch.empty_like(r), torch.empty_like(R)

    def calls():
        M.apply_A(r, y)
        M.precond(y, z)
        M.coarse_solve(R, Z)

    calls()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    for rep in range(4):  # other inputs in the same buffers, the program's own work between the replays
        r.copy_(residual(M, 10 + rep, getattr(torch, dtype)))
        R.copy_(torch.rand_like(R))
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (y, z, Z)]
        calls()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, (y, z, Z)))
    M.close()


def test_threads_and_streams():
    from paper_1506_05996_amd import sem
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    work = [((5, 4, 3), 4, sem.SOLVE_FP64, False), ((6, 6, 5), 5, sem.SOLVE_FP32_REFINED, False),
            ((17, 16, 15), 2, sem.SOLVE_FP64, False), ((6, 5, 5), 7, sem.SOLVE_FP64, True)]
    handles, want = [], []
    for i, (k, N, mode, amg) in enumerate(work):
        M = handle(k, N, i)
        if amg:
            M.set_coarse_solver(sem.COARSE_AMG)
        b = residual(M, i)
        handles.append((M, b, mode))
        want.append(M.solve(b, mode=mode, rtol=1e-10)[0].clone())
    torch.cuda.synchronize()
    got = [None] * len(work)

    def loop(i):
        M, b, mode = handles[i]
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            xs = [M.solve(b, mode=mode, rtol=1e-10)[0] for _ in range(5)]
            s.synchronize()
        got[i] = xs

    threads = [threading.Thread(target=loop, args=(i,)) for i in range(len(work))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for (M, _, _), xs, ref in zip(handles, got, want):
        assert xs is not None and all(torch.equal(x, ref) for x in xs)
        M.close()
