"""The meshes of the GPU tests reach the launch shapes they are there for: every
instance of the coarse sweeps, and counts of partial sums on both sides of 512."""
import launch_probe
import pytest
import test_gpu_coarse_launches as launches
import test_gpu_pcg_limits as limits


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    return launch_probe.build(str(tmp_path_factory.mktemp("probe")))


def test_every_sweep_instance_is_run(probe):
    seen, heights = set(), set()
    for k in launches.MESHES:
        shapes = launch_probe.coarse_launches(probe, launches.mesh_of(k))
        seen |= {(forward, rw, wide) for forward, rw, wide, _ in shapes}
        heights.add(sum(forward for forward, _, _, _ in shapes))
    for forward in (0, 1):
        assert {rw for f, rw, wide in seen if f == forward and not wide} == {1, 2, 4, 8}
        assert {rw for f, rw, wide in seen if f == forward and wide} == {1, 2, 4}
    assert {2, 3, 4} <= heights


def test_partial_sums_on_both_sides_of_the_limit(probe):
    pAp, rz, heights = [], [], []
    for k, N, tile, pc in limits.CASES:
        E = k[0] * k[1] * k[2]
        shapes = launch_probe.coarse_launches(probe, limits.mesh_of(k))
        pAp.append(launch_probe.grid(E, tile or probe.packing(N, 0)))
        rz.append((launch_probe.grid(E, probe.packing(N, 1)) if pc & 1 else 0)
                  + (sum(n for forward, _, _, n in shapes if forward) if pc & 2 else 0))
        heights.append(sum(forward for forward, _, _, _ in shapes))
    assert pAp[:4] == [512, 520, 80, 80] and rz[2:4] == [512, 520]
    assert max(rz[:2]) <= 512 < min(pAp[4:]) and rz[5] <= 512 < rz[4]
    assert heights[4] == heights[5] == 2
