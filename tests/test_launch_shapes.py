"""The meshes of the GPU tests reach the launch shapes they are there for: every
instance of the coarse sweeps."""
import launch_probe
import pytest
import test_gpu_coarse_launches as launches


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
