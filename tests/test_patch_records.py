"""Every mesh that the patch tables take has affine patch records (the form that
orders from 5 on read on the device): boxes with turned and shuffled elements, single
layers, and irregular meshes whose edges and vertices have other valences than
4 and 8, where parts of the patches are NULL."""
import launch_probe
import pytest

import meshgen


def meshes():
    for k in ((1, 1, 1), (2, 1, 1), (3, 3, 1), (3, 4, 3)):
        box = meshgen.cube_mesh(k, perturb=0.1, seed=sum(k))
        yield box
        turned, _ = meshgen.rotate_elements(box, seed=3)
        yield meshgen.permute_elements(turned, seed=4)[0]
    for m in (3, 4, 5, 6):
        for layers in (1, 3):
            turned, _ = meshgen.rotate_elements(meshgen.star_mesh(m, layers), seed=m)
            yield turned


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    return launch_probe.build(str(tmp_path_factory.mktemp("probe")))


@pytest.mark.parametrize("N", [5, 6, 7, 8, 15])
def test_records_exist(probe, N):
    for mesh in meshes():
        assert launch_probe.has_patch_records(probe, mesh, N)
