"""The octant grids built one after another, which take less scratch, against
the eight built together: the same bytes, and the same images of a scene
uploaded that way.  A budget without room for the larger scratch selects the
smaller form."""
import numpy as np
import pytest

import synth
from gpu_helpers import gpu_render

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture()
def merf():
    from paper_2302_12249_amd import merf as m
    m.load()
    yield m
    m.set_hbm_budget(2 ** 63)


@pytest.mark.parametrize("r,pools", [(1, (1,)), (5, (1,)), (16, (4, 1)), (30, (2, 1)), (64, (8, 2, 1)), (100, (1,)),
                                     (130, (2, 1)), (256, (8, 2, 1))])
@pytest.mark.parametrize("density", [0.0, 0.001, 0.1])
def test_octant_forms_agree(torch, merf, r, pools, density):
    rng = np.random.default_rng(r)
    occ = (rng.random((r, r, r)) < density).astype(np.uint8)
    levels = [torch.from_numpy(synth.maxpool(occ, p) if p > 1 else occ).cuda() for p in pools]
    want = merf.distance_grid(levels, octants=True)
    merf.set_hbm_budget(merf.hbm_in_use() + r ** 3)
    got = merf.distance_grid(levels, octants=True)
    assert torch.equal(got, want)


def test_upload_with_little_room_renders_the_same(torch, merf, tiny_scene, tiny_cams):
    want = gpu_render(torch, merf, tiny_scene, tiny_cams)
    r = merf.Renderer(tiny_scene)
    need = merf.scene_bytes(r.handle)
    r.close()
    merf.set_hbm_budget(merf.hbm_in_use() + need)
    assert np.array_equal(gpu_render(torch, merf, tiny_scene, tiny_cams), want)
