"""Small launches divide each tile over up to eight waves.  Their images must be
bit for bit those of one wave a tile (the measuring variants never divide) at
every number of waves a tile, on both sides of each limit, with tiles cut by the
image's edge, several cameras in a launch, and every precision and skip mode."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def merf():
    from paper_2302_12249_amd import merf as m
    m.load()
    return m


@pytest.fixture(scope="module")
def renderer(merf):
    r = merf.Renderer(synth.make_scene(64, 128, 0.3, 1.99, 0.1, 0.4, seed=61))
    yield r
    r.close()


def both(torch, merf, renderer, cams, **params):
    """The image, and the image of the measuring variant."""
    n = cams.num_pixels()
    a = torch.full((n, 4), -1.0, device="cuda")
    b = torch.full((n, 4), -2.0, device="cuda")
    renderer.render(cams, out=a, **params)
    merf.render_phases(renderer.handle, cams, b, **params)
    torch.cuda.synchronize()
    return a.cpu().numpy(), b.cpu().numpy()


# tiles 1, 2, 256, 257, 384 | 385, 512, 513, 768 | 769, 1024, 1025, 1536 | 1537
@pytest.mark.parametrize("w,h", [(1, 1), (9, 7), (128, 128), (2056, 8), (3072, 8), (3080, 8), (125, 255), (4104, 8),
                                 (255, 190), (6152, 8), (255, 249), (1639, 35), (383, 255), (231, 423)])
def test_divided_tiles_give_the_same_image(torch, merf, renderer, w, h):
    a, b = both(torch, merf, renderer, synth.orbit_cameras(1, w=w, h=h))
    assert np.array_equal(a, b)
    if w * h > 1000:
        assert a[:, 3].max() > 0.0                 # something was hit


@pytest.mark.parametrize("mlp", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("feat", ["f32", "f16", "f16_interp"])
@pytest.mark.parametrize("skip", ["distance", "levels"])
def test_divided_tiles_in_every_variant(torch, merf, renderer, mlp, feat, skip):
    cams = synth.orbit_cameras(3, w=77, h=61)      # 240 tiles of three cameras
    a, b = both(torch, merf, renderer, cams, mlp_prec=mlp, feat_prec=feat, skip=skip)
    assert np.array_equal(a, b)
