"""Images of the float16 and bfloat16 modes, bit for bit.  Rounding the MLP's
operands to 16 bits turns a change in the last bit of a colour or feature into
up to a thousandth of a pixel, so a kernel that rounds its sums in another way
shows here and hardly anywhere else.

golden/reduced_precision.npz holds images that an MI355X gave in these modes
when every mode took the sigmoid of Eq. 8's plain result (the fp32 mode now
folds the two scales).  Equal roundings give equal bits: the tolerance is
zero."""
import os

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

GOLD = os.path.join(os.path.dirname(__file__), "golden", "reduced_precision.npz")
CASES = {"bf16": {"mlp_prec": "bf16"}, "bf16_fine": {"mlp_prec": "bf16", "step": 2.0 / 256},
         "f16": {"mlp_prec": "f16"}, "f16_interp": {"mlp_prec": "f16", "feat_prec": "f16_interp"},
         "bf16_f16": {"mlp_prec": "bf16", "feat_prec": "f16", "delta_mode": 1}}


def cameras():
    """One view from inside the cube and one from outside."""
    return synth.concat_cameras([synth.full_camera(seed=5, w=40, h=30), synth.tiny_camera(seed=6, w=40, h=30)])


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.fixture(scope="module")
def merf():
    from paper_2302_12249_amd import merf as m
    m.load()
    return m


@pytest.mark.parametrize("case", sorted(CASES))
def test_reduced_precision_images_keep_their_bits(torch, merf, tiny_scene, case):
    with np.load(GOLD, allow_pickle=False) as z:
        want = z[case]
    r = merf.Renderer(tiny_scene)
    got = r.render(cameras(), **CASES[case]).cpu().numpy()
    r.close()
    print(f"{case}: {np.mean((got != want).any(1)):.2%} of pixels differ, max {np.abs(got - want).max():.3e}", flush=True)
    assert np.array_equal(got, want)


def test_tile_orders_agree_beyond_65536_tiles(torch, merf, tiny_scene):
    """129600 tiles: the ordering prepass counts no samples there."""
    cams = synth.full_camera(seed=5, w=3840, h=2160)
    r = merf.Renderer(tiny_scene)
    a = r.render(cams, mlp_prec="bf16", step=2.0 / 256)
    b = r.render(cams, mlp_prec="bf16", step=2.0 / 256, order="plain")
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    r.close()
