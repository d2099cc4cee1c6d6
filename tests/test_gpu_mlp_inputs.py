"""The fp32 deferred MLP on colours and features that are not zero, from 1e-5 to
1, against float64 on the very inputs the kernel has: they are read back
through MLPs that copy one input each to an output, times 2^60 (weights of such
sizes take the float32 matrix instructions, which multiply by powers of two and
add zeros exactly, and the colour added last is below half a step of the
result).  The direction's rows are zero, so the sines' own error is not in it.

Bound: a layer's operands may be off by 2^-23 each (a pair of float16 values
holds 23 bits) and every one of its at most 160 products and sums may round to
2^-24, relative to the layer's sum of magnitudes; three layers, and the last
sum with the colour."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from scene_builders import dense_scene

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


CAMS = synth.full_camera(seed=3, w=61, h=40)


def _pack(W0, W1, W2):
    z = np.zeros
    return np.concatenate([W0.ravel(), z(16), W1.ravel(), z(16), W2.ravel(), z(3)]).astype(np.float32)


def _rgb(torch, merf, scene, mlp):
    r = merf.Renderer(dataclasses.replace(scene, mlp=mlp))
    out = r.render(CAMS).cpu().numpy().astype(np.float64)
    r.close()
    return out[:, :3]


def _inputs(torch, merf, scene):
    x = []
    for first in (0, 3, 6):
        W0, W1, W2 = np.zeros((34, 16)), np.zeros((16, 16)), np.zeros((16, 3))
        for i in range(3):
            W0[min(first + i, 6), i], W1[i, i], W2[i, i] = 2.0 ** 60, 1.0, 1.0
        x.append(_rgb(torch, merf, scene, _pack(W0, W1, W2)) * 2.0 ** -60)
    return np.concatenate(x, 1)[:, :7]


@pytest.fixture(scope="module", params=["1e-5", "1e-3", "1e-1", "1"])
def lit(request, torch, merf):
    """A scene whose colours and features are of that size, and their values."""
    lo, hi = {"1e-5": (92, 108), "1e-3": (102, 119), "1e-1": (112, 132), "1": (140, 160)}[request.param]
    sc = dense_scene(L=32, R=64, seed=4)
    rng = np.random.default_rng(4)
    sc.blocks[..., 0] = rng.integers(lo, hi, sc.blocks.shape[:-1])
    sc.planes[..., 0] = rng.integers(lo, hi, sc.planes.shape[:-1])
    x = _inputs(torch, merf, sc)
    assert float(request.param) / 10 < np.median(x) < 10 * float(request.param) and np.all(x >= 0)
    cd = _rgb(torch, merf, sc, np.zeros(synth.mlp_param_count(), np.float32))
    assert np.array_equal(cd, x[:, :3])               # (h = 0: the image is the colour)
    return request.param, sc, x


@pytest.mark.parametrize("scale", [0.1, 1.0, 100.0])
@pytest.mark.parametrize("rows", ["all", "one large"])
def test_mlp_of_colours_and_features(torch, merf, lit, scale, rows):
    size, sc, x = lit
    rng = np.random.default_rng(7)
    W0, W1, W2 = np.zeros((34, 16)), rng.normal(size=(16, 16)), rng.normal(size=(16, 3))
    W0[:7] = scale * rng.normal(size=(7, 16))
    if rows == "one large":                           # one input's weights a thousand times the others'
        W0[:7] *= 1e-3
        W0[5] *= 1e3
    w = [np.float32(a).astype(np.float64) for a in (W0, W1, W2)]
    y = np.maximum(np.maximum(x @ w[0][:7], 0.0) @ w[1], 0.0) @ w[2] + x[:, :3]
    top = x @ np.abs(w[0][:7]) @ np.abs(w[1]) @ np.abs(w[2])
    bound = 3 * (2 * 2.0 ** -23 + 160 * 2.0 ** -24) * top + 2.0 ** -24 * np.abs(y)
    # the same function by the float32 instructions: scales that only they take
    exact = _pack(W0.astype(np.float32) * np.float32(2.0 ** 60), W1.astype(np.float32) * np.float32(2.0 ** -60), W2)
    for name, mlp in (("float32 instructions", exact), ("default", _pack(W0, W1, W2))):
        err = np.abs(_rgb(torch, merf, sc, mlp) - y)
        print(f"inputs {size} weights {scale} {rows}, {name}: max err {np.max(err[x.all(1)] / top[x.all(1)]):.2e} of the sums of magnitudes, "
              f"norm {np.linalg.norm(err) / np.linalg.norm(y):.2e}", flush=True)
        assert np.all(err <= bound)


def _direction():
    w, h = (int(v) for v in CAMS.size[0])
    r, c = np.divmod(np.arange(w * h), w)
    _, d = oracle.camera_rays(CAMS, 0, r, c)
    return np.concatenate([d] + [np.sin(2.0 ** k * d) for k in range(4)] + [np.cos(2.0 ** k * d) for k in range(4)], 1)


@pytest.mark.parametrize("scale", [0.1, 1.0, 100.0])
@pytest.mark.parametrize("direction", [True, False])
def test_mlp_error_next_to_float32_instructions(torch, merf, lit, scale, direction):
    """2-norm of the error, six MLPs of normal weights.  With weights on every
    input it is no larger than the float32 instructions' (whose mode takes the
    hardware's sines).  With none on the direction only the split differs: two
    operands off by a 2^-24 (rms) each at every product, where a float32 product
    rounds once, stay within four times their error; colours of 1e-5 alone are
    too far below the bound of the hidden units for that."""
    size, sc, x = lit
    X = np.concatenate([x, _direction()], 1)
    norms = {"float32 instructions": [], "default": []}
    for seed in range(6):
        rng = np.random.default_rng(seed)
        W0, W1, W2 = (scale * rng.normal(size=s) for s in ((34, 16), (16, 16), (16, 3)))
        if not direction:
            W0[7:] = 0.0
        w = [np.float32(a).astype(np.float64) for a in (W0, W1, W2)]
        y = np.maximum(np.maximum(X @ w[0], 0.0) @ w[1], 0.0) @ w[2] + x[:, :3]
        exact = _pack(W0.astype(np.float32) * np.float32(2.0 ** 60), W1.astype(np.float32) * np.float32(2.0 ** -60), W2)
        for name, mlp in (("float32 instructions", exact), ("default", _pack(W0, W1, W2))):
            norms[name].append(np.linalg.norm(_rgb(torch, merf, sc, mlp) - y) / np.linalg.norm(y))
    a, b = (float(np.sqrt(np.mean(np.square(v)))) for v in norms.values())
    print(f"inputs {size} weights {scale} direction {direction}: float32 instructions {a:.2e}, default {b:.2e}", flush=True)
    if direction:
        assert b <= a
    elif size != "1e-5":
        assert b <= 4 * a
