"""The fp32 deferred MLP against float64 on an empty scene, where a pixel is
h(0, 0, d) alone: parameters of every magnitude (the matrix kernels hold
float32 operands as scaled pairs of float16 values, so neither large nor small
ones may lose precision), columns of very different sizes, and parameters that
are not finite.

Bound: the encoded sines and cosines are within 1e-5 and every float32 step
rounds to 2^-24 relative, so an output is off by at most the largest gain of
the layers times 1e-5 plus 64 roundings of the largest value it can pass
through."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import gpu_render

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


def _params(case, rng):
    w = rng.normal(0.0, 1.0, synth.mlp_param_count())
    n0, n1 = 34 * 16, 34 * 16 + 16
    if case == "columns":                        # units and inputs of very different sizes
        w *= np.exp(rng.normal(0.0, 4.0, w.size))
    elif case == "layers":                       # layers of very different sizes
        w[:n1] *= 1e-6
        w[n1:n1 + 272] *= 1e7
        w[n1 + 272:] *= 1e-3
    elif case == "zero":
        w[:n0] = 0.0
    else:
        w *= float(case)
    return w.astype(np.float32)


def _reference(w, cams):
    p = w.astype(np.float64)
    W0, b0, p = p[:544].reshape(34, 16), p[544:560], p[560:]
    W1, b1, p = p[:256].reshape(16, 16), p[256:272], p[272:]
    W2, b2 = p[:48].reshape(16, 3), p[48:]
    wd, ht = int(cams.size[0, 0]), int(cams.size[0, 1])
    r, c = np.divmod(np.arange(wd * ht), wd)
    _, d = oracle.camera_rays(cams, 0, r, c)
    x = np.concatenate([np.zeros((len(d), 7)), d] + [np.sin(2.0 ** k * d) for k in range(4)] +
                       [np.cos(2.0 ** k * d) for k in range(4)], 1)
    with np.errstate(all="ignore"):
        h = np.fmax(np.fmax(x @ W0 + b0, 0.0) @ W1 + b1, 0.0)
        y = h @ W2 + b2
        g0 = np.abs(W0).sum(0)
        gain = (g0 @ np.abs(W1)) @ np.abs(W2)
        top = ((g0 + np.abs(b0)) @ np.abs(W1) + np.abs(b1)) @ np.abs(W2) + np.abs(b2)
    return y, 1e-5 * gain + 64 * 2.0 ** -24 * top


@pytest.mark.parametrize("case", ["0.1", "1", "1e-3", "1e-9", "1e-14", "1e6", "1e12", "columns", "layers", "zero"])
@pytest.mark.parametrize("seed", [0, 1])
def test_mlp_magnitudes(torch, merf, tiny_scene, case, seed):
    rng = np.random.default_rng(seed)
    w = _params(case, rng)
    sc = dataclasses.replace(tiny_scene, mlp=w, occ=[(r, np.zeros_like(o)) for r, o in tiny_scene.occ])
    cams = synth.tiny_camera(seed=30 + seed, w=52, h=37)
    y, bound = _reference(w, cams)
    got = gpu_render(torch, merf, sc, cams)
    assert np.all(got[:, 3] == 0.0)
    err = np.abs(got[:, :3] - y).max(0)
    print(f"mlp {case}: max err {err} bound {bound}", flush=True)
    assert np.all(err <= bound)


@pytest.mark.parametrize("where,value", [(5, np.nan), (16 * 20 + 3, np.nan), (544 + 2, np.inf), (560 + 7, np.nan), (560 + 256 + 1, -np.inf)])
def test_mlp_parameters_that_are_not_finite(torch, merf, tiny_scene, where, value):
    """A NaN before a ReLU gives 0, as fmax does; the other units are as ever."""
    rng = np.random.default_rng(3)
    w = _params("0.1", rng)
    w[where] = value
    sc = dataclasses.replace(tiny_scene, mlp=w, occ=[(r, np.zeros_like(o)) for r, o in tiny_scene.occ])
    cams = synth.tiny_camera(seed=31, w=17, h=9)
    y, _ = _reference(w, cams)
    got = gpu_render(torch, merf, sc, cams)[:, :3]
    assert np.array_equal(np.isnan(got), np.isnan(y)) and np.array_equal(np.isinf(got), np.isinf(y))
    ok = np.isfinite(y)
    assert np.all(np.abs(got - y)[ok] <= 1e-4)
