"""Ingest kernels at the edges of their ranges: pooling with every vector
width, unaligned masks, levels pooled from levels, rows that are split over
workgroups and rows that share one.  The results are whole numbers and must
equal numpy's."""
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


@pytest.mark.parametrize("density", [0.0, 0.0005, 0.3])
@pytest.mark.parametrize("res,factors,offset", [
    (1, (1,), 0), (2, (1, 2), 0), (5, (5, 1), 0), (7, (7,), 1), (12, (3, 4, 6, 12), 0), (12, (3, 4), 4), (45, (15, 9, 5), 0),
    (60, (4, 6), 8), (64, (64, 16, 4, 1), 0), (64, (32,), 3), (128, (2, 1), 0), (128, (8, 8), 16), (160, (32, 5), 0),
    (256, (256, 128), 0), (192, (48, 64, 3), 0)])
def test_pyramid_sizes(torch, merf, res, factors, offset, density):
    rng = np.random.default_rng(res + offset)
    mask = (rng.random((res,) * 3) < density).astype(np.uint8) * rng.integers(1, 256, (res,) * 3, dtype=np.uint8)
    buf = torch.zeros(res ** 3 + offset, dtype=torch.uint8, device="cuda")
    dev = buf[offset:].view(res, res, res)       # offset: a mask not aligned to the vectors
    dev.copy_(torch.from_numpy(mask))
    outs = merf.occupancy_pyramid(dev, factors)
    torch.cuda.synchronize()
    occ = (mask > 0).astype(np.uint8)
    for f, o in zip(factors, outs):
        assert np.array_equal(o.cpu().numpy(), synth.maxpool(occ, f) if f > 1 else occ), (res, f)

