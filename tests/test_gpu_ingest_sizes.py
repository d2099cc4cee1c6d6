"""Ingest kernels at the edges of their ranges: pooling with every vector
width, unaligned masks, levels pooled from levels, rows that are split over
workgroups and rows that share one; empty-space octants at rows of one lane,
of a part of a wave, of a whole one and of the wide form (octant by octant).
The results are whole numbers and must equal numpy's."""
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


def _extent_at(comb, cells):
    """Octant extents [8, n] of the cells (x, y, z) by bisection in a table of
    prefix sums: the largest empty cube, clipped to the grid, at most 255."""
    r = comb.shape[0]
    sat = np.zeros((r + 1,) * 3, np.int64)
    sat[1:, 1:, 1:] = comb.astype(np.int64).cumsum(0).cumsum(1).cumsum(2)
    out = np.zeros((8, len(cells)), np.int64)
    for o in range(8):
        lo, hi = np.zeros(len(cells), np.int64), np.full(len(cells), 255)
        while np.any(lo < hi):
            k = (lo + hi + 1) // 2
            a = [np.maximum(cells[:, i] - k + 1, 0) if o >> i & 1 else cells[:, i] for i in range(3)]
            b = [cells[:, i] + 1 if o >> i & 1 else np.minimum(cells[:, i] + k, r) for i in range(3)]
            n = 0
            for s, (x, y, z) in ((1, (b[0], b[1], b[2])), (-1, (a[0], b[1], b[2])), (-1, (b[0], a[1], b[2])),
                                 (-1, (b[0], b[1], a[2])), (1, (a[0], a[1], b[2])), (1, (a[0], b[1], a[2])),
                                 (1, (b[0], a[1], a[2])), (-1, (a[0], a[1], a[2]))):
                n = n + s * sat[z, y, x]
            lo, hi = np.where(n == 0, k, lo), np.where(n == 0, hi, k - 1)
        out[o] = lo
    return out


@pytest.mark.parametrize("density", [0.0, 2e-5, 0.002, 0.2])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 16, 17, 24, 33, 48, 63, 64, 100, 130, 192, 241, 256, 257, 320])
def test_octant_extent_sizes(torch, merf, r, density):
    rng = np.random.default_rng(r)
    fine = (rng.random((r,) * 3) < density).astype(np.uint8)
    coarse = [synth.maxpool(fine, f) for f in (4, 2) if r % 4 == 0]
    if coarse:                                   # levels that are no max-pools: the AND of all decides
        coarse[0] = coarse[0] & (rng.random(coarse[0].shape) < 0.8)
    levels = [o.astype(np.uint8) for o in coarse] + [fine]
    got = merf.distance_grid([torch.from_numpy(np.ascontiguousarray(o)).cuda() for o in levels], octants=True)
    torch.cuda.synchronize()
    comb = fine > 0
    for o in levels[:-1]:
        k = r // o.shape[0]
        comb &= np.repeat(np.repeat(np.repeat(o > 0, k, 0), k, 1), k, 2)
    n = min(r ** 3, 40000)
    cells = np.stack(np.unravel_index(rng.choice(r ** 3, n, replace=False), (r,) * 3)[::-1], 1)
    got = got[:, torch.from_numpy(cells[:, 2]).cuda(), torch.from_numpy(cells[:, 1]).cuda(),
              torch.from_numpy(cells[:, 0]).cuda()].cpu().numpy()
    assert np.array_equal(got, _extent_at(comb, cells))
