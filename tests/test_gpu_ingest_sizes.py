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


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("n,off_in,off_out", [(1, 0, 0), (15, 0, 0), (16, 0, 0), (17, 0, 0), (4099, 0, 0), (65536, 0, 0),
                                              (100, 1, 0), (300, 16, 3), (257, 5, 1), (70001, 0, 8)])
def test_dequantize_sizes_and_alignments(torch, merf, prec, n, off_in, off_out):
    """Every size and alignment gives the values of the 256 codes one by one,
    and nothing past the n outputs is written."""
    dt = [torch.float32, torch.float16, torch.bfloat16][prec]
    rng = np.random.default_rng(n)
    codes = torch.from_numpy(rng.integers(0, 256, n + off_in, dtype=np.uint8)).cuda()
    out = torch.full((n + off_out + 8,), 99.0, dtype=dt, device="cuda")
    table = torch.empty(256, dtype=dt, device="cuda")
    one = torch.arange(256, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    for c in range(256):                         # one code a call: the scalar form
        merf.merf_dequantize(one.data_ptr() + c, 1, 7.0, prec, table.data_ptr() + c * table.element_size(), st)
    merf.merf_dequantize(codes.data_ptr() + off_in, n, 7.0, prec, out.data_ptr() + off_out * out.element_size(), st)
    torch.cuda.synchronize()
    assert torch.equal(out[off_out:off_out + n], table[codes[off_in:].long()])
    assert bool((out[:off_out] == 99.0).all()) and bool((out[off_out + n:] == 99.0).all())
