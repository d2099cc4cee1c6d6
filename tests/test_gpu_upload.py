"""Uploads that share the library's kept scratch and pinned buffers: scenes
opened and closed in turn, from several threads at once (one stages, the others
copy plainly), from pageable, pinned and device memory, and empty-space grids
built on several streams.  Every result must equal the one of a lone upload."""
import dataclasses
import threading

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


@pytest.fixture(scope="module")
def merf():
    from paper_2302_12249_amd import merf as m
    m.load()
    return m


@pytest.fixture(scope="module")
def scenes():
    # planes of 25 MB (staged, with a last piece that is no whole chunk) and blocks of some MB
    return [synth.make_scene(128, 1023 + i, 0.05, 1.99, 0.1, 0.3, seed=40 + i) for i in range(2)]


def test_uploads_in_turn_and_from_threads_agree(torch, merf, scenes):
    cams = synth.orbit_cameras(1, w=160, h=96)
    want = [gpu_render(torch, merf, s, cams) for s in scenes]
    for _ in range(2):
        for s, w in zip(scenes, want):
            assert np.array_equal(gpu_render(torch, merf, s, cams), w)
    bad = []

    def work(k):
        stream = torch.cuda.Stream()
        for i in range(4):
            s, w = scenes[(i + k) % 2], want[(i + k) % 2]
            r = merf.Renderer(s)
            out = torch.empty((cams.num_pixels(), 4), device="cuda")
            torch.cuda.current_stream().synchronize()
            r.render(cams, out=out, stream=stream)
            stream.synchronize()
            if not np.array_equal(out.cpu().numpy().astype(np.float64), w):
                bad.append((k, i))
            r.close()

    ts = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad


def test_upload_sources_agree(torch, merf, scenes):
    cams = synth.orbit_cameras(1, w=64, h=48)
    s = scenes[0]
    want = gpu_render(torch, merf, s, cams)
    pinned = torch.from_numpy(s.planes).pin_memory()
    for planes in (pinned.numpy(), torch.from_numpy(s.planes).cuda(), s.planes[::1].copy()):
        assert np.array_equal(gpu_render(torch, merf, dataclasses.replace(s, planes=planes), cams), want)


def test_empty_space_grids_on_streams_agree(torch, merf):
    rng = np.random.default_rng(1)
    levels = [[torch.from_numpy((rng.random((r,) * 3) < 0.002).astype(np.uint8)).cuda()] for r in (96, 130, 64)]
    want = [[merf.distance_grid(l, octants=o).cpu() for o in (True, False)] for l in levels]
    bad = []

    def work(k):
        st = torch.cuda.Stream()
        for i in range(6):
            j = (i + k) % 3
            with torch.cuda.stream(st):
                got = merf.distance_grid(levels[j], stream=st, octants=i % 2 == 0)
            st.synchronize()
            if not torch.equal(got.cpu(), want[j][i % 2]):
                bad.append((k, i))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad
