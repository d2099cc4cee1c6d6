"""The host side of uploads on the CPU: csrc/merf_api.hip over a stand-in for
the HIP runtime (fake_hip.cpp), which counts what waits for the device and has
as much memory as a test gives it."""
import ctypes as C
import os
import subprocess
import sys
import time

import numpy as np
import pytest

import synth
from paper_2302_12249_amd import merf
from scene_builders import dense_scene

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2302_12249_amd", "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")


def build(out):
    flags = ["-std=c++17", "-O1", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))",
             "-DHIP_SYMBOL(x)=&x", "-I/opt/rocm/include", "-I" + INCLUDE, "-I" + CSRC]
    subprocess.run(["g++", *flags, "-shared", "-Wl,-Bsymbolic", "-x", "c++", os.path.join(CSRC, "merf_api.hip"),
                    os.path.join(HERE, "fake_hip.cpp"), "-o", out, "-pthread"], check=True)


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("fake") / "libmerf_fake.so")
    build(path)
    return path


@pytest.fixture()
def lib(so, tmp_path):
    """A library of its own for each test: the state of uploads is the process's."""
    path = str(tmp_path / "libmerf_fake.so")
    with open(so, "rb") as f, open(path, "wb") as g:
        g.write(f.read())
    return declare(C.CDLL(path))


def declare(lib):
    for name in ("fake_held", "fake_pool_kept", "fake_pinned", "fake_peak", "merf_hbm_in_use", "merf_scene_bytes"):
        getattr(lib, name).restype = C.c_size_t
    lib.fake_capacity.argtypes = [C.c_size_t]
    lib.merf_set_hbm_budget.argtypes = [C.c_size_t]
    lib.fake_waits.restype = lib.fake_fail_new.restype = C.c_long
    lib.fake_fail_new.argtypes = [C.c_long]
    lib.merf_free.argtypes = lib.merf_scene_bytes.argtypes = lib.fake_image.argtypes = lib.fake_release_on.argtypes = [C.c_void_p]
    lib.merf_last_error.restype = C.c_char_p
    return lib


def upload(lib, scene, ordered=False):
    d, keep = merf.scene_desc(scene)
    h = C.c_void_p()
    rc = (lib.fake_upload_on if ordered else lib.merf_scene_upload)(C.byref(d), C.byref(h))
    del keep
    return rc, h.value


def large_scene():
    """300 MB of blocks and the rest small: its scratch is beyond what is kept."""
    sc = dense_scene(L=16, R=16)
    nb = 42
    sc.L, sc.block_index = 8 * nb, np.arange(nb ** 3, dtype=np.int32)
    sc.blocks = np.zeros((nb ** 3, 8, 8, 8, 8), np.uint8)
    return sc


SCENES = {"small": lambda: dense_scene(L=16, R=16), "medium": lambda: dense_scene(L=64, R=1024), "large": large_scene}


@pytest.mark.parametrize("size", sorted(SCENES))
def test_ordered_uploads_wait_for_no_other_work(lib, size):
    """The serving runtime's uploads: no call in them waits for the device."""
    sc = SCENES[size]()
    before = lib.fake_waits()
    rc, h = upload(lib, sc, ordered=True)
    assert rc == 0 and lib.fake_waits() == before
    assert lib.fake_release_on(h) == 0 and lib.fake_waits() == before
    assert lib.merf_hbm_in_use() == 0 and lib.fake_held() == lib.fake_pool_kept()


def test_ordered_release_keeps_what_would_have_to_wait(lib):
    """Evicting the last scene frees its memory in stream order and no more;
    the kept scratch and pinned buffers go back where the caller waits anyway."""
    sc = SCENES["medium"]()
    rc, h = upload(lib, sc, ordered=True)
    assert rc == 0 and lib.fake_pinned() > 0 and lib.fake_pool_kept() > 0
    time.sleep(1.1)                                # longer than memory is kept after its last use
    before = lib.fake_waits()
    assert lib.fake_release_on(h) == 0 and lib.fake_waits() == before
    lib.fake_release_unused()
    assert lib.fake_pinned() == lib.fake_held() == 0


def test_free_gives_back_what_was_kept(lib):
    rc, h = upload(lib, SCENES["medium"]())
    assert rc == 0 and lib.fake_pinned() > 0 and lib.fake_pool_kept() > 0
    time.sleep(1.1)
    assert lib.merf_free(h) == 0
    assert lib.fake_pinned() == lib.fake_held() == 0


def test_setting_the_budget_gives_back_what_is_kept(lib):
    rc, h = upload(lib, SCENES["medium"]())
    assert rc == 0 and lib.merf_free(h) == 0       # within a second of its use
    assert lib.fake_pinned() > 0 and lib.fake_pool_kept() > 0
    assert lib.merf_set_hbm_budget(2 ** 63) == 0
    assert lib.fake_pinned() == lib.fake_held() == 0


def test_scenes_and_kept_scratch_stay_below_the_budget(lib):
    sc = SCENES["medium"]()
    rc, h = upload(lib, sc)
    one = lib.merf_scene_bytes(h)
    assert rc == 0 and lib.merf_free(h) == 0
    room = 256 << 20                               # of scratch that may be kept
    for spare in (0, room - 1, room):
        budget = 3 * one + spare
        assert lib.merf_set_hbm_budget(budget) == 0
        hs = []
        for i in range(3):
            rc, h = upload(lib, sc, ordered=i == 1)
            assert rc == 0 and lib.fake_held() <= budget
            hs.append(h)
        assert lib.merf_hbm_in_use() == 3 * one
        assert (lib.fake_pool_kept() > 0) == (spare == room)
        rc, h = upload(lib, sc)                    # scratch takes nothing from the scenes' share
        assert rc == (merf.MERF_E_OOM if spare < one else 0) and lib.fake_held() <= budget
        if rc == 0:
            assert lib.merf_free(h) == 0
        rc = [lib.fake_release_on(h) if i == 1 else lib.merf_free(h) for i, h in enumerate(hs)]
        assert not any(rc)


def test_kept_scratch_does_not_stand_in_the_way(lib):
    """A device with room for a scene but not for the kept scratch beside it."""
    sc = SCENES["medium"]()
    rc, h = upload(lib, sc, ordered=True)
    one = lib.merf_scene_bytes(h)
    assert rc == 0 and lib.fake_image(h) == 0 and lib.fake_release_on(h) == 0
    assert lib.fake_pool_kept() > 0
    lib.fake_capacity(one)
    back = C.c_void_p()
    assert lib.fake_restore(C.byref(back)) == 0    # admitted again from its image
    assert lib.fake_held() == one


def octants(lib, r):
    occ, out = np.zeros(r ** 3, np.uint8), np.zeros(8, np.uint8)
    levels, res = (C.c_void_p * 1)(occ.ctypes.data), (C.c_int32 * 1)(r)
    return lib.merf_octant_extent_grid(levels, res, 1, C.c_void_p(out.ctypes.data), None)


@pytest.mark.parametrize("r", [16, 96, 100, 256, 272])
def test_octant_grids_need_no_more_memory_than_five_grids(lib, r):
    """A device with 5 r^3 bytes free (a little more where rows are padded by
    much) builds the grids, one octant after another."""
    assert octants(lib, r) == 0 and lib.fake_octants_together() == (r <= 256)
    lib.merf_set_hbm_budget(2 ** 64 - 1)
    lib.fake_capacity(5 * r ** 3)
    assert octants(lib, r) == 0 and not lib.fake_octants_together()
    assert lib.fake_held() <= 5 * r ** 3
    lib.fake_capacity(2 * r ** 3)
    assert octants(lib, r) == merf.MERF_E_OOM and lib.fake_held() == 0


def test_octants_respect_the_budget(lib):
    lib.merf_set_hbm_budget(10 * 64 ** 3 - 1)
    assert octants(lib, 64) == 0 and not lib.fake_octants_together()
    lib.merf_set_hbm_budget(10 * 64 ** 3)
    assert octants(lib, 64) == 0 and lib.fake_octants_together()


@pytest.mark.parametrize("ordered", [False, True])
def test_uploads_fit_where_they_did(lib, ordered):
    """Memory for the scene, its staging and five grids beside them."""
    sc = dense_scene(L=64, R=64)
    r = 128
    sc.occ = [(r, np.ones((r, r, r), np.uint8))]
    rc, h = upload(lib, sc, ordered)
    one = lib.merf_scene_bytes(h)
    assert rc == 0 and lib.fake_octants_together()
    assert (lib.fake_release_on(h) if ordered else lib.merf_free(h)) == 0
    lib.merf_set_hbm_budget(2 ** 64 - 1)
    staging = sc.blocks.nbytes + sc.block_index.nbytes + 4 * 8 ** 3
    lib.fake_capacity(one + staging + 5 * r ** 3)
    rc, h = upload(lib, sc, ordered)
    assert rc == 0 and not lib.fake_octants_together()
    lib.fake_capacity(one + staging + r ** 3)
    assert upload(lib, sc, ordered)[0] == merf.MERF_E_OOM
    assert lib.merf_hbm_in_use() == one == lib.fake_held()


SWEEP = """
import sys
sys.path[:0] = [{root!r}, {here!r}]
import ctypes as C
import test_upload_host as T
from scene_builders import dense_scene
from paper_2302_12249_amd import merf
lib = T.declare(C.CDLL({so!r}))
sc = dense_scene(L=16, R=512)
for ordered in (False, True):
    n, failed = 0, 0
    while True:
        n += 1
        lib.fake_fail_new(n)
        rc, h = T.upload(lib, sc, ordered)
        left = lib.fake_fail_new(0)
        assert rc in (0, merf.MERF_E_OOM, merf.MERF_E_DEVICE), rc
        failed += rc != 0
        if rc == 0:
            assert (lib.fake_release_on(h) if ordered else lib.merf_free(h)) == 0
        assert lib.merf_hbm_in_use() == 0 and lib.fake_held() == lib.fake_pool_kept(), (n, rc)
        if left > 0:
            break
    print(ordered, n, failed, flush=True)
    assert failed > 5
"""


def test_uploads_without_host_memory_fail_cleanly(so, tmp_path):
    """Each allocation of an upload fails in turn (those of the copying threads
    among them): an error code or an upload all the same, and nothing left.  In
    a process of its own, which an exception in the wrong place would end."""
    path = str(tmp_path / "libmerf_fake.so")
    with open(so, "rb") as f, open(path, "wb") as g:
        g.write(f.read())
    code = SWEEP.format(root=os.path.dirname(HERE), here=HERE, so=path)
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
