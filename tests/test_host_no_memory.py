"""What the library does when the device runs out of memory (CPU).

libpt.so runs on stand-ins of the HIP calls (hip_host_stub.c) whose memory has a
budget and whose kernels do nothing, each test in a process of its own.
"""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, sys
stub = C.CDLL({stub!r}, mode=C.RTLD_GLOBAL)
stub.stub_held.restype = stub.stub_peak.restype = C.c_size_t
stub.stub_budget.argtypes = [C.c_size_t]
stub.stub_mallocs.restype = stub.stub_launches.restype = C.c_long
stub.stub_fail_malloc.argtypes = [C.c_long]
sys.path.insert(0, {root!r})
import numpy as np
from paper_2407_19977_amd import pt, scenes


class Mem:
    # a buffer of the stand-in's memory with what the binding asks of a tensor
    def __init__(self, *shape):
        self.shape, self.a = shape, np.zeros(shape, np.float64)
    def data_ptr(self):
        return self.a.ctypes.data
    def numel(self):
        return self.a.size


def status(f, *args, **kw):
    try:
        f(*args, **kw)
    except pt.PtError as e:
        return e.status
    return 0
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_host_stub.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_host_stub.c")], check=True)
    return so


def _run(stub, body):
    code = PRELUDE.format(stub=stub, root=ROOT) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_failed_allocation_is_reported_once(stub):
    """The call after one that ran out of memory does not report that error again."""
    _run(stub, """
    sc = scenes.cornell()
    rays, hits = Mem(4, 8), Mem(4, 6)
    s = pt.PtScene(0)
    stub.stub_fail_malloc(1)
    assert status(s.build_bvh, sc.meshes) == -3
    stub.stub_fail_malloc(0)
    assert status(s.build_bvh, sc.meshes) == 0, pt.last_error()
    s.upload_materials(sc.materials)
    out = Mem(16, 16, 3)
    cam = sc.with_camera(width=16, height=16).camera
    stub.stub_fail_malloc(3)
    assert status(s.render, cam, 1, 3, 0, out) == -3
    stub.stub_fail_malloc(0)
    assert status(s.trace_closest, rays, hits) == 0, pt.last_error()
    """)


def test_failed_two_level_build_leaves_no_bvh(stub):
    """Whatever allocation fails, a two-level build that replaced part of the old hierarchy leaves none."""
    _run(stub, """
    def mesh(level):
        v, f = scenes.icosphere(level)
        return scenes.Mesh(v.astype(np.float32), f.astype(np.int32), np.zeros(len(f), np.int32))
    def placed(n):
        return [scenes.Instance(np.array([[1, 0, 0, 3 * k], [0, 1, 0, 0], [0, 0, 1, 0]], np.float32), 0, -1) for k in range(n)]
    rays, hits = Mem(4, 8), Mem(4, 6)
    failed = 0
    for k in range(1, 40):
        s = pt.PtScene(0)
        s.build_bvh([mesh(1)], placed(3))
        assert status(s.trace_closest, rays, hits) == 0
        stub.stub_fail_malloc(k)
        r = status(s.build_bvh, [mesh(3), mesh(2)], placed(40))
        stub.stub_fail_malloc(0)
        if r == 0:
            break
        failed += 1
        assert r == -3, r
        launched = stub.stub_launches()
        assert status(s.trace_closest, rays, hits) == -5, k
        assert stub.stub_launches() == launched
        s.build_bvh([mesh(3)], placed(2))
        assert status(s.trace_closest, rays, hits) == 0, pt.last_error()
        s.close()
    assert failed >= 5
    """)


def test_long_passes_leave_room_and_shrink(stub):
    """Passes of many samples leave the device as much free memory as they hold, down to one sample."""
    _run(stub, """
    sc = scenes.cornell()
    s = pt.scene_from(sc, device=0)
    cam = sc.with_camera(width=512, height=512).camera
    out, base = Mem(512, 512, 3), stub.stub_held()
    one = None
    for gib in (64.0, 16.0, 4.0, 1.0, 0.25):
        stub.stub_budget(base + int(gib * 2 ** 30))
        assert status(s.render, cam, 400, 5, 0, out) == 0, (gib, pt.last_error())
        held = stub.stub_held() - base
        assert held <= 0.5 * gib * 2 ** 30 + 2 ** 24, (gib, held)  # (the sums and counters beside the paths)
        s.close()
        s = pt.scene_from(sc, device=0)
    # one sample of every pixel, and no more, fits
    stub.stub_budget(1 << 40)
    s.render(cam, 1, 5, 0, out)
    one = stub.stub_held()
    s.close()
    s = pt.scene_from(sc, device=0)
    stub.stub_budget(one)
    assert status(s.render, cam, 400, 5, 0, out) in (0, -3)
    assert status(s.render, cam, 1, 5, 0, out) == 0, pt.last_error()
    """)


def test_idle_path_sets_are_given_back(stub):
    """What a long render holds is there again for the scene's other calls when the device is full."""
    _run(stub, """
    sc = scenes.cornell()
    cam = sc.with_camera(width=512, height=512).camera
    big = sc.with_camera(width=1024, height=1024).camera
    out = Mem(1024, 1024, 3)
    v, f = scenes.icosphere(5)
    mesh = scenes.Mesh(v.astype(np.float32), f.astype(np.int32), np.zeros(len(f), np.int32))

    def frames(s):
        s.set_radiance_cache(pt.cache_config())
        s.render(big, 3, 5, 0, out)

    def records(s):
        s.set_radiance_cache(pt.cache_config(train_paths=1 << 20))
        x, t = Mem(64, 12), Mem(64, 3)
        s.nrc_training_records(cam, 0, 5, 0, x, t)

    calls = dict(
        one_sample=lambda s: s.render(big, 1, 5, 0, out),
        tail_off=lambda s: (s.set_tail(0, 0.0), s.render(big, 1, 5, 0, out)),
        frames=frames, records=records,
        host_build=lambda s: s.build_bvh([mesh]),
        sums=lambda s: s.set_accumulation(Mem(4096, 4096, 3), 1),
        environment=lambda s: s.set_environment(np.ones((512, 1024, 3), np.float32)),
        rays=lambda s: s.trace_closest(Mem(1 << 20, 8), Mem(1 << 20, 6)),
    )
    for name, call in calls.items():
        s = pt.scene_from(sc, device=0)
        stub.stub_budget(1 << 36)
        s.render(cam, 400, 5, 0, out)   # two path sets
        held = stub.stub_held()
        assert held > 4 << 30
        stub.stub_budget(held)          # others took the rest
        assert status(call, s) == 0, (name, pt.last_error())
        s.render(cam, 4, 5, 0, out)     # and the path sets are there again
        s.close()
        stub.stub_budget(1 << 36)
        assert stub.stub_held() == 0, name
    """)


def test_device_build_gets_idle_path_sets(stub):
    """As above for a build on the device.  Its kernels do nothing here, so it ends in their error: what
    it must not report is the lack of memory."""
    _run(stub, """
    sc = scenes.cornell()
    cam = sc.with_camera(width=512, height=512).camera
    v, f = scenes.icosphere(5)
    mesh = scenes.Mesh(v.astype(np.float32), f.astype(np.int32), np.zeros(len(f), np.int32))
    place = [scenes.Instance(np.eye(3, 4, dtype=np.float32), 0, -1)]
    for instances in ((), place):
        s = pt.scene_from(sc, device=0)
        s.render(cam, 400, 5, 0, Mem(512, 512, 3))
        stub.stub_budget(stub.stub_held())
        assert status(s.build_bvh, [mesh], instances, on_device=True) != 0
        assert "build failed" in pt.last_error() and "memory" not in pt.last_error(), pt.last_error()
        s.close()
        stub.stub_budget(1 << 36)
    """)


def test_failed_replacements_do_not_count_as_there(stub):
    """Materials, sums, the cache's workspace and its configuration: a call that ran out of memory after
    it gave up the old buffer leaves none, and later calls refuse or allocate again."""
    _run(stub, """
    sc = scenes.cornell()
    cam, big = (sc.with_camera(width=w, height=w).camera for w in (16, 512))
    out = Mem(512, 512, 3)

    def full(f, *args, **kw):
        stub.stub_fail_malloc(1)
        r = status(f, *args, **kw)
        stub.stub_fail_malloc(0)
        return r

    # materials (more of them than before)
    s = pt.scene_from(sc, device=0)
    assert full(s.upload_materials, np.tile(np.asarray(sc.materials, np.float32).reshape(-1, 39), (50, 1))) == -3
    assert status(s.render, cam, 1, 3, 0, out) == -5
    s.upload_materials(sc.materials)
    assert status(s.render, cam, 1, 3, 0, out) == 0
    # sums (a larger image)
    s.accumulate(cam, 0, 1, 3, 0)
    assert full(s.accumulate, big, 0, 1, 3, 0) == -3
    launched = stub.stub_launches()
    assert status(s.resolve, out) == -5 and status(s.display, Mem(512, 512)) == -5
    assert stub.stub_launches() == launched
    # the cache's workspace: a gradient of more samples, then one of fewer
    s.set_radiance_cache(pt.cache_config())
    g = Mem(pt.NRC_PARAMS)
    assert status(s.nrc_gradient, Mem(64, 12), Mem(64, 3), g) == 0
    assert full(s.nrc_gradient, Mem(1 << 16, 12), Mem(1 << 16, 3), g) == -3
    allocated = stub.stub_mallocs()
    assert status(s.nrc_gradient, Mem(64, 12), Mem(64, 3), g) == 0
    assert stub.stub_mallocs() > allocated
    # its configuration: self-training needs a buffer per training path
    s.set_radiance_cache(pt.cache_config(train_end_bounce=3))
    assert full(s.set_radiance_cache, pt.cache_config(train_end_bounce=3, train_paths=1 << 20)) == -3
    assert status(s.nrc_gradient, Mem(64, 12), Mem(64, 3), g) == -5
    """)
