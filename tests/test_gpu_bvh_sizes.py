"""Device BVH builds at the sizes where their kernels change form (GPU).

One triangle, clusters at the edges of a block of 256, the limit of the
one-workgroup finish (2048 clusters), the scans' tile (4096 counts: 8 radix
tiles of 2048 keys are 2048 counts, 17 are 4352) and a build whose first
clustering rounds have more than 8192 blocks, so that their counts are scanned
instead of summed.  Any valid tree is accepted; the checks are exact.
"""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _mesh(kind, n):
    from paper_2407_19977_amd import scenes
    r = np.random.default_rng(n)
    if kind == "random":
        v = r.uniform(-1, 1, (n, 1, 3)) + r.normal(0, 0.02, (n, 3, 3))
    elif kind == "equal":  # every box the same: ties everywhere
        v = np.tile(r.uniform(-1, 1, (1, 3, 3)), (n, 1, 1))
    else:  # areas overflow to infinity
        v = r.uniform(-3e38, 3e38, (n, 3, 3))
    return scenes.Mesh(np.ascontiguousarray(v.reshape(-1, 3), np.float32),
                       np.arange(3 * n, dtype=np.int32).reshape(-1, 3), np.zeros(n, np.int32))


def _check(nodes, tris, n):
    f = nodes.view(np.float32).reshape(-1, 32)
    u = nodes.view(np.uint32).reshape(-1, 32)
    lo = np.stack([f[:, 0:4], f[:, 8:12], f[:, 16:20]], -1)
    hi = np.stack([f[:, 4:8], f[:, 12:16], f[:, 20:24]], -1)
    child, kids = u[:, 24:28], u[:, 28]
    used = np.arange(4)[None, :] < kids[:, None]
    assert np.all((kids >= 1) & (kids <= 4)) and np.all(child[~used] == 0xFFFFFFFF)
    leaf = used & ((child & 0x80000000) != 0)
    inner = used & ~leaf
    # every node but the root is one child, every triangle is in one leaf
    assert np.array_equal(np.sort(child[inner]), np.arange(1, len(f)))
    first, cnt = child[leaf] & ((1 << 27) - 1), (child[leaf] >> 27) & 7
    o = np.argsort(first)
    assert np.all((cnt >= 1) & (cnt <= 4)) and first[o][0] == 0
    assert np.array_equal(first[o][1:], (first[o] + cnt[o])[:-1]) and first[o][-1] + cnt[o][-1] == n
    prim = tris.view(np.uint32).reshape(-1, 12)[:, 3]
    assert np.array_equal(np.sort(prim), np.arange(n))
    # boxes: the children of a child lie in its box, triangles in their leaf's
    c = child[inner]
    inf = np.float32(np.inf)
    box_lo = np.where(used[:, :, None], lo, inf).min(1)
    box_hi = np.where(used[:, :, None], hi, -inf).max(1)
    assert np.all(box_lo[c] >= lo[inner]) and np.all(box_hi[c] <= hi[inner])
    v = tris.view(np.float32).reshape(-1, 12)[:, [0, 1, 2, 4, 5, 6, 8, 9, 10]].reshape(-1, 3, 3)
    rep = np.repeat(np.arange(len(o)), cnt[o])
    assert np.all(v.min(1) >= lo[leaf][o][rep]) and np.all(v.max(1) <= hi[leaf][o][rep])


@pytest.mark.parametrize("builder", ["ploc", "lbvh"])
@pytest.mark.parametrize("kind,n", [("random", k) for k in (1, 2, 3, 255, 256, 257, 2048, 2049, 16384, 34817, 2097409)] +
                         [("equal", k) for k in (257, 2049, 5000)] + [("huge", k) for k in (257, 5000)])
def test_device_build_is_a_bvh_of_the_mesh(builder, kind, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[build] {builder} {kind} {n}", flush=True)
    from paper_2407_19977_amd import pt
    m = _mesh(kind, n)
    s = pt.PtScene(0)
    try:
        s.set_gpu_bvh_builder(builder)
        s.build_bvh([m], on_device=True)
        assert s.bvh_info()["n_tris"] == n
        nodes, tris = s.copy_bvh()
        _check(nodes, tris, n)
        src = m.vertices.reshape(n, 9)
        t = tris.view(np.float32).reshape(-1, 12)
        prim = tris.view(np.uint32).reshape(-1, 12)[:, 3]
        assert np.array_equal(t[:, [0, 1, 2, 4, 5, 6, 8, 9, 10]], src[prim])
    finally:
        s.close()
