"""Several samples per pixel in one sampling pass (GPU).

A call of n samples runs them in as few passes as fit, its pixels in blocks
of 8x8 and a pixel's samples in neighbouring slots.  The FP64 sums must not
depend on that grouping (each path's radiance is the same floats, added in
sample order), so every comparison here is bit for bit.
"""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# block edges and remainders in each direction, one pixel, one row, one column
SIZES = [(1, 1), (7, 3), (8, 8), (9, 17), (65, 1), (1, 23), (40, 31)]


@pytest.fixture(scope="module")
def scene():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_19977_amd import pt, scenes
    sc = scenes.cornell()
    s = pt.scene_from(sc, device=0)
    yield sc, s
    s.close()


@pytest.mark.parametrize("w,h", SIZES)
@pytest.mark.parametrize("spp", [2, 5])
def test_sums_do_not_depend_on_the_grouping(scene, w, h, spp):
    print(f"[passes] {w}x{h}, {spp} spp", flush=True)
    sc, s = scene
    cam = sc.with_camera(width=w, height=h).camera
    mean = torch.empty((h, w, 3), dtype=torch.float32, device="cuda:0")
    sums = [torch.empty((h, w, 3), dtype=torch.float64, device="cuda:0") for _ in range(2)]
    s.reset_accumulation()
    for k in range(spp):
        s.accumulate(cam, 3 + k, 1, 4, 11)
    s.resolve(mean, sums[0])
    s.reset_accumulation()
    s.accumulate(cam, 3, spp, 4, 11)
    s.resolve(mean, sums[1])
    assert torch.equal(sums[0], sums[1])
    # per sample: the rows, columns and sample indices of the debug output are the image's
    per = torch.empty((h, w, spp, 3), dtype=torch.float32, device="cuda:0")
    sig = torch.empty((h, w, spp), dtype=torch.int64, device="cuda:0")
    s.render_debug(cam, 0, 0, w, h, 3, spp, 4, 11, per, sig)
    acc = np.zeros((h, w, 3))
    for k in range(spp):
        acc += per[:, :, k].cpu().numpy().astype(np.float64)
    assert np.array_equal(acc, sums[1].cpu().numpy())
    if w > 2 and h > 2:  # a crop gives the same paths
        pc = torch.empty((h - 2, w - 2, spp, 3), dtype=torch.float32, device="cuda:0")
        sg = torch.empty((h - 2, w - 2, spp), dtype=torch.int64, device="cuda:0")
        s.render_debug(cam, 1, 2, w - 2, h - 2, 3, spp, 4, 11, pc, sg)
        assert torch.equal(pc, per[2:, 1:w - 1]) and torch.equal(sg, sig[2:, 1:w - 1])


@pytest.mark.parametrize("which", ["material_zoo", "instanced", "cornell"])
def test_one_shading_launch_equals_one_per_class(which):
    """Passes of at most 2^20 slots shade all material classes in one launch, larger ones launch a
    kernel per class: three samples of 640x640 (1.23M slots) in one pass against one by one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[passes] {which} 640x640, 3 spp, classes", flush=True)
    from paper_2407_19977_amd import pt, scenes
    sc = getattr(scenes, which)()
    cam = sc.with_camera(width=640, height=640).camera
    s = pt.scene_from(sc, device=0)
    mean = torch.empty((640, 640, 3), dtype=torch.float32, device="cuda:0")
    sums = [torch.empty((640, 640, 3), dtype=torch.float64, device="cuda:0") for _ in range(2)]
    s.set_tail(0, 0.0)  # every vertex in the wavefront kernels
    s.accumulate(cam, 0, 3, 6, 11)
    s.resolve(mean, sums[0])
    s.reset_accumulation()
    for k in range(3):
        s.accumulate(cam, k, 1, 6, 11)
    s.resolve(mean, sums[1])
    s.close()
    assert torch.equal(sums[0], sums[1])


@pytest.mark.parametrize("w,h,spp", [(1, 1, 2100), (5, 3, 300), (17, 9, 9), (3, 2, 2048)])
def test_sums_of_many_samples(scene, w, h, spp):
    """Accumulation stages 2048 slots at a time: fewer pixels a tile for more than 8 samples, and parts
    of one pixel's samples for more than 2048."""
    print(f"[passes] {w}x{h}, {spp} spp", flush=True)
    sc, s = scene
    cam = sc.with_camera(width=w, height=h).camera
    mean = torch.empty((h, w, 3), dtype=torch.float32, device="cuda:0")
    sums = torch.empty((h, w, 3), dtype=torch.float64, device="cuda:0")
    s.reset_accumulation()
    s.accumulate(cam, 1, spp, 3, 7)
    s.resolve(mean, sums)
    per = torch.empty((h, w, spp, 3), dtype=torch.float32, device="cuda:0")
    sig = torch.empty((h, w, spp), dtype=torch.int64, device="cuda:0")
    s.render_debug(cam, 0, 0, w, h, 1, spp, 3, 7, per, sig)
    acc = np.zeros((h, w, 3))
    for k in range(spp):
        acc += per[:, :, k].cpu().numpy().astype(np.float64)
    assert np.array_equal(acc, sums.cpu().numpy())
    # the debug output's samples are the ones of passes of their own
    one = torch.empty((h, w, 1, 3), dtype=torch.float32, device="cuda:0")
    sg = torch.empty((h, w, 1), dtype=torch.int64, device="cuda:0")
    for k in (0, 1, spp // 2, spp - 1):
        s.render_debug(cam, 0, 0, w, h, 1 + k, 1, 3, 7, one, sg)
        assert torch.equal(one[:, :, 0], per[:, :, k]) and torch.equal(sg[:, :, 0], sig[:, :, k])
