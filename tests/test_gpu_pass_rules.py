"""The persistent kernel's share of a pass (GPU).

A pass of at most 327,680 slots runs in the persistent kernel from its first
vertex; larger ones start in the wavefront kernels and hand over once few
paths are left.  Both run the same arithmetic on the same random numbers, so
the images, sums of radiances included, are compared bit for bit with the
wavefront kernels' own (hand-over switched off).
"""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# one path, less than a wave, the rule's edge (640 x 512 x 1 = 327,680 slots) and one block row more
CASES = [(1, 1, 1), (5, 3, 4), (101, 67, 5), (640, 512, 1), (640, 520, 1), (320, 256, 5)]


@pytest.fixture(scope="module", params=["cornell", "instanced"])
def scene(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_19977_amd import pt, scenes
    sc = scenes.cornell() if request.param == "cornell" else scenes.instanced()
    s = pt.scene_from(sc, device=0)
    yield sc, s
    s.close()


@pytest.mark.parametrize("w,h,spp", CASES)
def test_hand_over_rule_keeps_the_bits(scene, w, h, spp):
    print(f"[rule] {w}x{h}, {spp} spp", flush=True)
    sc, s = scene
    cam = sc.with_camera(width=w, height=h).camera
    out = [torch.empty((h, w, 3), dtype=torch.float32, device="cuda:0") for _ in range(3)]
    try:
        s.render(cam, spp, 6, 5, out[0])
        s.set_tail(0, 0.0)
        s.render(cam, spp, 6, 5, out[1])
        s.set_tail(0, 1.0)
        s.render(cam, spp, 6, 5, out[2])
    finally:
        s.set_tail()
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


@pytest.mark.parametrize("w,h,spp", [(101, 67, 2), (1024, 1024, 3)])
@pytest.mark.parametrize("first", [1, 3])
def test_a_set_hand_over_holds_at_any_size(scene, w, h, spp, first):
    """min_bounce and max_fraction that a caller set are used as they are, by passes of few slots
    and of more than 2^21: the persistent kernel takes over every path at vertex `first`."""
    print(f"[rule] {w}x{h}, {spp} spp, from bounce {first}", flush=True)
    sc, s = scene
    cam = sc.with_camera(width=w, height=h).camera
    out = torch.empty((h, w, 3), dtype=torch.float32, device="cuda:0")
    rays = []
    try:
        for args in ((first, 1.0), (0, 0.0)):
            s.set_tail(*args)
            for depth in (first - 1, 6):
                s.reset_stats()
                s.render(cam, spp, depth, 5, out)
                st = s.stats()
                rays.append((st["extension_rays"], st["tail_extension_rays"]))
    finally:
        s.set_tail()
    # the rays of the vertices before `first`, as a render of that depth traces them
    assert rays[1][0] == rays[3][0] and rays[3][1] == 0
    assert rays[1][0] - rays[1][1] == rays[2][0]
