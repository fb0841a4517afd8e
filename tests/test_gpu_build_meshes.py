"""Meshes gathered and checked on the device by a device build (GPU).

Large meshes are copied one by one, many small ones joined first; both have to
give the primitives, materials, lights and box of the host build, so closest
hits and renders are compared bit for bit.  Inputs that the host build refuses
are refused with its words, and leave the scene as it was.
"""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _split(mesh, parts):
    """The mesh as `parts` meshes with their own vertices."""
    from paper_2407_19977_amd import scenes
    out = []
    for ids in np.array_split(np.arange(mesh.n_triangles), parts):
        used, inv = np.unique(mesh.indices[ids], return_inverse=True)
        out.append(scenes.Mesh(np.ascontiguousarray(mesh.vertices[used]), inv.reshape(-1, 3).astype(np.int32),
                               np.ascontiguousarray(mesh.material_ids[ids])))
    return out


@pytest.mark.parametrize("which,parts", [("cornell", 1), ("cornell", 7), ("spheres", 1), ("spheres", 3), ("spheres", 200),
                                         ("material_zoo", 5)])
def test_device_gather_equals_host_build(which, parts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gather] {which} in {parts}", flush=True)
    from paper_2407_19977_amd import pt, scenes
    sc = getattr(scenes, which)()
    assert not sc.instances
    meshes = [p for m in sc.meshes for p in (_split(m, parts) if parts > 1 else [m])]
    cam = sc.with_camera(width=96, height=64).camera
    res = []
    for dev in (False, True):
        s = pt.scene_from(sc, device=0)
        try:
            s.build_bvh(meshes, on_device=dev)
            out = torch.empty((64, 96, 3), dtype=torch.float32, device="cuda:0")
            s.render(cam, 3, 5, 9, out)
            # another material table: the lights follow it
            mats = np.asarray(sc.materials, np.float32).reshape(-1, 39).copy()
            s.upload_materials(mats[::-1].copy())
            out2 = torch.empty_like(out)
            s.render(cam, 2, 5, 9, out2)
            res.append((out.cpu(), out2.cpu()))
        finally:
            s.close()
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("parts", [1, 6])
@pytest.mark.parametrize("fault", ["index", "low_index", "nan", "inf_unused", "material"])
def test_refused_meshes_leave_the_scene(parts, fault):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[refuse] {fault} in {parts}", flush=True)
    from paper_2407_19977_amd import pt, scenes
    sc = scenes.cornell()
    s = pt.scene_from(sc, device=0)
    try:
        cam = sc.with_camera(width=32, height=32).camera
        before, after = (torch.empty((32, 32, 3), dtype=torch.float32, device="cuda:0") for _ in range(2))
        s.render(cam, 2, 4, 1, before)
        meshes = _split(sc.meshes[0], parts)
        m = meshes[-1]
        v, ix, mid = m.vertices.copy(), m.indices.copy(), m.material_ids.copy()
        if fault == "index":
            ix[-1, 2] = len(v)
        elif fault == "low_index":
            ix[0, 1] = -1
        elif fault == "nan":
            v[0, 1] = np.nan
        elif fault == "inf_unused":
            v = np.concatenate([v, np.full((1, 3), np.inf, np.float32)])
        else:
            mid[0] = -3
        meshes[-1] = scenes.Mesh(v, ix, mid)
        said = []
        for dev in (False, True):
            with pytest.raises(Exception) as e:
                s.build_bvh(meshes, on_device=dev)
            said.append(str(e.value))
        assert said[0] == said[1]
        s.render(cam, 2, 4, 1, after)
        assert torch.equal(before, after)
    finally:
        s.close()


@pytest.mark.parametrize("parts", [1, 3, 40])
@pytest.mark.parametrize("fault", ["index", "low_index", "nan", "inf_unused", "material"])
def test_refused_large_meshes(parts, fault):
    """Builds of 2000 triangles and more are checked on the device: refused with the host build's words,
    and a mesh of 1999 or 2000 triangles gives the host build's hits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[refuse] {fault} in {parts}, large", flush=True)
    from paper_2407_19977_amd import pt, scenes
    sc = scenes.spheres(level=2, env_size=(64, 32))
    meshes = _split(sc.meshes[0], parts)
    assert sum(m.n_triangles for m in meshes) > 2000
    s = pt.PtScene(0)
    try:
        m = meshes[-1]
        v, ix, mid = m.vertices.copy(), m.indices.copy(), m.material_ids.copy()
        if fault == "index":
            ix[-1, 2] = len(v)
        elif fault == "low_index":
            ix[0, 1] = -1
        elif fault == "nan":
            v[0, 1] = np.nan
        elif fault == "inf_unused":
            v = np.concatenate([v, np.full((1, 3), np.inf, np.float32)])
        else:
            mid[0] = -3
        said = []
        for dev in (False, True):
            with pytest.raises(Exception) as e:
                s.build_bvh(meshes[:-1] + [scenes.Mesh(v, ix, mid)], on_device=dev)
            said.append(str(e.value))
        assert said[0] == said[1] and f"mesh {parts - 1}" in said[0]
        r = np.random.default_rng(1)
        rays = np.zeros((2000, 8), np.float32)
        rays[:, 0:3], rays[:, 4:7] = r.uniform(-8, 8, (2000, 3)), r.normal(size=(2000, 3))
        rays[:, 3], rays[:, 7] = 1e-4, np.inf
        rays = torch.from_numpy(rays).to("cuda:0")
        m = sc.meshes[0]
        for n in (1999, 2000):
            part = [scenes.Mesh(m.vertices, m.indices[:n], m.material_ids[:n])]
            hits = []
            for dev in (False, True):
                s.build_bvh(part, on_device=dev)
                hits.append(s.trace_closest(rays, torch.empty((2000, 6), dtype=torch.int32, device="cuda:0")).clone())
            assert torch.equal(hits[0], hits[1]) and int(hits[0][:, 5].sum()) > 10
    finally:
        s.close()
