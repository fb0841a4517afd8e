"""Closest-hit walk on rays at the edges of its box test (GPU).

The walk prunes with distances fma(plane, 1/d, -o/d), moved to the safe side,
and near and far planes chosen by the direction's signs.  Whatever the ray, the
hits must be the ones of testing every triangle, bit for bit: directions with
zero, negative-zero and tiny components, origins on box planes and far away,
negative and large tmin, finite tmax.
"""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _scene(which):
    from paper_2407_19977_amd import scenes
    if which == "box":
        return scenes.cornell()
    if which == "field":
        return scenes.spheres(level=2, env_size=(64, 32))
    sc = scenes.instanced(env_size=(64, 32))
    sc.instances = sc.instances[:12] + sc.instances[-2:]
    return sc


def _rays(sc, n, kind, seed):
    r = np.random.Generator(np.random.PCG64(seed))
    if sc.instances:
        verts = np.concatenate([i.object_to_world[:, :3] @ sc.meshes[i.mesh].vertices[::97].T
                                + i.object_to_world[:, 3:] for i in sc.instances[:-2]], 1).T
    else:
        verts = sc.meshes[0].vertices
    lo, hi = verts.min(0), verts.max(0)
    rays = np.zeros((n, 8), np.float32)
    target = verts[r.integers(0, len(verts), n)]
    o = r.uniform(lo, hi, (n, 3)) + r.normal(size=(n, 3)) * 0.3
    d = r.normal(size=(n, 3))
    rays[:, 3], rays[:, 7] = 1e-4, np.inf
    if kind == "axis":  # along one axis, through a vertex's coordinates: on the planes of the boxes around it
        ax = r.integers(0, 3, n)
        o = target.copy()
        o[np.arange(n), ax] += r.choice([-5.0, 5.0], n)
        d = np.where(r.uniform(size=(n, 3)) < 0.5, 0.0, -0.0)
        d[np.arange(n), ax] = np.sign(target[np.arange(n), ax] - o[np.arange(n), ax])
    elif kind == "plane":  # one zero component, aimed at a vertex
        ax = r.integers(0, 3, n)
        d = target - o
        o[np.arange(n), ax] = target[np.arange(n), ax]
        d[np.arange(n), ax] = r.choice([0.0, -0.0], n)
    elif kind == "tiny":  # denormal and very small components
        d = target - o
        k = r.integers(0, 3, n)
        d[np.arange(n), k] = r.choice([1e-45, -1e-40, 1e-38, -1e-31, 1e-30, 1e-20], n)
    elif kind == "far":  # from far away
        d = r.normal(size=(n, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        o = target - d * r.choice([100.0, 1e4], (n, 1))
    elif kind == "range":  # negative and large tmin, finite tmax
        d = target - o
        rays[:, 3] = r.choice([-2.0, -0.1, 0.0, 0.9], n)
        rays[:, 7] = r.choice([0.5, 1.0, 1.5, np.inf], n)
    rays[:, 0:3], rays[:, 4:7] = o, d
    return rays


@pytest.mark.parametrize("kind", ["axis", "plane", "tiny", "far", "range"])
@pytest.mark.parametrize("which", ["box", "field", "instanced"])
def test_hits_equal_brute_force(which, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_19977_amd import pt
    print(f"[walk] {which} {kind}", flush=True)
    sc = _scene(which)
    n = 3000 if which != "instanced" else 1200
    rays = torch.from_numpy(_rays(sc, n, kind, 17)).to("cuda:0")
    s = pt.scene_from(sc, device=0)
    a = torch.empty((n, 6), dtype=torch.int32, device="cuda:0")
    b = torch.empty_like(a)
    s.trace_closest(rays, a)
    s.trace_closest(rays, b, brute_force=True)
    s.close()
    assert int(b[:, 5].sum()) > n // 10, "too few rays hit to tell anything"
    bad = torch.nonzero((a != b).any(1)).ravel()
    assert len(bad) == 0, f"{len(bad)} of {n} rays differ, first {bad[:5].tolist()}: {rays[bad[:2]].tolist()}"


@pytest.mark.parametrize("kind", ["axis", "plane", "spread", "far"])
@pytest.mark.parametrize("which", ["box", "field", "instanced"])
def test_short_directions_equal_brute_force(which, kind):
    """Directions of any length, down to about 2^-104: the walk's margins have to follow the largest
    component (t grows as it shrinks), and small components may be far below it or below 2^-100."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_19977_amd import pt
    print(f"[walk] {which} short {kind}", flush=True)
    sc = _scene(which)
    n = 3000 if which != "instanced" else 1200
    rays = _rays(sc, n, "tiny" if kind == "spread" else kind, 23)
    r = np.random.Generator(np.random.PCG64(29))
    d = rays[:, 4:7].astype(np.float64)
    if kind == "spread":  # one component a factor of up to 2^12 below the rest, beside denormal ones
        d[np.arange(n), r.integers(0, 3, n)] *= 2.0 ** -r.integers(0, 12, n)
    rays[:, 4:7] = d * 2.0 ** r.choice([-20, -41, -60, -78, -92, -104], (n, 1))
    rays = torch.from_numpy(rays).to("cuda:0")
    s = pt.scene_from(sc, device=0)
    a = torch.empty((n, 6), dtype=torch.int32, device="cuda:0")
    b = torch.empty_like(a)
    s.trace_closest(rays, a)
    s.trace_closest(rays, b, brute_force=True)
    s.close()
    assert int(b[:, 5].sum()) > n // 10, "too few rays hit to tell anything"
    bad = torch.nonzero((a != b).any(1)).ravel()
    assert len(bad) == 0, f"{len(bad)} of {n} rays differ, first {bad[:5].tolist()}: {rays[bad[:2]].tolist()}"


def test_walk_with_64_bit_node_addresses():
    """Node arrays of 4 GiB and more (here 33.6M triangles, whose device build reserves a node each) are
    walked with 64-bit addresses: hits equal the ones of testing every triangle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_19977_amd import pt, scenes
    n = 4098  # grid of n x n vertices, two triangles a cell
    print(f"[walk] height field of {2 * (n - 1) ** 2} triangles", flush=True)
    x, z = np.meshgrid(np.linspace(-1, 1, n, dtype=np.float32), np.linspace(-1, 1, n, dtype=np.float32))
    v = np.stack([x, np.float32(0.1) * np.sin(9 * x) * np.cos(7 * z), z], -1).reshape(-1, 3)
    c = (np.arange(n - 1, dtype=np.int32)[:, None] * n + np.arange(n - 1, dtype=np.int32)[None, :]).reshape(-1)
    f = np.concatenate([np.stack([c, c + n, c + 1], 1), np.stack([c + 1, c + n, c + n + 1], 1)])
    assert 128 * (len(f) - 1) > 2 ** 32
    s = pt.PtScene(0)
    s.build_bvh([scenes.Mesh(v, f, np.zeros(len(f), np.int32))], on_device=True)
    r = np.random.Generator(np.random.PCG64(3))
    rays = np.zeros((256, 8), np.float32)
    rays[:, 0:3] = r.uniform([-1, 0.2, -1], [1, 0.5, 1], (256, 3))
    rays[:, 4:7] = r.uniform([-1, -1, -1], [1, 0, 1], (256, 3))
    rays[:, 3], rays[:, 7] = 1e-4, np.inf
    rays = torch.from_numpy(rays).to("cuda:0")
    a = torch.empty((256, 6), dtype=torch.int32, device="cuda:0")
    b = torch.empty_like(a)
    s.trace_closest(rays, a)
    s.trace_closest(rays, b, brute_force=True)
    s.close()
    assert int(b[:, 5].sum()) > 100 and torch.equal(a, b)
