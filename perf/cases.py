"""The work that users of this path tracer have it do, as timed cases.

A case is one call (or one short sequence of calls) through the public Python
binding: a render of one of the repository's seeded scenes, progressive frames
with their display image, frames of the radiance cache, closest-hit queries, the
cache's network alone, and a rebuild of a deformed mesh's BVH on the device.
Sizes are the ones of this repository's own workloads (the box at 128x128 and
16 spp, the paper's 512x512 at 100 spp, the icosphere field and the instanced
scene at 1920x1080) and ranges around them.
"""
import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2407_19977_amd import pt, scenes

DEV = "cuda:0"


def listed():
    return [
        # the smallest scene as configured: a preview render, where launches and waits count
        {"name": "box_128", "kind": "render", "scene": "box", "level": 0, "w": 128, "h": 128, "spp": 16, "depth": 4},
        # every material class in one small odd-sized image: a material preview
        {"name": "zoo_101x67", "kind": "render", "scene": "zoo", "level": 0, "w": 101, "h": 67, "spp": 9, "depth": 6},
        # the shape of the paper's Table 2 at its middle level of detail
        {"name": "paper_512", "kind": "render", "scene": "field", "level": 3, "w": 512, "h": 512, "spp": 100,
         "depth": 5},
        # the flagship: a finished frame of the 1.31M-triangle field
        {"name": "field_1080p", "kind": "render", "scene": "field", "level": 5, "w": 1920, "h": 1080, "spp": 64,
         "depth": 8},
        # two-level scene with glass, long paths
        {"name": "instanced_1080p", "kind": "render", "scene": "instanced", "level": 0, "w": 1920, "h": 1080,
         "spp": 32, "depth": 12},
        # an interactive viewer: one sample per pixel and call, the tone-mapped image after every call
        {"name": "progressive_1080p", "kind": "progressive", "scene": "field", "level": 5, "w": 1920, "h": 1080,
         "frames": 4, "depth": 8},
        # the radiance cache trained from scratch while it renders
        {"name": "cache_1080p", "kind": "cache", "scene": "field", "level": 5, "w": 1920, "h": 1080, "frames": 8,
         "depth": 8},
        # a batch of incoherent visibility rays against the large mesh
        {"name": "rays_1m", "kind": "rays", "scene": "field", "level": 5, "n": 1 << 20},
        # a handful of picking rays: latency
        {"name": "rays_1000", "kind": "rays", "scene": "box", "level": 0, "n": 1000},
        # the cache's network alone: all queries of a frame, and one training batch's gradient
        {"name": "forward_2m", "kind": "forward", "n": (1 << 21) + 37},
        {"name": "gradient_16k", "kind": "gradient", "n": 1 << 14},
        # a deforming mesh: BVH rebuilt on the device, then queried
        {"name": "rebuild_field", "kind": "rebuild", "scene": "field", "level": 5, "n": 65536},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["render", "render", "render", "progressive", "cache", "rays", "forward", "gradient",
                       "rebuild"])
    case = {"kind": kind}
    if kind in ("render", "progressive", "cache", "rays"):
        case["scene"] = rng.choice(["field", "field", "instanced", "box", "zoo"])
        case["level"] = rng.randint(2, 5) if case["scene"] == "field" else 0
    if kind in ("render", "progressive", "cache"):
        case["w"], case["h"] = _log(rng, 48, 1920), _log(rng, 48, 1080)
        case["depth"] = rng.randint(3, 12)
    if kind == "render":
        case["spp"] = min(_log(rng, 1, 128), max(1, (1 << 25) // (case["w"] * case["h"])))
    elif kind in ("progressive", "cache"):
        case["frames"] = rng.randint(2, 8)
    elif kind == "rays":
        case["n"] = _log(rng, 1, 1 << 21)
    elif kind == "forward":
        case["n"] = _log(rng, 1, 1 << 21)
    elif kind == "gradient":
        case["n"] = _log(rng, 16, 1 << 16)
    else:
        case["scene"], case["level"], case["n"] = "field", rng.randint(2, 5), _log(rng, 64, 65536)
    return case


@functools.lru_cache(maxsize=None)
def _scene(name, level):
    if name == "box":
        return scenes.cornell()
    if name == "zoo":
        return scenes.material_zoo()
    if name == "instanced":
        return scenes.instanced()
    return scenes.spheres(level=level)


def _rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def _camera(sc, w, h, seed):
    """The scene's camera at another size, its eye moved a little: a user walking around the scene."""
    r = _rng(seed)
    eye, at = np.array(sc.camera.eye), np.array(sc.camera.look_at)
    d = eye - at
    if sc.name in ("spheres", "instanced"):
        a = r.uniform(-0.35, 0.35)
        d = np.array([d[0] * math.cos(a) + d[2] * math.sin(a), d[1], d[2] * math.cos(a) - d[0] * math.sin(a)])
        d *= r.uniform(0.95, 1.05)
    else:
        d = d + r.uniform(-0.08, 0.08, 3)
    return dataclasses.replace(sc.camera, eye=tuple(float(x) for x in at + d), width=w, height=h)


def _bounds(sc):
    """The box that rays start in: the meshes', or the instances' field with its lights."""
    if sc.name == "instanced":
        return np.array([-28.0, 0.1, -28.0]), np.array([28.0, 11.0, 28.0])
    if sc.name == "spheres":
        return np.array([-12.0, 0.1, -12.0]), np.array([12.0, 3.0, 12.0])
    return np.array([0.02, 0.02, 0.02]), np.array([0.98, 0.98, 0.98])


def _rays(sc, n, seed):
    """Rays from uniform points of the scene's box in uniform directions, [n][8]: origin, tmin, direction, tmax."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    lo, hi = (torch.tensor(v, dtype=torch.float32, device=DEV) for v in _bounds(sc))
    r = torch.empty((n, 8), dtype=torch.float32, device=DEV)
    r[:, 0:3] = lo + (hi - lo) * torch.rand((n, 3), generator=g, device=DEV)
    d = torch.randn((n, 3), generator=g, device=DEV)
    r[:, 4:7] = d / d.norm(dim=1, keepdim=True)
    r[:, 3] = 1e-4
    r[:, 7] = math.inf
    return r


def _network(n, seed):
    """Cache inputs as vertices give them (all in [0, 1]), targets, and trained-sized weights."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.rand((n, 12), generator=g, device=DEV)
    t = torch.rand((n, 3), generator=g, device=DEV) * 2.0
    w = (torch.rand(pt.NRC_PARAMS, generator=g, device=DEV) * 2.0 - 1.0) * math.sqrt(6.0 / 64.0)
    return x, t, w


def prepare(case, seed):
    st = {"case": case, "seed": seed}
    kind = case["kind"]
    if kind in ("forward", "gradient"):
        s = pt.PtScene(0)
        s.set_radiance_cache(pt.cache_config())
        st["x"], st["t"], st["w"] = _network(case["n"], seed)
        s.nrc_set_weights(st["w"])
        st["y"] = torch.empty((case["n"], 3), dtype=torch.float32, device=DEV)
        st["grad"] = torch.empty(pt.NRC_PARAMS, dtype=torch.float32, device=DEV)
        st["s"] = s
        return st
    sc = _scene(case["scene"], case["level"])
    if kind == "rebuild":
        # the mesh of this frame of a deformation: a smooth wave through the vertices
        p = _rng(seed).uniform(0.0, 2.0 * math.pi, 3).astype(np.float32)
        m = sc.meshes[0]
        v = m.vertices + np.float32(0.05) * np.sin(m.vertices[:, [1, 2, 0]] * np.float32(2.0) + p)
        st["meshes"] = [scenes.Mesh(np.ascontiguousarray(v), m.indices, m.material_ids)]
        st["s"] = pt.PtScene(0)
    else:
        st["s"] = pt.scene_from(sc, device=0)
    if kind in ("rays", "rebuild"):
        st["rays"] = _rays(sc, case["n"], seed)
        st["hits"] = torch.empty((case["n"], 6), dtype=torch.int32, device=DEV)
    else:
        w, h = case["w"], case["h"]
        st["cam"] = _camera(sc, w, h, seed)
        st["out"] = torch.empty((h, w, 3), dtype=torch.float32, device=DEV)
        if kind == "progressive":
            st["rgba8"] = [torch.empty((h, w, 4), dtype=torch.uint8, device=DEV) for _ in range(case["frames"])]
            st["sums"] = torch.empty((h, w, 3), dtype=torch.float64, device=DEV)
        if kind == "cache":
            st["weights"] = torch.empty(pt.NRC_PARAMS, dtype=torch.float32, device=DEV)
            st["config"] = pt.cache_config(init_seed=seed)
    return st


def run(st):
    case, s, kind = st["case"], st["s"], st["case"]["kind"]
    if kind == "render":
        s.render(st["cam"], case["spp"], case["depth"], st["seed"], st["out"])
        return st["out"]
    if kind == "progressive":
        s.reset_accumulation()
        for k in range(case["frames"]):
            s.accumulate(st["cam"], k, 1, case["depth"], st["seed"])
            s.display(rgba8=st["rgba8"][k])
        s.resolve(st["out"], st["sums"])
        return {"rgba8": st["rgba8"], "mean": st["out"], "sums": st["sums"]}
    if kind == "cache":
        s.set_radiance_cache(st["config"])
        s.render(st["cam"], case["frames"], case["depth"], st["seed"], st["out"])
        s.nrc_get_weights(st["weights"])
        return {"mean": st["out"], "weights": st["weights"]}
    if kind == "rays":
        s.trace_closest(st["rays"], st["hits"])
        return st["hits"]
    if kind == "rebuild":
        s.build_bvh(st["meshes"], on_device=True)
        s.trace_closest(st["rays"], st["hits"])
        return st["hits"]
    if kind == "forward":
        s.nrc_forward(st["x"], st["y"])
        return st["y"]
    loss = s.nrc_gradient(st["x"], st["t"], st["grad"])
    return {"grad": st["grad"], "loss": loss}


# rays (closest-hit and shadow) that one path sample of a scene takes at depth 8, measured with the
# library's ray counters, and the operations of one ray: about ten node steps of four boxes, three
# triangle tests and one vertex's shading
RAYS_PER_SAMPLE = {"box": 6.0, "zoo": 6.0, "field": 2.9, "instanced": 4.0}
FLOP_PER_RAY = 1000.0
NODE, TRI, RAY, HIT = 128, 48, 32, 24
NETWORK_MACS = 5 * 64 * 64 + 3 * 64


def work(case):
    kind = case["kind"]
    if kind == "forward":
        return {"bytes": case["n"] * (12 + 3) * 4.0, "flops": 2.0 * NETWORK_MACS * case["n"]}
    if kind == "gradient":
        return {"bytes": case["n"] * (12 + 3) * 4.0 + 4.0 * NETWORK_MACS, "flops": 6.0 * NETWORK_MACS * case["n"]}
    sc = _scene(case["scene"], case["level"])
    tris = sum(m.n_triangles for m in sc.meshes)
    scene_bytes = tris * (TRI + 0.25 * NODE) + (0 if sc.env is None else sc.env.shape[0] * sc.env.shape[1] * 16)
    if kind == "rays":
        return {"bytes": case["n"] * (RAY + HIT) + min(scene_bytes, case["n"] * 10.0 * NODE),
                "flops": case["n"] * FLOP_PER_RAY}
    if kind == "rebuild":
        m = sc.meshes[0]
        soup = m.vertices.nbytes + m.indices.nbytes + m.material_ids.nbytes
        return {"bytes": soup + tris * (TRI + 0.25 * NODE) + case["n"] * (RAY + HIT),
                "flops": tris * 200.0 + case["n"] * FLOP_PER_RAY}
    pixels = case["w"] * case["h"]
    samples = pixels * (case["spp"] if kind == "render" else case["frames"])
    flops = samples * RAYS_PER_SAMPLE[case["scene"]] * min(1.0, case["depth"] / 8.0) * FLOP_PER_RAY
    out = pixels * 12.0
    if kind == "progressive":
        out += pixels * (24.0 + 4.0 * case["frames"])
    if kind == "cache":
        flops += case["frames"] * 4 * (1 << 14) * 6.0 * NETWORK_MACS
    return {"bytes": scene_bytes + out, "flops": flops}


def _features(x):
    """The cache's 64-feature encoding of the 12 inputs, in 64 bits."""
    f = []
    for a in range(3):
        for k in range(6):
            f += [torch.sin(math.pi * x[:, a] * 2 ** k), torch.cos(math.pi * x[:, a] * 2 ** k)]

    def blob(s, i, periodic=False):
        d = s - (i + 0.5) * 0.25
        if periodic:
            d = d - torch.floor(d + 0.5)
        return torch.exp(-0.5 * (4.0 * d) ** 2)

    for c in range(4):
        f += [blob(x[:, 3 + c], i, c % 2 == 1) for i in range(4)]
    f += [blob(1.0 - torch.exp(-x[:, 7]), i) for i in range(4)]
    f += [x[:, 8 + i] for i in range(4)]
    f += [torch.ones_like(x[:, 0])] + [torch.zeros_like(x[:, 0])] * 3
    return torch.stack(f, 1)


def _mlp(w, x):
    a = _features(x)
    for l in range(5):
        a = torch.relu(a @ w[l * 4096:(l + 1) * 4096].view(64, 64).t())
    return a @ w[5 * 4096:].view(3, 64).t()


def exact(case, seed):
    """The network's outputs and its loss gradient in 64 bits.  Images, hits and trained weights have no
    other value than the estimator's own: a different path is another sample of the same integral, and
    hits are compared word by word."""
    if case["kind"] not in ("forward", "gradient"):
        return None
    x, t, w = (v.double() for v in _network(case["n"], seed))
    if case["kind"] == "forward":
        return torch.cat([_mlp(w, part) for part in x.split(1 << 18)])
    w.requires_grad_(True)
    y = _mlp(w, x)
    loss = ((y - t) ** 2 / (y.detach() ** 2 + 0.01)).mean()
    loss.backward()
    return {"grad": w.grad, "loss": float(loss.detach())}
