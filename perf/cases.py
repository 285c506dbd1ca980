"""Workloads of the ray-cast renderer and of its shadow denoiser, through the package's public entry points.

listed() holds the cases that stand for the work a user has the library do, draw() more of the same ranges;
prepare() makes what a program holds before the call (scene handles, cameras, lights, output buffers, network
weights), run() is one pass, work() the bytes and operations that the pass cannot do without, and exact() the
64-bit value of its computed numbers where a plain tensor program gives it.
"""
import functools
import math

import numpy as np
import torch

from paper_2410_05095_amd import _native as N
from paper_2410_05095_amd import denoise as D
from paper_2410_05095_amd import scenegen as sg

DEV = "cuda:0"


def listed():
    return [
        # the smallest frame: a 1292-triangle room with one lamp, where launches and latency count
        {"name": "tiny_room_128", "kind": "room", "w": 128, "h": 128},
        # the interactive frame: 300 of 1500 bodies moved, tree refit, one camera and one hard-shadow ray per pixel
        {"name": "moving_hard_1080p", "kind": "point", "tris": 7300000, "bodies": 1500, "w": 1920, "h": 1080, "ssaa": 1,
         "lights": 1, "tree": "sah", "moving": 300, "normals": False, "watertight": False},
        # the anti-aliased still: 2x2 samples, four lights, smooth normals
        {"name": "ssaa_4lights_1080p", "kind": "point", "tris": 1130000, "bodies": 400, "w": 1920, "h": 1080, "ssaa": 2,
         "lights": 4, "tree": "sah", "moving": 0, "normals": True, "watertight": False},
        # the plain soft-shadow frame: 64 light samples per pixel
        {"name": "soft64_1080p", "kind": "rect", "tris": 7300000, "bodies": 1500, "w": 1920, "h": 1080, "samples": 64,
         "tree": "sah", "moving": 0, "watertight": False, "features": False},
        # the learned path's input: one light sample per pixel and the network's features, shaded later
        {"name": "soft1_features_1080p", "kind": "rect", "tris": 2000000, "bodies": 400, "w": 1920, "h": 1080,
         "samples": 1, "tree": "sah", "moving": 0, "watertight": False, "features": True},
        # many small views of several scenes in one graph replay (data generation, multi-camera serving)
        {"name": "batch_64_views", "kind": "batch", "scale": 1.0, "views": 64, "ssaa": 1},
        # instances under a top level that is rebuilt every frame, a few light samples, 720p
        {"name": "two_level_soft8_720p", "kind": "rect", "tris": 1000000, "bodies": 300, "w": 1280, "h": 720,
         "samples": 8, "tree": "two", "moving": 100, "watertight": False, "features": False},
        # a scene whose topology changed: tree built on the GPU, then the frame that needs it
        {"name": "build_sah_1M", "kind": "build", "tris": 1000000, "bodies": 300, "w": 512, "h": 512, "method": "sah"},
        # the denoiser on one frame
        {"name": "denoise_1080p", "kind": "infer", "n": 1, "h": 1080, "w": 1920, "fp32": False},
        # one optimiser step on the benchmark's crops
        {"name": "train_8x512", "kind": "train", "n": 8, "h": 512, "w": 512},
        # the full-precision copy that the 16-bit network is checked against
        {"name": "denoise_fp32_540p", "kind": "infer", "n": 1, "h": 540, "w": 960, "fp32": True},
        # tone map, sRGB and FXAA of a finished frame
        {"name": "display_1080p", "kind": "post", "w": 1920, "h": 1080, "fxaa": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("room", "point", "point", "rect", "rect", "batch", "build", "infer", "infer", "train", "post"))
    if kind == "room":
        return {"kind": kind, "w": _log_int(rng, 16, 400), "h": _log_int(rng, 16, 400)}
    if kind in ("point", "rect"):
        tris = _log_int(rng, 20000, 2000000)
        bodies = max(4, tris // rng.randint(2500, 5000))
        two = rng.random() < 0.25
        c = {"kind": kind, "tris": tris, "bodies": bodies, "w": _log_int(rng, 100, 1920), "h": _log_int(rng, 100, 1080),
             "tree": "two" if two else rng.choice(("sah", "sah", "lbvh")),
             "moving": max(1, bodies // 4) if two or rng.random() < 0.4 else 0, "watertight": rng.random() < 0.2}
        if kind == "point":
            c.update(ssaa=rng.choice((1, 2)), lights=rng.randint(1, 4), normals=rng.random() < 0.4)
        else:
            c.update(samples=_log_int(rng, 1, 64), features=rng.random() < 0.4)
        return c
    if kind == "batch":
        return {"kind": kind, "scale": round(rng.uniform(0.1, 0.5), 3), "views": rng.randint(5, 48), "ssaa": rng.choice((1, 1, 2))}
    if kind == "build":
        tris = _log_int(rng, 10000, 1000000)
        return {"kind": kind, "tris": tris, "bodies": max(4, tris // 3500), "w": _log_int(rng, 64, 512),
                "h": _log_int(rng, 64, 512), "method": rng.choice(("sah", "lbvh", "two"))}
    if kind == "infer":
        fp32 = rng.random() < 0.4
        return {"kind": kind, "n": rng.randint(1, 3), "h": 4 * _log_int(rng, 8, 135 if fp32 else 200),
                "w": 4 * _log_int(rng, 8, 160 if fp32 else 220), "fp32": fp32}
    if kind == "train":
        return {"kind": kind, "n": rng.randint(1, 8), "h": 4 * _log_int(rng, 8, 128), "w": 4 * _log_int(rng, 8, 128)}
    return {"kind": kind, "w": _log_int(rng, 30, 2600), "h": _log_int(rng, 30, 1500), "fxaa": rng.random() < 0.7}


# ------------------------------------------------------------------ scenes

@functools.lru_cache(maxsize=4096)
def _mesh(kind, target):
    """Unit-size sphere, box or torus of about `target` triangles: (vertices float64, faces uint32)."""
    if kind == "box":
        n = max(1, int(round(math.sqrt(target / 12.0))))
        g = np.linspace(-1.0, 1.0, n + 1)
        a, b = np.meshgrid(g, g, indexing="ij")
        v = []
        for axis in range(3):
            for sign in (-1.0, 1.0):
                p = np.empty((n + 1, n + 1, 3))
                ta, tb = ((axis + 1) % 3, (axis + 2) % 3) if sign > 0 else ((axis + 2) % 3, (axis + 1) % 3)
                p[..., axis], p[..., ta], p[..., tb] = sign, a, b
                v.append(p.reshape(-1, 3))
        i, j = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
        q = (i * (n + 1) + j).reshape(-1)
        f = np.concatenate([np.stack([q, q + n + 1, q + n + 2], 1), np.stack([q, q + n + 2, q + 1], 1)])
        f = np.concatenate([f + s * (n + 1) * (n + 1) for s in range(6)])
        return np.concatenate(v), f.astype(np.uint32)
    n = max(3, int(round(math.sqrt(target / 4.0))))
    if kind == "sphere":
        n_lat, n_lon = n, 2 * n
        th, ph = np.meshgrid(np.pi * np.arange(n_lat + 1) / n_lat, 2 * np.pi * np.arange(n_lon) / n_lon, indexing="ij")
        v = np.stack([np.sin(th) * np.cos(ph), np.cos(th), np.sin(th) * np.sin(ph)], -1).reshape(-1, 3)
        i, j = np.meshgrid(np.arange(n_lat), np.arange(n_lon), indexing="ij")
        a, b = i * n_lon + j, i * n_lon + (j + 1) % n_lon
        c, d = a + n_lon, b + n_lon
        f = np.concatenate([np.stack([a, b, d], -1)[1:].reshape(-1, 3), np.stack([a, d, c], -1)[:-1].reshape(-1, 3)])
        return v, f.astype(np.uint32)
    n_u, n_v, minor = 2 * n, n, 0.3
    u, w = np.meshgrid(2 * np.pi * np.arange(n_u) / n_u, 2 * np.pi * np.arange(n_v) / n_v, indexing="ij")
    r = 1.0 + minor * np.cos(w)
    v = np.stack([r * np.cos(u), minor * np.sin(w), r * np.sin(u)], -1).reshape(-1, 3)
    i, j = np.meshgrid(np.arange(n_u), np.arange(n_v), indexing="ij")
    a, b = i * n_v + j, (i + 1) % n_u * n_v + j
    c, d = (i + 1) % n_u * n_v + (j + 1) % n_v, i * n_v + (j + 1) % n_v
    f = np.concatenate([np.stack([a, d, c], -1).reshape(-1, 3), np.stack([a, c, b], -1).reshape(-1, 3)])
    return v, f.astype(np.uint32)


def _scene(rng, tris, bodies, lights=0):
    """Rigid bodies (spheres, boxes, tori of unequal triangle counts, 0.2-1 m) in a 20 m block over a ground."""
    counts = np.exp(rng.uniform(math.log(2000.0), math.log(10000.0), bodies))
    counts = np.maximum(12, counts * (tris / counts.sum())).astype(np.int64)
    gv, gf = sg.ground_plane(20.0)
    verts, faces, vr, tr, owner = [gv], [gf.astype(np.uint32)], [(0, 4)], [(0, 2)], [0, 0]
    nv, nt = 4, 2
    kinds = rng.integers(0, 3, bodies)
    sizes = rng.uniform(0.2, 1.0, bodies)
    places = rng.uniform((-10.0, 0.0, -10.0), (10.0, 20.0, 10.0), (bodies, 3))
    for b in range(bodies):
        v, f = _mesh(sg.KINDS[int(kinds[b])], int(counts[b]))
        verts.append(v @ (sizes[b] * sg.random_rotation(rng).T) + places[b])
        faces.append(f + np.uint32(nv))
        vr.append((nv, len(v)))
        tr.append((nt, len(f)))
        nv += len(v)
        nt += len(f)
    tr = np.asarray(tr, np.uint32)
    mats = np.stack([sg.random_material(rng) for _ in range(bodies + 1)]).astype(np.float32)
    return sg.Scene(positions=np.concatenate(verts).astype(np.float32), indices=np.concatenate(faces),
                    tri_material=np.repeat(np.arange(bodies + 1, dtype=np.uint32), tr[:, 1]), materials=mats,
                    body_vertex_range=np.asarray(vr, np.uint32), body_tri_range=tr,
                    point_lights=np.asarray(sg.random_point_lights(rng, lights), np.float32).reshape(-1, 6),
                    rect_light=sg.DEFAULT_RECT, cameras=[], name="bodies")


def _normals(scene):
    """Area-weighted vertex normals, summed by vertex with bincount."""
    p, f = scene.positions.astype(np.float64), scene.indices.astype(np.int64)
    fn = np.cross(p[f[:, 1]] - p[f[:, 0]], p[f[:, 2]] - p[f[:, 0]])
    acc = np.stack([np.bincount(f.reshape(-1), np.repeat(fn[:, k], 3), len(p)) for k in range(3)], 1)
    ln = np.linalg.norm(acc, axis=1, keepdims=True)
    return np.where(ln > 0, acc / np.where(ln > 0, ln, 1.0), (0.0, 1.0, 0.0)).astype(np.float32)


def _camera(rng, c, ssaa=1):
    eye = np.array((0.0, 10.0, -28.0)) + rng.uniform(-2.0, 2.0, 3)
    return sg.Camera(eye=tuple(float(x) for x in eye), target=(0.0, 5.0, 0.0), up=(0.0, 1.0, 0.0), vfov_deg=50.0,
                     width=c["w"], height=c["h"], ssaa=ssaa, seed=int(rng.integers(1 << 31)), frame=0)


def _room(c, seed):
    """The closed box around a sphere, with its camera and lamp a little elsewhere for each seed."""
    rng = np.random.default_rng(seed)
    sc = sg.tiny_box_scene(int(rng.integers(1 << 20)), c["w"], c["h"])
    move = lambda p, r: tuple(float(x) for x in np.asarray(p) + rng.uniform(-r, r, 3))  # noqa: E731
    base = sc.cameras[0]
    cam = sg.Camera(eye=move(base.eye, 0.04), target=move(base.target, 0.05), up=base.up, vfov_deg=75.0, width=c["w"],
                    height=c["h"], ssaa=1, seed=base.seed)
    light = np.concatenate([np.asarray((0.0, 0.42, 0.0)) + rng.uniform(-0.05, 0.05, 3), np.ones(3)]).astype(np.float32)
    return sc, cam, light.reshape(1, 6)


# ------------------------------------------------------------------ the denoiser's inputs

_LAYERS = ((8, 32), (32, 32), (32, 64), (64, 64), (64, 128), (128, 128), (192, 64), (64, 64), (96, 32), (32, 32))


def _params(seed):
    """He-normal weights with small biases, in the library's parameter order."""
    rng = np.random.default_rng(seed)
    p = []
    for cin, cout in _LAYERS:
        p += [rng.normal(0.0, math.sqrt(2.0 / (9 * cin)), cout * 9 * cin), rng.normal(0.0, 0.02, cout)]
    p += [rng.normal(0.0, math.sqrt(1.0 / 32), 32), rng.normal(0.0, 0.02, 1)]
    return np.concatenate(p).astype(np.float32)


def _features(c, seed):
    """Noisy 0/1 visibility, smooth log depth, unit normals and albedo in patches; a tenth of it background."""
    g = torch.Generator(DEV).manual_seed(seed)
    n, h, w = c["n"], c["h"], c["w"]

    def field(channels, cells):
        small = torch.rand((n, channels, max(2, h // cells), max(2, w // cells)), generator=g, device=DEV)
        return torch.nn.functional.interpolate(small, (h, w), mode="bilinear", align_corners=False).permute(0, 2, 3, 1)

    lit = field(1, 48)
    lit = ((lit - 0.5) * 6 + 0.5).clamp(0, 1)                     # the many-sample visibility
    vis = (torch.rand(lit.shape, generator=g, device=DEV) < lit).float()
    nrm = torch.nn.functional.normalize(field(3, 32) - 0.5, dim=-1)
    feat = torch.cat([vis, 0.4 + 0.4 * field(1, 64), nrm, 0.2 + 0.7 * field(3, 24)], -1)
    hit = field(1, 96) > 0.3
    back = torch.tensor([1.0, 1, 0, 0, 0, 0, 0, 0], device=DEV)
    feat = torch.where(hit, feat, back).to(torch.bfloat16).contiguous()
    return feat, lit[..., 0].contiguous(), hit[..., 0].float().contiguous()


# ------------------------------------------------------------------ prepare / run

def prepare(case, seed):
    c, kind = case, case["kind"]
    rng = np.random.default_rng([seed, 17])
    ctx = N.Context(0)
    s = {"case": c, "ctx": ctx}
    if kind == "room":
        sc, s["cam"], s["lights"] = _room(c, seed)
        s["gs"] = ctx.scene_from(sc).build()
        s["out"] = {}
    elif kind in ("point", "rect"):
        sc = _scene(rng, c["tris"], c["bodies"], c.get("lights", 0))
        if c.get("normals"):
            sc.normals = _normals(sc)
        gs = ctx.scene_from(sc)
        gs.build(two_level=c["tree"] == "two", device=c["tree"] == "lbvh", device_sah=c["tree"] == "sah",
                 watertight=c["watertight"])
        s.update(gs=gs, cam=_camera(rng, c, c.get("ssaa", 1)), lights=sc.point_lights, rect=sc.rect_light, out={},
                 diag=D.scene_diagonal(sc), feat=None, frame=0)
        if c["moving"]:
            anim = sg.RigidAnimation(sc, c["moving"], seed=int(rng.integers(1 << 20)))
            s["ids"] = torch.from_numpy(anim.body_ids.astype(np.int32)).to(DEV)
            s["poses"] = [torch.from_numpy(anim.transforms(f)).to(DEV) for f in (1, 2)]
    elif kind == "batch":
        handles, views, lights, scenes = [], [], [], []
        for n_inst in (36, 182, 364, 727):
            b = max(1, int(round(n_inst * c["scale"])))
            sc = _scene(rng, b * 2750, b, int(rng.integers(1, 5)))
            handles.append(ctx.scene_from(sc).build(device_sah=True))
            scenes.append((len(lights), len(sc.point_lights)))
            lights.extend(sc.point_lights.tolist())
        cams = sg.orbit_cameras(rng, c["views"], seed=int(rng.integers(1 << 20)),
                                sizes=(256, 384, 512, 768, 1024) if c["ssaa"] == 1 else (101, 200, 256, 384))
        order = np.random.default_rng(7).integers(0, 5 if c["ssaa"] == 1 else 4, c["views"])
        side = ((256, 384, 512, 768, 1024) if c["ssaa"] == 1 else (101, 200, 256, 384))
        for i, cam in enumerate(cams):
            cam.width = cam.height = side[int(order[i])]      # the same sizes for every seed
            cam.ssaa = c["ssaa"]
            views.append((i % 4, cam, *scenes[i % 4]))
        s.update(handles=handles, views=views, lights=np.asarray(lights, np.float32).reshape(-1, 6),
                 outs=[{} for _ in views])
    elif kind == "build":
        sc = _scene(rng, c["tris"], c["bodies"], 1)
        s.update(gs=ctx.scene_from(sc), cam=_camera(rng, c), lights=sc.point_lights, out={})
    elif kind in ("infer", "train"):
        s["den"] = N.Denoiser(ctx, seed=0)
        s["den"].set_params(_params(seed))
        s["feat"], s["target"], s["mask"] = _features(c, seed)
        if kind == "infer":
            s["y"] = torch.empty((c["n"], c["h"], c["w"]), dtype=torch.float32, device=DEV)
    elif kind == "post":
        g = torch.Generator(DEV).manual_seed(seed)
        h, w = c["h"], c["w"]
        # flat regions with hard edges, a smooth gradient and some highlights: linear HDR
        ids = torch.nn.functional.interpolate(torch.rand((1, 4, max(2, h // 23), max(2, w // 31)), generator=g, device=DEV),
                                              (h, w), mode="nearest")[0].permute(1, 2, 0)
        img = ids * ids * (0.3 + torch.rand((1, 1, 1), generator=g, device=DEV) + torch.linspace(0, 3, w, device=DEV)[None, :, None])
        img = img + 0.002 * torch.rand(img.shape, generator=g, device=DEV)
        img[..., 3] = (ids[..., 3] > 0.2).float()
        s["rgba"] = img.float().contiguous()
        s["out8"] = torch.empty((h, w, 4), dtype=torch.uint8, device=DEV)
    else:
        raise ValueError(kind)
    return s


def run(state):
    s, c, ctx = state, state["case"], state["ctx"]
    kind = c["kind"]
    if kind == "room":
        return ctx.render(s["gs"], s["cam"], s["lights"], out=s["out"])
    if kind in ("point", "rect"):
        if c["moving"]:
            s["gs"].set_transforms(s["poses"][s["frame"] & 1], s["ids"])
            s["gs"].refit()
            s["frame"] += 1
        if kind == "point":
            return ctx.render(s["gs"], s["cam"], s["lights"], out=s["out"])
        out = ctx.render(s["gs"], s["cam"], (), rect=s["rect"], area_samples=c["samples"], out=s["out"],
                         shade=not c["features"])
        if not c["features"]:
            return out
        s["feat"] = N.pack_features(ctx, s["gs"], s["cam"], out, s["diag"], feat=s["feat"])
        return {"hit": out["hit"], "visibility": out["visibility"], "features": s["feat"]}
    if kind == "batch":
        outs = ctx.render_batch(s["handles"], s["views"], s["lights"], graph=True, outs=s["outs"])
        # 21 views of three tensors each: as many outputs as are looked at
        return [{k: o[k] for k in ("rgba", "hit", "shadow")} for o in outs[:: max(1, -(-len(outs) // 21))]]
    if kind == "build":
        s["gs"].build(device_sah=c["method"] == "sah", device=c["method"] == "lbvh", two_level=c["method"] == "two")
        return ctx.render(s["gs"], s["cam"], s["lights"], out=s["out"])
    if kind == "infer":
        return s["den"].infer(s["feat"], out=s["y"], fp32=c["fp32"])
    if kind == "train":
        # a late step of the schedule: passes on the same state stay comparable
        loss = s["den"].train_step(s["feat"], s["target"], s["mask"], 1e-7)
        return {"loss": loss, "grads": s["den"].grads()}
    return ctx.postprocess(s["rgba"], fxaa=c["fxaa"], out=s["out8"])


# ------------------------------------------------------------------ work

# operations of one ray's own walk: 17.6 node visits of 52 and 7.3 triangle tests of 37 operations on the
# 7.3M-triangle frame, fewer visits on smaller trees (one 4-wide level less per factor of 4)
def _ray_ops(tris):
    return 52.0 * max(2.0, 17.6 - math.log(7.3e6 / max(tris, 4), 4)) + 37.0 * 7.3


def _net_flops(pixels):
    f = 0.0
    for (cin, cout), share in zip(_LAYERS, (1, 1, 4, 4, 16, 16, 4, 4, 1, 1)):
        f += 2.0 * 9 * cin * cout * pixels / share
    return f + 64.0 * pixels


def _batch_side(c):
    side = (256, 384, 512, 768, 1024) if c["ssaa"] == 1 else (101, 200, 256, 384)
    return [side[int(k)] for k in np.random.default_rng(7).integers(0, len(side), c["views"])]


def work(case):
    c, kind = case, case["kind"]
    if kind in ("room", "point", "rect", "build"):
        tris = c.get("tris", 1292)
        samples = c["w"] * c["h"] * c.get("ssaa", 1) ** 2
        per = c.get("lights", 1) if kind != "rect" else c["samples"]
        rays = samples * (1 + per)
        geo = 48.0 * min(tris, rays)                               # each triangle that is met, once
        out = samples * (16.0 + (4.0 if kind != "rect" else 0.0)) + c["w"] * c["h"] * (16.0 + (4.0 if kind == "rect" else 0.0))
        b = geo + out
        f = rays * _ray_ops(tris) + samples * 300.0
        if c.get("moving"):
            b += 24.0 * tris / 2 * c["moving"] / c["bodies"] + 48.0 * tris * c["moving"] / c["bodies"]
        if kind == "build":
            b += 36.0 * tris + 48.0 * tris + 128.0 * tris / 4
            f += 60.0 * tris * math.log(max(tris, 4), 2)
        return {"bytes": b, "flops": f}
    if kind == "batch":
        samples = sum(x * x for x in _batch_side(c)) * c["ssaa"] ** 2
        tris = 3.6e6 * c["scale"]
        return {"bytes": samples * 20.0 + samples / c["ssaa"] ** 2 * 16.0 + 48.0 * min(tris, samples),
                "flops": 3.5 * samples * _ray_ops(tris / 3) + samples * 600.0}
    if kind == "post":
        return {"bytes": c["w"] * c["h"] * 20.0, "flops": c["w"] * c["h"] * 60.0}
    pixels = c["n"] * c["h"] * c["w"]
    if kind == "infer":
        return {"bytes": pixels * 20.0 + 472993 * 2.0, "flops": _net_flops(pixels)}
    # the step keeps every activation for its backward: written once, read once
    acts = pixels * (32 * 4 + (64 * 4 + 32) / 4 + (64 + 256) / 16)
    return {"bytes": pixels * 24.0 + 4.0 * acts + 472993 * 28.0, "flops": 3.0 * _net_flops(pixels)}


# ------------------------------------------------------------------ 64-bit values

def _conv64(x, w, b):
    """3x3 convolution of (n, h, w, cin) in float64 as nine matrix products; w: (cout, 9, cin)."""
    n, h, wd, cin = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b.expand(n * h * wd, -1)
    for t in range(9):
        xs = p[:, t // 3:t // 3 + h, t % 3:t % 3 + wd].reshape(-1, cin)
        y = y + xs @ w[:, t].t().contiguous()
    return torch.relu(y).reshape(n, h, wd, -1)


def _net64(feat, p):
    """The U-Net in float64 from its parameter vector: visibility (n, h, w)."""
    o, ws = 0, []
    for cin, cout in _LAYERS:
        w = p[o:o + cout * 9 * cin].reshape(cout, 9, cin)
        o += cout * 9 * cin
        ws.append((w, p[o:o + cout]))
        o += cout
    pool = lambda t: (t[:, ::2, ::2] + t[:, 1::2, ::2] + t[:, ::2, 1::2] + t[:, 1::2, 1::2]) / 4  # noqa: E731
    up = lambda t: t.repeat_interleave(2, 1).repeat_interleave(2, 2)  # noqa: E731
    e1 = _conv64(_conv64(feat, *ws[0]), *ws[1])
    e2 = _conv64(_conv64(pool(e1), *ws[2]), *ws[3])
    bn = _conv64(_conv64(pool(e2), *ws[4]), *ws[5])
    d2 = _conv64(_conv64(torch.cat([up(bn), e2], -1), *ws[6]), *ws[7])
    d1 = _conv64(_conv64(torch.cat([up(d2), e1], -1), *ws[8]), *ws[9])
    return torch.sigmoid(d1 @ p[o:o + 32] + p[o + 32])


def _room64(case, seed):
    """Radiance of the room by brute force: every camera ray against every triangle, then every shadow ray."""
    sc, cam, lights = _room(case, seed)
    t64 = lambda a: torch.as_tensor(np.asarray(a, np.float32).astype(np.float64), device=DEV)  # noqa: E731
    unit = lambda v: v / v.norm(dim=-1, keepdim=True)  # noqa: E731
    tri = t64(sc.positions)[torch.from_numpy(sc.indices.astype(np.int64)).to(DEV)]
    a, e1, e2 = tri[:, 0], tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0]
    mats = t64(sc.materials)[torch.from_numpy(sc.tri_material.astype(np.int64)).to(DEV)]
    eye = t64(cam.eye)
    f = unit(t64(cam.target) - eye)
    r = unit(torch.linalg.cross(f, t64(cam.up)))
    u = torch.linalg.cross(r, f)
    th = math.tan(cam.vfov_deg * math.pi / 360.0)
    W, H = cam.width, cam.height
    px = ((torch.arange(W, device=DEV, dtype=torch.float64) + 0.5) * 2 / W - 1) * th * W / H
    py = (1 - (torch.arange(H, device=DEV, dtype=torch.float64) + 0.5) * 2 / H) * th
    d = unit((f + px[None, :, None] * r + py[:, None, None] * u).reshape(-1, 3))

    def cast(o, d, near, far):
        """First triangle with near < t < far for each ray: (t, index), t infinite where there is none."""
        best, which = [], []
        for i in range(0, len(d), 8192):
            oo, dd = o[i:i + 8192, None], d[i:i + 8192, None]
            pv = torch.linalg.cross(dd.expand(-1, len(a), -1), e2.expand(dd.shape[0], -1, -1))
            det = (pv * e1).sum(-1)
            s = oo - a
            q = torch.linalg.cross(s, e1.expand(dd.shape[0], -1, -1))
            bu, bv, t = (s * pv).sum(-1) / det, (q * dd).sum(-1) / det, (q * e2).sum(-1) / det
            ok = (bu >= 0) & (bv >= 0) & (bu + bv <= 1) & (t > near) & (t < far)
            m = torch.where(ok, t, torch.inf).min(1)
            best.append(m.values)
            which.append(m.indices)
        return torch.cat(best), torch.cat(which)

    t, k = cast(eye.expand(len(d), 3), d, 0.0, math.inf)
    hit = torch.isfinite(t)
    p = eye + torch.where(hit, t, 1.0)[:, None] * d
    n = unit(torch.linalg.cross(e1, e2))[k]
    n = torch.where((n * d).sum(-1, keepdim=True) > 0, -n, n)
    light = t64(lights)[0]
    os = p + n * 2.0 ** -18 * p.abs().amax(-1, keepdim=True).clamp(min=1.0)
    seg = light[:3] - os
    occ, _ = cast(os, seg, 0.0, 1.0)
    lit = hit & ((n * seg).sum(-1) > 0) & ~torch.isfinite(occ)
    wo, tl = -d, light[:3] - p
    wi, d2 = unit(tl), (tl * tl).sum(-1)
    h = unit(wo + wi)
    m = mats[k]
    rough, metal, alb = m[:, 3], m[:, 4], m[:, :3]
    no, ni, nh, ho = ((x * y).sum(-1) for x, y in ((n, wo), (n, wi), (n, h), (h, wo)))
    a2 = rough ** 4
    D_ = a2 / (math.pi * (nh * nh * (a2 - 1) + 1) ** 2)
    kk = (rough + 1) ** 2 / 8
    G = no / (no * (1 - kk) + kk) * ni / (ni * (1 - kk) + kk)
    f0 = 0.04 * (1 - metal)[:, None] + alb * metal[:, None]
    F = f0 + (1 - f0) * ((1 - ho) ** 5)[:, None]
    brdf = (1 - F) * (1 - metal)[:, None] * alb / math.pi + (D_ * G / (4 * no * ni))[:, None] * F
    on = lit & (no > 0) & (ni > 0)
    rgb = torch.where(on[:, None], brdf * light[3:] * (ni / d2)[:, None], 0.0)
    rgba = torch.cat([rgb, hit.double()[:, None]], 1).reshape(H, W, 4)
    return {"hit": None, "rgba": rgba, "shadow": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "room":
        return _room64(case, seed)
    if kind not in ("infer", "train"):
        return None                  # a traversal of a million triangles has no plain 64-bit program of seconds
    feat, target, mask = _features(case, seed)
    p = torch.from_numpy(_params(seed).astype(np.float64)).to(DEV)
    if kind == "infer":
        with torch.no_grad():
            return torch.cat([_net64(feat[i:i + 1].double(), p) for i in range(case["n"])])
    p.requires_grad_()
    total = mask.double().sum().clamp(min=1.0)
    loss = 0.0
    for i in range(case["n"]):
        y = _net64(feat[i:i + 1].double(), p)
        part = (mask[i:i + 1].double() * (y - target[i:i + 1].double()) ** 2).sum() / total
        part.backward()
        loss += float(part.detach())
    return {"grads": p.grad, "loss": loss}
