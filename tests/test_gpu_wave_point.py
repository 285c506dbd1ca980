"""Wave-uniform point-light shadow rays towards lights amid the geometry: the per-lane kernel's masks, and a walk
of the order of the rays' own paths."""
import numpy as np
import pytest

from paper_2410_05095_amd import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,w,h,ssaa", [(0, 96, 54, 1), (1, 45, 31, 2)])
def test_lights_amid_the_geometry(seed, w, h, ssaa):
    import torch
    from paper_2410_05095_amd import _native as N
    scene = sg.city_scene(seed, n_instances=120, width=w, height=h, ssaa=ssaa)
    # lights among the bodies (y 0..20), so that most of the scene lies beyond them
    rng = np.random.default_rng(seed)
    lights = np.concatenate([rng.uniform((-6, 4, -6), (6, 16, 6), (4, 3)), np.full((4, 3), 50.0)], 1).astype(np.float32)
    ctx = N.Context(0)
    gs = ctx.scene_from(scene).build(device_sah=True)
    got = {}
    for wave in (True, False):
        print(f"[wave_point] seed {seed} {w}x{h}x{ssaa} wave {wave}", flush=True)
        out = ctx.render(gs, scene.cameras[0], lights, wave=wave, per_lane=not wave, count=True)
        torch.cuda.synchronize()
        assert ctx.last_error() == 0
        got[wave] = (out["shadow"].clone(), ctx.stage_times()["shadow_nodes"])
    assert torch.equal(got[True][0], got[False][0])
    # a wave visits the union of its 64 rays' paths: a few times a ray's own at this resolution, where a walk
    # that accepted boxes beyond the light would visit a large part of the 50,000-node tree
    assert got[True][1] <= 16 * got[False][1], (got[True][1], got[False][1])
    gs.close()
    ctx.close()


def test_batch_wave_pass_equals_per_lane():
    """The batch's wave-uniform shadow pass forced on views below its size (odd sizes, both sample grids, a view
    without lights, trees of one and two stack registers), eager and replayed: the masks of the per-lane pass."""
    import ctypes as C
    import torch
    from paper_2410_05095_amd import _native as N
    from tests.test_gpu_batch import small_batch
    from tests.test_gpu_render import deep_scene
    ctx = N.Context(0)
    scenes, cams = small_batch()
    deep = deep_scene()
    scenes.append(deep)
    cams.append([sg.Camera(**{**deep.cameras[0].__dict__, "width": 33, "height": 19, "ssaa": 2})])
    handles = [ctx.scene_from(sc).build() for sc in scenes]
    rng = np.random.default_rng(3)
    lights, views = [], []
    for si, sc in enumerate(scenes):
        lf = len(lights)
        ls = sc.point_lights.tolist() if si < 3 else np.concatenate([rng.uniform(-3, 9, (2, 3)), np.ones((2, 3))], 1).tolist()
        lights.extend(ls)
        views += [(si, cam, lf, len(ls)) for cam in cams[si]]
    lights = np.asarray(lights, np.float32).reshape(-1, 6)
    assert any(v[3] == 0 for v in views)
    for n_scenes in (3, 4):      # without and with the deep tree
        vs = [v for v in views if v[0] < n_scenes]
        hs = handles[:n_scenes]
        print(f"[wave_point] batch of {len(vs)} views, max stack {max(h.stats()['max_stack'] for h in hs)}", flush=True)
        ref = ctx.render_batch(hs, vs, lights)
        torch.cuda.synchronize()
        outs = [{} for _ in vs]
        sarr, varr = ctx._batch_args(hs, vs, outs)
        arr = N.light_array(lights)
        for flags in (N.RC_FLAG_WAVE, N.RC_FLAG_WAVE | N.RC_FLAG_COUNT, N.RC_FLAG_WAVE | N.RC_FLAG_GRAPH,
                      N.RC_FLAG_WAVE | N.RC_FLAG_GRAPH):
            for o in outs:
                for t in o.values():
                    if t is not None:
                        t.fill_(-1)
            N.check(N.lib().rc_render_batch(ctx.h, sarr, len(hs), varr, len(vs), arr, len(lights), None, flags), "batch")
            torch.cuda.synchronize()
            assert ctx.last_error() == 0
            for i, (a, b) in enumerate(zip(outs, ref)):
                for k in ("hit", "shadow", "rgba"):
                    assert (a[k] is None and b[k] is None) or torch.equal(a[k], b[k]), (flags, i, k)
    for h in handles:
        h.close()
    ctx.close()
