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
