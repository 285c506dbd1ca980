"""Four lanes per ray (small passes): the per-lane kernels' hits, masks and visibility bit for bit, at partial tiles and
waves, every sample grid and light count, both triangle tests, trees with short and deep stacks."""
import dataclasses

import numpy as np
import pytest

from paper_2410_05095_amd import scenegen as sg

pytestmark = pytest.mark.gpu


def scenes():
    from tests.test_gpu_render import deep_scene
    one = deep_scene(0)   # two triangles: the root holds a leaf only
    return [one, deep_scene(40), sg.city_scene(0, n_instances=60, width=96, height=54)]


@pytest.mark.parametrize("watertight", [False, True])
@pytest.mark.parametrize("two_level", [False, True])
def test_equals_the_per_lane_kernels(watertight, two_level):
    import torch
    from paper_2410_05095_amd import _native as N
    ctx = N.Context(0)
    rng = np.random.default_rng(4)
    for scene in scenes():
        gs = ctx.scene_from(scene).build(watertight=watertight, two_level=two_level)
        assert gs.stats()["max_stack"] <= 128
        lights = np.concatenate([rng.uniform((-3, 1, -3), (3, 9, 3), (5, 3)), np.ones((5, 3))], 1).astype(np.float32)
        for (w, h, ssaa) in ((1, 1, 1), (8, 8, 1), (17, 9, 1), (33, 70, 1), (3, 5, 2), (20, 11, 2)):
            cam = dataclasses.replace(scene.cameras[0], width=w, height=h, ssaa=ssaa)
            runs = [dict(lights=lights[:n]) for n in (0, 1, 2, 5)]
            if ssaa == 1:
                runs += [dict(lights=lights[:1], rect=scene.rect_light, area_samples=n, area_stream=1) for n in (1, 5, 64)]
            for kw in runs:
                kw = dict(kw)
                li = kw.pop("lights")
                print(f"[quad] {scene.name} wt {watertight} {w}x{h}x{ssaa} lights {len(li)} {kw.get('area_samples')}", flush=True)
                outs = []
                for per_lane in (False, True):
                    outs.append(ctx.render(gs, cam, li, per_lane=per_lane, **kw))
                    torch.cuda.synchronize()
                    assert ctx.last_error() == 0
                for key in ("hit", "shadow", "visibility", "rgba"):
                    if outs[0].get(key) is not None:
                        assert torch.equal(outs[0][key], outs[1][key]), key
        gs.close()
    ctx.close()
