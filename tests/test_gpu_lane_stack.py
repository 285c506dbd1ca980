"""Node visits of the per-lane walks: trees whose stacks end below, at and beyond the LDS part, seen from every octant
(near and far planes picked by address), against the oracle; counted and uncounted kernels give the same hits."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 12, 40, 300])
def test_stack_edges_in_every_octant(n, oracle_mod):
    import torch
    from paper_2410_05095_amd import _native as N
    from tests.test_gpu_render import compare_rect, deep_scene
    ctx = N.Context(0)
    scene = deep_scene(n)
    gs = ctx.scene_from(scene).build()
    osc = oracle_mod.OracleScene.from_scene(scene)
    for o in range(8):
        sx, sy, sz = (1 - 2 * (o >> a & 1) for a in range(3))
        # towards the point that the triangles shrink to: camera rays cross many nested boxes
        cam = dataclasses.replace(scene.cameras[0], eye=(0.9 * sx, 0.3 + 0.8 * sy, 1.1 * sz), target=(0.02, 0.3, 0.01),
                                  width=21, height=13)
        print(f"[lane stack] n {n} octant {o} depth {gs.stats()['depth']}", flush=True)
        compare_rect(ctx, oracle_mod, scene, cam, 4, o, gs=gs, osc=osc)
        outs = [ctx.render(gs, cam, (), rect=scene.rect_light, area_samples=4, area_stream=o, per_lane=True, count=c)
                for c in (False, True)]
        torch.cuda.synchronize()
        assert torch.equal(outs[0]["hit"], outs[1]["hit"]) and torch.equal(outs[0]["visibility"], outs[1]["visibility"])
    gs.close()
    ctx.close()
