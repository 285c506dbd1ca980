"""Passes on either side of the sizes up to which rays are traced four lanes to a ray: the per-lane kernels' hits, masks and
visibility (at most a ten-thousandth of the samples, where FP32 does not decide, may differ)."""
import dataclasses

import numpy as np
import pytest

from paper_2410_05095_amd import scenegen as sg

pytestmark = pytest.mark.gpu


# (bodies, two-level, image, rect-light samples): camera rays of a large two-level scene around 180,000; point lights of it
# around 600,000 x 11 / 20; camera rays of a flat one around 600,000; rect light of a small one around 950,000
@pytest.mark.parametrize("n_inst,two,w,h,samples", [(400, True, 424, 424, 0), (400, True, 428, 428, 0), (400, True, 572, 572, 0),
                                                    (400, True, 580, 580, 0), (400, False, 768, 776, 0), (400, False, 776, 784, 0),
                                                    (40, False, 344, 344, 8), (40, False, 352, 344, 8)])
def test_either_side(n_inst, two, w, h, samples):
    import torch
    from paper_2410_05095_amd import _native as N
    ctx = N.Context(0)
    scene = sg.city_scene(0, n_instances=n_inst)
    gs = ctx.scene_from(scene).build(two_level=two, device=not two)
    cam = dataclasses.replace(scene.cameras[0], width=w, height=h, ssaa=1)
    kw = dict(rect=sg.DEFAULT_RECT, area_samples=samples) if samples else {}
    lights = () if samples else scene.point_lights[:1]
    print(f"[quad limits] {scene.n_tris} triangles two {two} {w}x{h} x {max(samples, 1)}, stack {gs.stats()['max_stack']}", flush=True)
    a, b = ({k: v.clone() for k, v in ctx.render(gs, cam, lights, per_lane=p, **kw).items() if v is not None} for p in (False, True))
    torch.cuda.synchronize()
    assert ctx.last_error() == 0
    differ = (a["hit"] != b["hit"]).any(1)
    for k in ("shadow", "visibility"):
        if k in a:
            differ |= (a[k] != b[k]).reshape(-1)
    n = int(differ.sum())
    print(f"[quad limits] {n} samples differ", flush=True)
    assert n <= 1e-4 * cam.n_samples
    gs.close()
    ctx.close()
