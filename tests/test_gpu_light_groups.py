"""Wave-uniform point-light shadow passes on either side of the size from which a packet's lights are walked in turn by one
wave instead of as units of their own (2.5M samples x (triangles / 20,000)^(1/4)): the per-lane kernel's masks."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("build", [{}, dict(watertight=True), dict(two_level=True)])
def test_units_and_lights_in_turn(build):
    import torch
    from paper_2410_05095_amd import _native as N
    from tests.test_gpu_render import deep_scene
    ctx = N.Context(0)
    scene = deep_scene(40)
    line = 2.5e6 * (scene.n_tris / 20000) ** 0.25
    gs = ctx.scene_from(scene).build(**build)
    rng = np.random.default_rng(8)
    lights = np.concatenate([rng.uniform((-3, 1, -3), (3, 9, 3), (16, 3)), np.ones((16, 3))], 1).astype(np.float32)
    for w, h, ssaa in ((719, 743, 1), (731, 737, 1), (365, 367, 2), (368, 369, 2)):
        in_turn = w * h * ssaa * ssaa >= line
        cam = dataclasses.replace(scene.cameras[0], width=w, height=h, ssaa=ssaa)
        for n in (1, 2, 3, 16):
            print(f"[light groups] {build} {w}x{h}x{ssaa} lights {n} in turn {in_turn}", flush=True)
            want = ctx.render(gs, cam, lights[:n], per_lane=True)["shadow"]
            assert 0.02 < float((want != 0).float().mean())
            for count in (False, True):
                out = {"shadow": torch.full_like(want, -1)}
                got = ctx.render(gs, cam, lights[:n], wave=True, count=count, out=out)["shadow"]
                torch.cuda.synchronize()
                assert ctx.last_error() == 0
                assert torch.equal(got, want), (n, count, int((got != want).sum()))
    gs.close()
    ctx.close()
