"""Refit by levels: small levels go several to a launch (runs longer than one launch takes, a run between large levels),
large ones alone.  Every box exact for the moved vertices."""
import numpy as np
import pytest

from paper_2410_05095_amd import scenegen as sg
from tests.parity import bvh_bound_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["deep", "wide"])
def test_levels_refit_exactly(which, oracle_mod):
    import torch
    from paper_2410_05095_amd import _native as N
    from tests.test_gpu_render import deep_scene
    # deep: 31 levels of a few nodes each; wide: levels on both sides of the small levels' size
    scene = deep_scene() if which == "deep" else sg.small_random_scene(5, n_instances=60, width=16, height=16, ssaa=1, n_lights=1)
    ctx = N.Context(0)
    gs = ctx.scene_from(scene).build()
    print(f"[refit levels] {which}: {gs.stats()['n_nodes']} nodes, depth {gs.stats()['depth']}", flush=True)
    ids = np.arange(0, len(scene.body_vertex_range), 2).astype(np.int32)
    rng = np.random.default_rng(2)
    xf = np.tile(np.eye(3, 4, dtype=np.float32), (len(ids), 1, 1))
    c, s = np.float32(np.cos(0.3)), np.float32(np.sin(0.3))
    xf[:, 0, 0], xf[:, 0, 2], xf[:, 2, 0], xf[:, 2, 2] = c, s, -s, c
    xf[:, :, 3] = rng.uniform(-0.5, 0.5, (len(ids), 3)).astype(np.float32)
    gs.set_transforms(torch.from_numpy(xf.reshape(len(ids), -1).copy()).cuda(), torch.from_numpy(ids).cuda())
    gs.refit()
    torch.cuda.synchronize()
    assert ctx.last_error() == 0
    nodes, order = gs.export()
    assert bvh_bound_errors(nodes, order, gs.positions(), scene.indices)[0] == 0
    gs.close()
    ctx.close()
