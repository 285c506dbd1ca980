"""Camera rays of flat 2x2-sample frames by wave-uniform walks (counted frames, and frames of more than five million
samples): the oracle's hits, and the per-lane kernel's bit for bit, with both triangle tests, at odd sizes, and in trees
whose walk needs one or two stack registers."""
import dataclasses

import numpy as np
import pytest

from paper_2410_05095_amd import scenegen as sg
from tests.parity import assert_clean, compare_point, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2410_05095_amd import _native as N
    c = N.Context(0)
    yield c
    c.close()


def scene_of(kind):
    from tests.test_gpu_render import deep_scene
    if kind == "deep":
        return deep_scene()
    return sg.small_random_scene(6, n_instances=50, width=8, height=8, n_lights=0)


@pytest.mark.parametrize("watertight", [False, True])
@pytest.mark.parametrize("kind,build", [("bodies", {}), ("bodies", dict(device_sah=True)), ("deep", {})])
def test_counted_frames(ctx, oracle_mod, kind, build, watertight):
    import torch
    scene = scene_of(kind)
    gs = ctx.scene_from(scene).build(watertight=watertight, **build)
    osc = oracle_mod.OracleScene.from_scene(scene, watertight=watertight)
    stack = gs.stats()["max_stack"]
    assert (64 < stack <= 128) if kind == "deep" else stack <= 64
    for w, h in ((1, 1), (4, 4), (5, 3), (33, 70), (101, 57)):
        cam = dataclasses.replace(scene.cameras[0], width=w, height=h, ssaa=2)
        print(f"[primary wave] {kind} {build} wt {watertight} {w}x{h} stack {stack}", flush=True)
        orc = osc.render_point(cam, scene.point_lights, np.arange(cam.n_samples))
        hits = []
        for kw in (dict(count=True), dict(per_lane=True)):
            out = ctx.render(gs, cam, (), **kw)
            torch.cuda.synchronize()
            assert ctx.last_error() == 0
            hits.append(to_np(out["hit"]).view(np.uint32))
            if kw.get("count"):   # the wave's lanes share their visits: more than the rays' own
                assert ctx.stage_times()["primary_rays"] == cam.n_samples
            assert_clean(compare_point(hits[-1], None, None, orc, 0), max_band_frac=1.0)
        clean = ~orc["band_primary"].astype(bool)
        assert np.array_equal(hits[0][clean], hits[1][clean])
    gs.close()


@pytest.mark.parametrize("watertight", [False, True])
def test_large_frame(ctx, oracle_mod, watertight):
    import torch
    scene = scene_of("bodies")
    gs = ctx.scene_from(scene).build(watertight=watertight)
    cam = dataclasses.replace(scene.cameras[0], width=1327, height=971, ssaa=2)
    assert cam.n_samples > 5_000_000
    print(f"[primary wave] {cam.n_samples} samples, wt {watertight}", flush=True)
    hits = [ctx.render(gs, cam, (), per_lane=p)["hit"].clone() for p in (False, True)]
    torch.cuda.synchronize()
    assert ctx.last_error() == 0
    # samples that differ lie in the oracle's FP32 band, where either answer stands
    differ = np.flatnonzero(to_np((hits[0] != hits[1]).any(1)))
    print(f"[primary wave] {len(differ)} samples differ", flush=True)
    assert len(differ) < 1e-4 * cam.n_samples
    if len(differ):
        orc = oracle_mod.OracleScene.from_scene(scene, watertight=watertight).render_point(cam, scene.point_lights, differ)
        assert orc["band_primary"].astype(bool).all()
    gs.close()
