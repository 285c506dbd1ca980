"""Node arrays of 4 GiB and more (2^25 nodes): the per-lane walks address them with 64-bit offsets.  One height field of
96 million triangles in a tree of one triangle per leaf, against the same in a tree small enough for 32-bit offsets."""
import numpy as np
import pytest

from paper_2410_05095_amd import scenegen as sg

pytestmark = pytest.mark.gpu


def height_field(n):
    """n x n quads over [-10, 10]^2, as (positions, indices)."""
    g = np.linspace(-10.0, 10.0, n + 1, dtype=np.float32)
    pos = np.empty((n + 1, n + 1, 3), np.float32)
    pos[..., 0], pos[..., 2] = g[:, None], g[None, :]
    pos[..., 1] = 0.4 * np.sin(2.1 * g)[:, None] * np.cos(1.7 * g)[None, :] + 0.02 * np.sin(91.0 * g)[:, None] * np.sin(83.0 * g)
    q = (np.arange(n, dtype=np.uint32)[:, None] * np.uint32(n + 1) + np.arange(n, dtype=np.uint32)[None, :]).reshape(-1)
    idx = np.empty((2 * n * n, 3), np.uint32)
    idx[0::2, 0], idx[0::2, 1], idx[0::2, 2] = q, q + np.uint32(1), q + np.uint32(n + 2)
    idx[1::2, 0], idx[1::2, 1], idx[1::2, 2] = q, q + np.uint32(n + 2), q + np.uint32(n + 1)
    return pos.reshape(-1, 3), idx


def test_node_array_beyond_4_gib():
    import torch
    from paper_2410_05095_amd import _native as N
    print("[wide] scene", flush=True)
    ctx = N.Context(0)
    pos, idx = height_field(6930)
    gs = N.Scene(ctx, pos, idx, np.zeros(len(idx), np.uint32), np.array([[0.5, 0.5, 0.5, 0.5, 0.0]], np.float32))
    cam = sg.Camera(eye=(3.0, 9.0, -14.0), target=(0.0, 0.0, 0.0), up=(0.0, 1.0, 0.0), vfov_deg=60.0, width=321, height=203,
                    ssaa=1, seed=2)
    lights = np.array([[6.0, 2.5, 2.0, 9.0, 9.0, 9.0], [-3.0, 1.6, -5.0, 9.0, 9.0, 9.0]], np.float32)
    rect = sg.RectLight(center=(0.0, 1.1, 0.0), edge_u=(2.0, 0.0, 0.0), edge_v=(0.0, 0.0, 2.0), radiance=(4.0, 4.0, 4.0))
    got = {}
    for max_leaf in (1, 4):
        gs.build(device=True, max_leaf=max_leaf)
        n = int(gs.stats()["n_nodes"])
        print(f"[wide] max_leaf {max_leaf}: {n} nodes", flush=True)
        assert (n >= 1 << 25) == (max_leaf == 1)
        for light, kw in (("points", dict(lights=lights)), ("rect", dict(lights=(), rect=rect, area_samples=5))):
            for count in (False, True):
                o = ctx.render(gs, cam, per_lane=max_leaf == 4, count=count, **kw)
                torch.cuda.synchronize()
                assert ctx.last_error() == 0
                got[max_leaf, light, count] = {k: o[k].clone() for k in ("hit", "shadow", "visibility", "rgba") if o.get(k) is not None}
    hit = got[4, "points", False]["hit"]
    assert float((hit[:, 0] != -1).float().mean()) > 0.5
    lit = got[4, "points", False]["shadow"]
    assert all(0.02 < float((lit >> l & 1).float().mean()) < 0.98 for l in (0, 1))
    assert 0.02 < float(got[4, "rect", False]["visibility"].mean()) < 0.98
    for (leaf, light, count), o in got.items():
        for k, v in o.items():
            assert torch.equal(v, got[4, light, False][k]), (leaf, light, count, k, int((v != got[4, light, False][k]).sum()))
    gs.close()
    ctx.close()
