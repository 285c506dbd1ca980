"""Post pass at the tile edges of its kernels (64 x 16 pixels, 13 around them) and at tone-map values around every
rounding boundary, bit for bit against the oracle."""
import numpy as np
import pytest

from tests.test_gpu_post import compare, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(15, 63), (16, 64), (17, 65), (13, 130), (42, 90), (1, 200), (200, 1)])
def test_long_edges_across_tiles(ctx, h, w):  # noqa: F811
    rng = np.random.default_rng([h, w])
    y, x = np.mgrid[0:h, 0:w]
    # nearly horizontal, nearly vertical and diagonal edges longer than the search, and single bright pixels
    img = np.where((y * 17 + x) % 31 < 15, 0.8, 0.1) + np.where((x * 19 + y) % 53 < 20, 0.5, 0.0)
    img = np.repeat(img[..., None], 4, -1) * np.array([1.0, 0.7, 0.4, 1.0])
    img[rng.random((h, w)) < 0.02] = (9.0, 9.0, 9.0, 0.3)
    compare(ctx, np.ascontiguousarray(img, np.float32), f"edges {h}x{w}")


def test_rounding_boundaries(ctx):  # noqa: F811
    # FP32 values around each c whose encoded value lies at k + 1/2, where FP32 alone cannot decide the byte
    k = (np.arange(255) + 0.5) / 255.0
    v = np.where(k <= 0.04045, k / 12.92, ((k + 0.055) / 1.055) ** 2.4)
    c = (v / (1.0 - v)).astype(np.float32)
    near = [c]
    for _ in range(24):
        near += [np.nextafter(near[-1], np.float32(np.inf))]
    lo = [c]
    for _ in range(24):
        lo += [np.nextafter(lo[-1], np.float32(0))]
    vals = np.concatenate(near + lo + [np.array([0.0, -1.0, 1e-30, 1e30, 3.4e38], np.float32)])
    vals = np.resize(vals, (128, 128))
    compare(ctx, np.ascontiguousarray(np.repeat(vals[..., None], 4, -1), np.float32), "rounding boundaries")
