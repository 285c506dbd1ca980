"""Post pass with 4 and with 16 rows to a workgroup's tile: around the sizes where the kernel changes (700,000 pixels, and
images of more rows than a grid of 4-row tiles takes) and at the edges of the small tiles, bit for bit against the oracle."""
import numpy as np
import pytest

from tests.test_gpu_post import compare, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(1, 1), (3, 64), (4, 64), (5, 65), (17, 129), (700, 1000), (701, 1000), (262140, 2), (262141, 2)])
def test_tiles(ctx, h, w):  # noqa: F811
    rng = np.random.default_rng([h, w])
    y, x = np.mgrid[0:h, 0:w]
    img = np.where((y * 17 + x) % 31 < 15, 0.8, 0.1) + np.where((x * 19 + y) % 53 < 20, 0.5, 0.0)
    img = np.repeat(img[..., None], 4, -1) * np.array([1.0, 0.7, 0.4, 1.0])
    img[rng.random((h, w)) < 0.02] = (9.0, 9.0, 9.0, 0.3)
    compare(ctx, np.ascontiguousarray(img, np.float32), f"tiles {h}x{w}")
