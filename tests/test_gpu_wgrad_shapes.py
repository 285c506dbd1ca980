"""Training gradients at sizes where the weight-gradient kernel's tiles (2 rows x 64 columns, chunks of several tiles)
end unevenly: columns beyond the last full tile, one column tile with few columns, levels of odd tile counts."""
import pytest

from oracle import unet as U
from tests import unet_flips as F
from tests.test_gpu_denoiser import cosine, ctx, oracle_params, random_batch, rel_frob, to_dev, unflat  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w", [(3, 20, 68), (2, 36, 132), (1, 100, 28)])
def test_gradients_on_ragged_tiles(ctx, n, h, w):  # noqa: F811
    from paper_2410_05095_amd import _native as N
    print(f"[wgrad] {n}x{h}x{w}", flush=True)
    den = N.Denoiser(ctx, seed=2)
    p = oracle_params(5)
    den.set_params(U.flat(p))
    x, t, m = random_batch(21 + h, n, h, w)
    den.train_step(*to_dev(ctx, x, t, m), lr=0.0)
    g = unflat(den.grads())
    _, cache = U.forward(p, x, bf16=True)
    want, _ = U.backward(p, cache, t, m, bf16_grads=True)
    scale, _ = F.flip_scale(p, x, t, m)
    for k in U.param_names():
        # the bound of the larger batches' test: BF16 rounding flips, as the oracle itself shows them
        assert rel_frob(g[k], want[k]) <= max(5e-3, 2.0 * scale[k]), (k, rel_frob(g[k], want[k]), scale[k])
        assert cosine(g[k], want[k]) >= 0.9999, k
    den.close()
