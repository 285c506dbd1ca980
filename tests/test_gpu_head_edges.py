"""Loss, head and head gradients where their chunks of pixels (512 per workgroup of the head's backward pass, 4096 of the
loss) are one partial chunk, exactly filled, or end in a remainder."""
import pytest

from oracle import unet as U
from tests import unet_flips as F
from tests.test_gpu_denoiser import cosine, ctx, oracle_params, random_batch, rel_frob, to_dev, unflat  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w", [(1, 4, 4), (1, 16, 32), (1, 4, 132), (1, 64, 64), (2, 12, 172)])
def test_loss_and_head_gradients(ctx, n, h, w):  # noqa: F811
    from paper_2410_05095_amd import _native as N
    print(f"[head] {n}x{h}x{w}", flush=True)
    den = N.Denoiser(ctx, seed=4)
    p = oracle_params(6)
    den.set_params(U.flat(p))
    x, t, m = random_batch(31 + w, n, h, w)
    loss = den.train_step(*to_dev(ctx, x, t, m), lr=0.0)
    g = unflat(den.grads())
    y, cache = U.forward(p, x, bf16=True)
    lo = U.masked_mse(y, t, m)
    want, _ = U.backward(p, cache, t, m, bf16_grads=True)
    scale, _ = F.flip_scale(p, x, t, m)
    # BF16 rounding flips, as the oracle itself shows them; a loss over few pixels moves by as much as a gradient
    assert abs(loss - lo) <= 5e-3 * lo, (loss, lo)
    for k in ("head.w", "head.b", "d1b.w", "e1a.w"):
        assert rel_frob(g[k], want[k]) <= max(5e-3, 2.0 * scale[k]), (k, rel_frob(g[k], want[k]), scale[k])
        assert cosine(g[k], want[k]) >= 0.9999, k
    den.close()
