"""The convolution kernels of small images against those of large ones: an image alone and in a batch large enough for the
other kernels gives the same output bit for bit, and the same gradients up to the order of the sums over pixels (256 copies
scale every gradient by 2^-8 exactly)."""
import numpy as np
import pytest

from oracle import unet as U
from tests.test_gpu_denoiser import ctx, oracle_params, random_batch, rel_frob, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(20, 68), (36, 132), (12, 28)])
def test_alone_and_in_a_large_batch(ctx, h, w):  # noqa: F811
    import torch
    from paper_2410_05095_amd import _native as N
    print(f"[conv small] {h}x{w}", flush=True)
    den = N.Denoiser(ctx, seed=8)
    den.set_params(U.flat(oracle_params(9)))
    x, t, m = random_batch(41 + h, 1, h, w)
    big = 256
    one = to_dev(ctx, x, t, m)
    many = to_dev(ctx, np.repeat(x, big, 0), np.repeat(t, big, 0), np.repeat(m, big, 0))
    y1, yn = den.infer(one[0]), den.infer(many[0])
    torch.cuda.synchronize()
    assert torch.equal(yn, y1.expand_as(yn))
    grads = []
    for b in (one, many):
        den.train_step(*b, lr=0.0)
        grads.append(np.asarray(den.grads(), np.float64))
    # FP32 sums over up to 256 x 4752 pixels in different orders: 2^-24 a step, random signs, log-depth trees and chunks
    assert rel_frob(grads[1], grads[0]) <= 2e-5
    den.close()
