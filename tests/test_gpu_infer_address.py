"""Output addresses of the denoiser that are not 4-byte aligned: the FP32 network writes the same bytes there, the BF16
network refuses them and writes nothing."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1, 2, 3, 4])
def test_output_address(shift):
    import torch
    from paper_2410_05095_amd import _native as N
    n, h, w = 2, 20, 36
    print(f"[infer address] shift {shift}", flush=True)
    ctx = N.Context(0)
    den = N.Denoiser(ctx, seed=3)
    g = torch.Generator("cuda").manual_seed(5)
    feat = torch.randn((n, h, w, 8), generator=g, device="cuda").to(torch.bfloat16)
    size = 4 * n * h * w
    for fn, fp32 in ((N.lib().rc_denoiser_infer_fp32, True), (N.lib().rc_denoiser_infer, False)):
        want = den.infer(feat, fp32=fp32).view(torch.uint8).reshape(-1)
        buf = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        rc = fn(ctx.h, den.h, C.c_void_p(feat.data_ptr()), n, h, w, C.c_void_p(buf.data_ptr() + 16 + shift))
        torch.cuda.synchronize()
        assert ctx.last_error() == 0
        if fp32 or shift % 4 == 0:
            assert rc == 0
            assert torch.equal(buf[16 + shift:16 + shift + size], want)
            buf[16 + shift:16 + shift + size] = 0xA5
        else:
            with pytest.raises(N.RcError):
                N.check(rc, "rc_denoiser_infer")
        assert bool((buf == 0xA5).all())
    den.close()
    ctx.close()
