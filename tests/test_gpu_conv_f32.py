"""The FP32 network at the sizes where its tile width changes (16, 32 and 64 columns) and at ragged ones, against a
float64 network of nine shifted products per layer."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LAYERS = ((8, 32), (32, 32), (32, 64), (64, 64), (64, 128), (128, 128), (192, 64), (64, 64), (96, 32), (32, 32))


def net64(x, p):
    import torch
    o, ws = 0, []
    for cin, cout in LAYERS:
        ws.append((p[o:o + cout * 9 * cin].reshape(cout, 9, cin), p[o + cout * 9 * cin:o + cout * (9 * cin + 1)]))
        o += cout * (9 * cin + 1)

    def conv(x, l):
        w, b = ws[l]
        n, h, wd, cin = x.shape
        q = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
        y = sum(q[:, t // 3:t // 3 + h, t % 3:t % 3 + wd].reshape(-1, cin) @ w[:, t].t().contiguous() for t in range(9))
        return torch.relu(y + b).reshape(n, h, wd, -1)

    pool = lambda t: (t[:, ::2, ::2] + t[:, 1::2, ::2] + t[:, ::2, 1::2] + t[:, 1::2, 1::2]) / 4  # noqa: E731
    up = lambda t: t.repeat_interleave(2, 1).repeat_interleave(2, 2)  # noqa: E731
    e1 = conv(conv(x, 0), 1)
    e2 = conv(conv(pool(e1), 2), 3)
    bn = conv(conv(pool(e2), 4), 5)
    d2 = conv(conv(torch.cat([up(bn), e2], -1), 6), 7)
    d1 = conv(conv(torch.cat([up(d2), e1], -1), 8), 9)
    return torch.sigmoid(d1 @ p[o:o + 32] + p[o + 32])


# 4x4: one partial tile everywhere; 68x132: ragged rows and columns; 400x1316 and 1000x1284: 32-column tiles in the
# full-resolution layers; 2x720x1284: 64-column tiles in the 64-channel layers
@pytest.mark.parametrize("n,h,w", [(1, 4, 4), (3, 20, 36), (1, 68, 132), (1, 400, 1316), (1, 1000, 1284), (2, 720, 1284)])
def test_infer_fp32_tile_widths(n, h, w):
    import torch
    from paper_2410_05095_amd import _native as N
    print(f"[conv f32] {n}x{h}x{w}", flush=True)
    ctx = N.Context(0)
    den = N.Denoiser(ctx, seed=11)
    rng = np.random.default_rng(h)
    p = den.params()
    p += rng.normal(0, 0.01, p.size).astype(np.float32)      # biases away from zero
    den.set_params(p)
    g = torch.Generator("cuda").manual_seed(w)
    feat = torch.randn((n, h, w, 8), generator=g, device="cuda").to(torch.bfloat16)
    got = den.infer(feat, fp32=True).double()
    torch.cuda.synchronize()
    with torch.no_grad():
        want = net64(feat.double(), torch.from_numpy(p.astype(np.float64)).cuda())
    # ten layers of FP32 sums of up to 1728 products: 10 x 2 sqrt(1728) x 2^-24 = 5e-5 of the logit's scale at worst
    # bounds a sigmoid's error by a quarter of it
    assert float((got - want).abs().max()) <= 1.25e-5
    den.close()
    ctx.close()
