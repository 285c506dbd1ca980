"""The box test of the exact wave-uniform walks (rc_slab_seg with doubled margins) enters every box that the per-lane
walk's test (rc_slab, segment 0 <= t <= 1) accepts, emulated exactly on the CPU at boxes on the verge of both."""
from fractions import Fraction

import numpy as np

from tests.test_slab_bound import F32, fr, random_ray, ray_consts, rnd, slab_fp32
from tests.test_slab_segment import seg_consts, slab_seg


def exact_consts(o, d):
    out = []
    for x, n, g, cn, cf in seg_consts(o, d):
        m = rnd(rnd(abs(fr(cn)) * Fraction(1, 2 ** 21)) + Fraction(1, 2 ** 120))
        mf = rnd(rnd(abs(fr(cf)) * Fraction(1, 2 ** 21)) + Fraction(1, 2 ** 120))
        out.append((x, n, g, rnd(fr(cn) - fr(m)), rnd(fr(cf) + fr(mf))))
    return out


def test_exact_walk_enters_what_the_per_lane_walk_enters():
    rng = np.random.default_rng(23)
    accepted = refused = margin_needed = 0
    for _ in range(4000):
        o, d = random_ray(rng)
        lane, seg, wide = ray_consts(o, d), seg_consts(o, d), exact_consts(o, d)
        dd = lane[0]
        # one corner of the box near the ray at t, each coordinate within a few units of the tests' margins of it
        t = float(rng.choice([0.0, 1e-6, rng.random(), 1.0 - 1e-6, 1.0]))
        lo, hi = [0.0] * 3, [0.0] * 3
        for a in range(3):
            scale = abs(float(o[a])) + abs(float(dd[a])) * t
            p = float(F32(float(o[a]) + float(dd[a]) * t + scale * rng.normal(0.0, 2.0 ** -21)))
            size = float(rng.choice([0.0, 1e-7, 1e-3])) * scale
            lo[a], hi[a] = (p, float(F32(p + size))) if rng.random() < 0.5 else (float(F32(p - size)), p)
        if slab_fp32(lane, lo, hi, 1.0):
            accepted += 1
            assert slab_seg(wide, lo, hi), (o, d, lo, hi)
            margin_needed += not slab_seg(seg, lo, hi)
        else:
            refused += 1
    assert accepted > 500 and refused > 500, (accepted, refused, margin_needed)
