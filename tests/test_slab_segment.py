"""The clamped slab test of the wave-uniform walks (segments 0 < t < 1), emulated exactly on the CPU.

Near planes use inv = (1/dd) (1 - 2^-20), far planes (1/dd) (1 + 2^-20), each with its offset moved outward;
entry and exit are clamped to [0, 1] and a box is entered when entry < exit.  Pinned: every box that the exact
segment meets at some 0 < t < 1 passes, and boxes that it clearly misses fail, those beyond t = 1 among them."""
from fractions import Fraction

import numpy as np

from tests.test_slab_bound import F32, box_through, fr, random_ray, rnd, segment_box_exact


def seg_consts(o, d):
    grow, shrink = fr(F32(1.000001)), fr(F32(1.0 - 2.0 ** -20))
    out = []
    for a in range(3):
        x = float(d[a])
        if abs(x) < 1e-20:
            x = float(np.copysign(F32(1e-20), F32(x)))
        i = rnd(1 / fr(x))
        n, g = rnd(fr(i) * shrink), rnd(fr(i) * grow)
        c, e = rnd(-(fr(o[a]) * fr(n))), rnd(-(fr(o[a]) * fr(g)))
        m = rnd(abs(fr(c)) * Fraction(1, 2 ** 21) + Fraction(1, 2 ** 120))
        mf = rnd(abs(fr(e)) * Fraction(1, 2 ** 21) + Fraction(1, 2 ** 120))
        out.append((x, n, g, rnd(fr(c) - fr(m)), rnd(fr(e) + fr(mf))))
    return out


def slab_seg(consts, lo, hi):
    near, far = [], []
    for a, (_, n, g, cn, cf) in enumerate(consts):
        p, q = (lo[a], hi[a]) if n >= 0 else (hi[a], lo[a])
        near.append(rnd(fr(p) * fr(n) + fr(cn)))
        far.append(rnd(fr(q) * fr(g) + fr(cf)))
    return min(max(max(near), 0.0), 1.0) < min(max(min(far), 0.0), 1.0)


def test_boxes_that_the_segment_enters_pass():
    rng = np.random.default_rng(17)
    for _ in range(1500):
        o, d = random_ray(rng)
        consts = seg_consts(o, d)
        dd = [c[0] for c in consts]
        for t in (Fraction(1, 2 ** 20), Fraction(int(rng.integers(1, 2 ** 20)), 2 ** 20), Fraction(1) - Fraction(1, 2 ** 22)):
            lo, hi = box_through(rng, o, dd, t, tuple(a for a in range(3) if rng.random() < 0.3))
            assert slab_seg(consts, lo, hi), (o, d, lo, hi, t)


def test_missed_boxes_fail_also_beyond_the_end():
    rng = np.random.default_rng(18)
    beside = beyond = 0
    for _ in range(3000):
        o, d = random_ray(rng)
        if min(abs(float(x)) for x in d) < 1e-6 * max(abs(float(x)) for x in d):
            continue
        consts = seg_consts(o, d)
        dd = [c[0] for c in consts]
        size = max(abs(float(o[k])) + abs(float(dd[k])) for k in range(3))
        t = Fraction(int(rng.integers(0, 2 ** 21)), 2 ** 19)      # up to four times the segment
        lo, hi = box_through(rng, o, dd, t)
        grow = 1e-5 * size
        if segment_box_exact(o, dd, [x - grow for x in lo], [x + grow for x in hi], 1.0) is None:
            assert not slab_seg(consts, lo, hi), (o, d, lo, hi)   # on the line, beyond the end
            beyond += 1
        a = int(rng.integers(3))
        shift = (1e-4 * size + (hi[a] - lo[a])) * (1 if rng.random() < 0.5 else -1)
        lo[a], hi[a] = float(F32(lo[a] + shift)), float(F32(hi[a] + shift))
        if segment_box_exact(o, dd, [x - grow for x in lo], [x + grow for x in hi], 1.0) is None:
            assert not slab_seg(consts, lo, hi), (o, d, lo, hi)
            beside += 1
    assert beside > 300 and beyond > 300, (beside, beyond)
