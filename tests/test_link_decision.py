"""The link step's FP64 decision without its divisions by det: the comparisons of un, vn and |det| that stand for
u >= 0, u <= 1, v >= 0 and fl(u + v) <= 1 of the rounded quotients give the same answers, at random, at the limits and
a few roundings beside them, for numbers over the whole range that products of FP32 numbers have."""
import numpy as np


def test_comparisons_stand_for_the_rounded_quotients():
    rng = np.random.default_rng(5)
    n = 400000
    det = rng.uniform(1, 2, n) * 2.0 ** rng.integers(-300, 300, n) * rng.choice([-1.0, 1.0], n)
    u = rng.choice([0.0, -0.0, 1.0, 0.5, 1 / 3], n)
    u = np.where(rng.random(n) < 0.7, rng.uniform(-0.2, 1.2, n), u)
    v = np.where(rng.random(n) < 0.3, rng.uniform(-0.2, 1.2, n), 1.0 - u)
    un, vn = u * det, v * det
    for x in (un, vn):   # up to eight roundings away
        for _ in range(8):
            go = rng.random(n) < 0.4
            x[go] = np.nextafter(x[go], x[go] * rng.choice([0.0, 4.0], int(go.sum())))
    un = np.where(rng.random(n) < 0.02, rng.choice([-1.0, 1.0], n) * 2.0 ** -447, un)
    uq, vq = un / det, vn / det
    want = ~((uq < 0) | (uq > 1)) & ~((vq < 0) | (uq + vq > 1))
    ad = np.abs(det)
    us, vs = np.where(det < 0, -un, un), np.where(det < 0, -vn, vn)
    over, m = (us + vs) - ad, ad * 2.0 ** -50
    close = (over >= -m) & ~(over > m)
    got = ~((us < 0) | (us > ad)) & ~((vs < 0) | (over > m)) & ~(close & (us / ad + vs / ad > 1))
    assert np.array_equal(got, want)
    near = (np.abs(uq + vq - 1) < 1e-14) & (uq >= 0) & (vq >= 0)
    assert want[near].any() and (~want[near]).any() and close.sum() > n // 4
