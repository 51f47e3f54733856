"""The link step's FP32 filter restated: the three barycentrics scaled by |D . n| held against one margin.  Every pair
that the exact decision finds must pass it, and every pair that it calls certain must be found: over face shapes down to
slivers, planes (nearly) along the direction, where the computed sign of D . n may be wrong, and hits at edges, corners
and segment ends; a face whose products overflow or that has no area may pass but is never called certain."""
import itertools

import numpy as np
import pytest

F = np.float32
DIRS = [d for d in itertools.product((-1, 0, 1), repeat=3) if d > (0, 0, 0)]


def _dot(a, b):
    return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2]


def _cross(a, b):
    return a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]


def _sum(d, x):
    """The direction's signed sum, as the filter forms it."""
    out = None
    for c, y in zip(d, x):
        if c:
            y = y if c > 0 else -y
            out = y if out is None else out + y
    return out


def _filter(v, o, dx, d):
    l1 = lambda x: (np.abs(x[0]) + np.abs(x[1])) + np.abs(x[2])
    a, e1, e2 = v[:, 0].T, (v[:, 1] - v[:, 0]).T, (v[:, 2] - v[:, 0]).T
    T = o.T - a
    n = _cross(e1, e2)
    nT, n1, n2 = l1(T), l1(e1), l1(e2)
    mx = dx.max() * F(2.0 ** -20)
    MU, MV, MD, MT = mx * nT * n2, mx * n1 * nT, mx * n1 * n2, F(2.0 ** -20) * nT * n1 * n2
    M = (MU + MV) + F(2) * MD
    Ms = M + F(0) * (MD * F(2.0 ** 24))   # NaN where D . n may overflow
    atn = np.abs(_dot(T, n))
    den, nu, nv = (_sum(d, [x[k] * dx[k] for k in range(3)]) for x in (n, _cross(T, e2), _cross(e1, T)))
    ad, neg = np.abs(den), np.signbit(den)
    su, sv = np.where(neg, -nu, nu), np.where(neg, -nv, nv)
    mn = np.minimum(np.minimum(su, sv), (ad - su) - sv)   # passes a NaN on
    return (atn - (MD + MT) <= ad) & (mn >= -M), (atn + (MD + MT) <= ad) & (mn > Ms)


def _hit(v, o, dx, d):
    v, o, D = v.astype(float), o.astype(float), np.array(d) * dx.astype(float)
    a, e1, e2, T = v[:, 0].T, (v[:, 1] - v[:, 0]).T, (v[:, 2] - v[:, 0]).T, (o - v[:, 0]).T
    P, Q = _cross(D, e2), _cross(T, e1)
    det = _dot(e1, P)
    with np.errstate(all="ignore"):
        u, w, t = _dot(T, P) / det, _dot(D, Q) / det, _dot(e2, Q) / det
    return (det != 0) & (u >= 0) & (w >= 0) & (u + w <= 1) & (np.abs(t) <= 1)


@pytest.mark.parametrize("flat", [0.0, 1e-8, 1e-7, 1e-6, 1e-3, 1.0])
def test_hits_pass_and_certain_ones_hit(flat):
    """flat: how far the face's plane is turned out of the direction (0: along it, up to the rounding of corners)."""
    rng = np.random.default_rng(17)
    n = 20000
    hits = certain = 0
    for d in DIRS:
        dx = (10.0 ** rng.uniform(-2, 0, 3)).astype(F)
        D = np.array(d) * dx.astype(float)
        o = rng.uniform(-3, 3, (n, 3)).astype(F)
        # two edges about along a plane through the direction, sheared out of it by `flat`
        side = rng.normal(size=(n, 3))
        out = np.cross(side, D)
        size = 10.0 ** rng.uniform(-1.5, 1, (n, 1)) * np.linalg.norm(D) / np.linalg.norm(side, axis=1)[:, None]
        out *= size * np.linalg.norm(side, axis=1)[:, None] / np.linalg.norm(out, axis=1)[:, None]
        e1 = side * size * rng.uniform(0.2, 1, (n, 1)) + D * rng.normal(size=(n, 1)) + flat * rng.normal(size=(n, 1)) * out
        e2 = (side * size * rng.normal(size=(n, 1)) * rng.choice([1, 1e-3], (n, 1)) + D * rng.normal(size=(n, 1))
              + flat * rng.normal(size=(n, 1)) * out)
        # a point of the face (or just beside it) at t of the segment
        w = rng.choice([0.0, 1.0, 0.5, 1e-7, -1e-7, 0.3], (n, 2)) + 1e-8 * rng.normal(size=(n, 2))
        t = rng.choice([0.0, 1.0, -1.0, 0.5, 1 + 1e-7], (n, 1))
        a = o + t * D - w[:, :1] * e1 - w[:, 1:] * (1 - w[:, :1]) * e2
        v = np.stack([a, a + e1, a + e2], 1).astype(F)
        may, sure = _filter(v, o, dx, d)
        hit = _hit(v, o, dx, d)
        assert not (hit & ~may).any()
        assert not (sure & ~hit).any()
        hits += int(hit.sum())
        certain += int(sure.sum())
    assert hits > n
    if flat == 1.0:
        assert certain > n // 10


def test_overflow_and_empty_faces_are_never_certain():
    rng = np.random.default_rng(4)
    dx = np.ones(3, F)
    with np.errstate(all="ignore"):
        for scale in (1e12, 1e13, 1e15, 1e19, 1e25, 1e38):
            v = (rng.uniform(-1, 1, (4000, 3, 3)) * scale).astype(F)
            o = rng.uniform(-1, 1, (4000, 3)).astype(F)
            for s in (F(1), F(scale) * F(0.5)):
                for d in DIRS:
                    _, sure = _filter(v, o, dx * s, d)
                    assert not (sure & ~_hit(v, o, dx * s, d)).any()
        p = rng.uniform(-1, 1, (4000, 1, 3)).astype(F)
        for v in (np.repeat(p, 3, 1), np.concatenate([p, p, p + F(1)], 1)):   # a point, a line
            for d in DIRS:
                assert not _filter(v, p[:, 0], dx, d)[1].any()
