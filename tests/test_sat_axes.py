"""The flag pass's short form of the FP32 triangle-box test, restated: where its largest separation is beyond delta =
2^-15 R^2 it has the answer of the full test, for cells within h of the face's box (the ones it is asked for), over face
shapes from regular to slivers and axis-aligned ones, sizes, offsets, and cells placed where an axis is just met; and it
is seldom undecided where nothing is aligned."""
import numpy as np
import pytest

F = np.float32


def _fma(a, b, c):
    return (a.astype(np.float64) * b + c).astype(F)


def _full(v, m, h):
    A, B, C = ((v[:, k] - m).T for k in range(3))
    out = np.ones(len(m), bool)

    def sep(p, r):
        out[(np.minimum(np.minimum(p[0], p[1]), p[2]) > r) | (np.maximum(np.maximum(p[0], p[1]), p[2]) < -r)] = False
    for a in range(3):
        sep((A[a], B[a], C[a]), h)
    E = [B - A, C - B, A - C]
    N = [E[0][i] * E[1][j] - E[0][j] * E[1][i] for i, j in ((1, 2), (2, 0), (0, 1))]
    s = (N[0] * A[0] + N[1] * A[1]) + N[2] * A[2]
    r = h * ((np.abs(N[0]) + np.abs(N[1])) + np.abs(N[2]))
    out[(s > r) | (s < -r)] = False
    for e in E:
        for (i, j), (au, av) in (((1, 2), (-e[2], e[1])), ((0, 2), (e[2], -e[0])), ((0, 1), (-e[1], e[0]))):
            sep([au * X[i] + av * X[j] for X in (A, B, C)], h * (np.abs(au) + np.abs(av)))
    return out


def _gap(v, m, h, eps):
    v0 = v[:, 0].T
    lo, hi = v.min(1).T, v.max(1).T
    b, c = (v[:, 1] - v[:, 0]).T, (v[:, 2] - v[:, 0]).T
    R = np.max((hi - lo) + (h + eps), 0) * F(1.0001)
    R2 = R * R
    inv = F(1) / R
    n = [(b[i] * c[j] - b[j] * c[i]) * inv for i, j in ((1, 2), (2, 0), (0, 1))]
    p = m.T - v0
    half = F(0.5)
    box = np.max([np.abs(p[a] - half * ((lo[a] - v0[a]) + (hi[a] - v0[a]))) - (half * (hi[a] - lo[a]) + h) for a in range(3)], 0)
    gap = np.maximum(box * R, np.abs(_fma(n[0], p[0], _fma(n[1], p[1], n[2] * p[2])))
                     - h * ((np.abs(n[0]) + np.abs(n[1])) + np.abs(n[2])))
    for e in (b, (v[:, 2] - v[:, 1]).T, -c):
        for (i, j), (au, av) in (((1, 2), (-e[2], e[1])), ((0, 2), (e[2], -e[0])), ((0, 1), (-e[1], e[0]))):
            p1, p2 = au * b[i] + av * b[j], au * c[i] + av * c[j]
            mn, mx = np.minimum(np.minimum(p1, p2), F(0)), np.maximum(np.maximum(p1, p2), F(0))
            w = np.where((au == 0) & (av == 0), R2, half * (mx - mn) + h * (np.abs(au) + np.abs(av)))
            gap = np.maximum(gap, np.abs(_fma(au, p[i], _fma(av, p[j], -half * (mn + mx)))) - w)
    delta = np.where((R2 >= F(1e-24)) & (R2 <= F(1e24)), F(2.0 ** -15) * R2, F(np.inf))
    return gap, delta


@pytest.mark.parametrize("scale", [1e-16, 1e-12, 1e-3, 1.0, 1e6, 1e12, 1e16])
@pytest.mark.parametrize("kind", ["any", "sliver", "aligned"])
def test_gap_beyond_delta_decides(kind, scale):
    rng = np.random.default_rng(11)
    n = 40000
    with np.errstate(all="ignore"):
        a = rng.normal(size=(n, 3))
        b, c = a + rng.normal(size=(n, 3)), a + rng.normal(size=(n, 3))
        if kind == "sliver":
            c = a + (b - a) * rng.uniform(-0.5, 1.5, (n, 1)) + rng.normal(size=(n, 3)) * 10.0 ** rng.uniform(-8, -1, (n, 1))
        elif kind == "aligned":   # edges along an axis, or corners on the cells' grid
            k = rng.integers(0, 3, n)
            b = a.copy()
            b[np.arange(n), k] += rng.normal(size=n)
        size = scale * 10.0 ** rng.uniform(-1.5, 1.5, (n, 1))
        at = rng.uniform(-1, 1, (n, 3)) * scale * 10.0 ** rng.uniform(0, 2, (n, 1))
        v = (np.stack([a, b, c], 1) * size[:, None] + at[:, None]).astype(F)
        h = (scale * 10.0 ** rng.uniform(-1, 0.5, n)).astype(F)
        if kind == "aligned":
            v[n // 2:] = (np.round(v[n // 2:] / h[n // 2:, None, None]) * h[n // 2:, None, None]).astype(F)
        eps = (np.abs(v).max((1, 2)) * F(2.0 ** -20)).astype(F)
        # cells: anywhere within h of the box, or where one of the axes is just met
        lo, hi = v.min(1), v.max(1)
        m = lo - h[:, None] + rng.uniform(0, 1, (n, 3)) * (hi - lo + 2 * h[:, None])
        w = rng.dirichlet([0.4] * 3, n)
        near = (w[:, :, None] * v).sum(1) + h[:, None] * rng.choice([-1, 1, 1 - 1e-6, 0.3], (n, 3))
        m = np.where(rng.random((n, 1)) < 0.5, m, near)
        if kind == "aligned":
            m[n // 2:] = np.round(m[n // 2:] / h[n // 2:, None]) * h[n // 2:, None]
        reach = (h + eps)[:, None]
        m = np.clip(m.astype(F), lo - reach, hi + reach).astype(F)
        full = _full(v, m, h)
        gap, delta = _gap(v, m, h, eps)
    assert not (full & (gap > delta)).any()
    assert not (~full & (gap < -delta)).any()
    decided = np.abs(gap) > delta
    if scale in (1e-16, 1e16):
        assert not decided.any()
    elif kind == "any":
        assert decided[np.isfinite(delta)].mean() > 0.5 and full.any() and not full.all()
