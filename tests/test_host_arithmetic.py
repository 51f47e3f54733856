"""The kernels' short forms, run from the library's own source compiled for the host: what a bound lets pass or decides
against the exact decision behind it.

Links: every (cell, direction) that the FP64 decision finds lies in the near cells, in the cells that reach the face's
plane and in the FP32 filter's mask; the filter passes no cell that the reach test drops; a certain pair is a hit; both
staged forms of a face give one mask; the decision is that of the definition with its divisions.  Flags: a separation
beyond the rounding bound is the full test's answer.  Own-bin: no accepted point is dropped, no sure one refused."""
import ctypes
import itertools

import numpy as np
import pytest

import _host

F = np.float32
DIRS = {3: [d for d in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1),
                        (0, 1, -1), (1, 1, 1), (1, 1, -1), (1, -1, 1), (-1, 1, 1))],
        2: [(1, 0), (0, 1), (1, 1), (1, -1)]}


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return _host.load("host_arithmetic", tmp_path_factory.mktemp("host"))


def _p(a):
    assert a.flags.c_contiguous
    return a.ctypes.data_as(ctypes.c_void_p)


def _links(lib, dim, v, lo, dx, eps, block):
    n, cells, pairs = len(v), 4 ** dim, len(DIRS[dim])
    out = {"near": np.zeros(n, np.uint64), "reach": np.zeros(n, np.uint64), "reach_each": np.zeros(n, np.uint64),
           "may": np.zeros((n, cells), np.uint32), "may_rows": np.zeros((n, cells), np.uint32),
           "sure": np.zeros((n, cells), np.uint8), "centre": np.zeros((n, cells, dim), F),
           "t": np.zeros((n, cells, pairs))}
    ins = [np.ascontiguousarray(x, F) for x in (v, lo, dx, eps)] + [np.ascontiguousarray(block, np.int32)]
    lib.links(ctypes.c_int(dim), ctypes.c_int64(n), *map(_p, ins), *(_p(x) for x in out.values()))
    return out


def _bits(mask, cells):
    return (mask[:, None] >> np.arange(cells, dtype=np.uint64)) & np.uint64(1) != 0


def _definition(dim, v, centre, dx):
    """t of every direction's segment-face decision with its divisions, NaN where there is none; one direction."""
    v, o = v.astype(float)[:, None], centre.astype(float)
    out = []
    with np.errstate(all="ignore"):
        for d in DIRS[dim]:
            D = (np.array(d) * dx.astype(F)).astype(F).astype(float)[:, None]
            if dim == 3:
                cross = lambda a, b: np.stack([a[..., 1] * b[..., 2] - a[..., 2] * b[..., 1],
                                               a[..., 2] * b[..., 0] - a[..., 0] * b[..., 2],
                                               a[..., 0] * b[..., 1] - a[..., 1] * b[..., 0]], -1)
                dot = lambda a, b: a[..., 0] * b[..., 0] + a[..., 1] * b[..., 1] + a[..., 2] * b[..., 2]
                e1, e2, T = v[:, :, 1] - v[:, :, 0], v[:, :, 2] - v[:, :, 0], o - v[:, :, 0]
                P, Qv = cross(D, e2), cross(T, e1)
                det = dot(e1, P)
                u, w, t = dot(T, P) / det, dot(D, Qv) / det, dot(e2, Qv) / det
                ok = (det != 0) & ~((u < 0) | (u > 1)) & ~((w < 0) | (u + w > 1))
            else:
                e, w0 = v[:, :, 1] - v[:, :, 0], v[:, :, 0] - o
                den = D[..., 0] * e[..., 1] - D[..., 1] * e[..., 0]
                t = (w0[..., 0] * e[..., 1] - w0[..., 1] * e[..., 0]) / den
                s = (w0[..., 0] * D[..., 1] - w0[..., 1] * D[..., 0]) / den
                ok = (den != 0) & (s >= 0) & (s <= 1)
            out.append(np.where(ok, t, np.nan))
    return np.stack(out, -1)


def _grid(rng, n, dim, scale):
    """Domains as the library makes them: dx = (hi - lo) / cells in FP32, eps = 2^-20 max(1, |lo|, |hi|)."""
    cells = 4 * rng.integers(1, 33, (n, dim)) << rng.integers(0, 6, (n, 1))
    lo = (scale * rng.uniform(-100, 100, (n, dim)) * (rng.random((n, 1)) < 0.7)).astype(F)
    hi = (lo + scale * cells * 10.0 ** rng.uniform(-1, 0.3, (n, dim))).astype(F)
    dx = ((hi - lo) / cells.astype(F)).astype(F)
    eps = (F(2.0 ** -20) * np.maximum(F(1), np.maximum(np.abs(lo), np.abs(hi)))).astype(F)
    block = rng.integers(0, cells // 4)
    return lo, dx, eps, block


def _check_links(lib, dim, v, lo, dx, eps, block):
    r = _links(lib, dim, v, lo, dx, eps, block)
    cells, pairs = 4 ** dim, len(DIRS[dim])
    near, reach = _bits(r["near"], cells), _bits(r["reach"], cells)
    assert np.array_equal(reach, _bits(r["reach_each"], cells))
    assert np.array_equal(r["may"], r["may_rows"])
    want = _definition(dim, v, r["centre"], dx)
    assert np.array_equal(np.isnan(want), np.isnan(r["t"]))
    assert np.array_equal(want[~np.isnan(want)], r["t"][~np.isnan(want)])
    with np.errstate(invalid="ignore"):
        hit = np.abs(r["t"]) <= 1
    may = (r["may"][..., None] >> np.arange(pairs, dtype=np.uint32)) & 1 != 0
    assert not (hit & ~may).any()
    assert not (may.any(-1) & ~reach).any()
    assert not (hit.any(-1) & ~near).any()
    assert not ((r["sure"] != 0) & ~hit.any(-1)).any()
    return int(hit.sum()), int((r["sure"] != 0).sum()), int((near & ~reach).sum()), int((near & reach).sum())


@pytest.mark.parametrize("scale", [1e-6, 1e-3, 1.0, 1e5])
@pytest.mark.parametrize("flat", [0.0, 1e-7, 1e-5, 1e-2, 1.0])
def test_links_through_a_direction(lib, flat, scale):
    """Faces through a point of some link, or just beside it, their plane turned out of the link by `flat`."""
    rng = np.random.default_rng(1)
    n = 3000
    hits = certain = 0
    for dim in (2, 3):
        lo, dx, eps, block = _grid(rng, n, dim, scale)
        cell = rng.integers(0, 4, (n, dim))
        o = lo.astype(float) + (4 * block + cell + 0.5) * dx
        D = np.array(DIRS[dim])[rng.integers(0, len(DIRS[dim]), n)] * dx.astype(float)
        side = rng.normal(size=(n, dim)) * dx
        length = 10.0 ** rng.uniform(-1.5, 1, (n, 1))
        t = rng.choice([0.0, 1.0, -1.0, 0.5, 1 + 1e-7], (n, 1))
        w = rng.choice([0.0, 1.0, 0.5, 1e-7, -1e-7, 0.3], (n, 2)) + 1e-8 * rng.normal(size=(n, 2))
        e1 = length * (side * flat + D * rng.normal(size=(n, 1))) if dim == 2 else \
            length * (side * rng.uniform(0.2, 1, (n, 1)) + D * rng.normal(size=(n, 1)))
        if dim == 3:
            out = rng.normal(size=(n, 3)) * dx
            e2 = length * (side * rng.normal(size=(n, 1)) * rng.choice([1, 1e-3], (n, 1)) + D * rng.normal(size=(n, 1))
                           + flat * out)
            a = o + t * D - w[:, :1] * e1 - w[:, 1:] * (1 - w[:, :1]) * e2
            v = np.stack([a, a + e1, a + e2], 1).astype(F)
        else:
            a = o + t * D - w[:, :1] * e1
            v = np.stack([a, a + e1], 1).astype(F)
        h, s, _, _ = _check_links(lib, dim, v, lo, dx, eps, block)
        hits += h
        certain += s
    assert hits > n
    if flat == 1.0:
        assert certain > n


@pytest.mark.parametrize("scale", [1e-6, 1e-3, 1.0, 1e5])
@pytest.mark.parametrize("seed", range(3))
def test_links_at_the_reach_of_a_plane(lib, scale, seed):
    """Faces whose plane some link of a cell just meets or just misses, corners in the plane from near to far."""
    rng = np.random.default_rng(20 + seed)
    n = 4000
    lo, dx, eps, block = _grid(rng, n, 3, scale)
    o = lo.astype(float) + (4 * block + rng.integers(0, 4, (n, 3)) + 0.5) * dx
    a = rng.normal(size=(n, 3))
    a[rng.random((n, 3)) < 0.2] = 0
    a[(a == 0).all(1)] = 1
    far = (np.abs(a) * dx).sum(1) / (a * a).sum(1)
    shift = rng.choice([-1, 1], n) * far * (1 + rng.choice([0, 1e-7, -1e-7, 1e-6, -1e-6, 1e-5, 1e-3, 0.2], n))
    w1 = np.cross(a, rng.normal(size=(n, 3)))
    w2 = np.cross(a, w1)
    w1, w2 = (w / np.linalg.norm(w, axis=1)[:, None] for w in (w1, w2))
    co = rng.normal(size=(n, 3, 2)) * (10.0 ** rng.uniform(-1, 1.5, n) * dx.mean(1))[:, None, None]
    v = (o[:, None] + (shift[:, None] * a)[:, None] + co[..., :1] * w1[:, None] + co[..., 1:] * w2[:, None]).astype(F)
    _, _, dropped, kept = _check_links(lib, 3, v, lo, dx, eps, block)
    assert dropped > n and kept > n


def test_links_of_overflow_and_empty_faces(lib):
    rng = np.random.default_rng(4)
    n = 1000
    lo, dx, eps = np.zeros((n, 3), F), np.ones((n, 3), F), np.full((n, 3), 1e-4, F)
    block = rng.integers(0, 8, (n, 3))
    p = (4 * block[:, None] + rng.uniform(0, 4, (n, 1, 3))).astype(F)
    with np.errstate(all="ignore"):
        cases = [(rng.uniform(-1, 1, (n, 3, 3)) * s).astype(F) for s in (1e12, 1e13, 1e15, 1e19, 1e25, 1e38)]
    cases += [np.repeat(p, 3, 1), np.concatenate([p, p, p + F(1)], 1)]   # a point, a line
    for v in cases:
        r = _links(lib, 3, v, lo, dx, eps, block)
        hit = (np.abs(np.nan_to_num(r["t"], nan=9.0)) <= 1).any(-1)
        assert not ((r["sure"] != 0) & ~hit).any()
        assert np.array_equal(r["reach"], r["reach_each"])


def test_cells_of_near_codes(lib):
    lib.cells_of_code.restype = ctypes.c_uint64
    for dim in (2, 3):
        for c in range(1 << (4 * dim)):
            want = 0
            for pos in itertools.product(range(4), repeat=dim):
                bits = sum(1 << (4 * a + x) for a, x in enumerate(pos))
                if c & bits == bits:
                    want |= 1 << sum(x << (2 * a) for a, x in enumerate(pos))
            assert lib.cells_of_code(ctypes.c_int(dim), ctypes.c_uint32(c)) == want


@pytest.mark.parametrize("scale", [1e-16, 1e-12, 1e-3, 1.0, 1e6, 1e12, 1e16])
@pytest.mark.parametrize("kind", ["any", "sliver", "aligned"])
def test_separation_beyond_its_bound_decides(lib, kind, scale):
    rng = np.random.default_rng(11)
    n = 40000
    with np.errstate(all="ignore"):
        a = rng.normal(size=(n, 3))
        b, c = a + rng.normal(size=(n, 3)), a + rng.normal(size=(n, 3))
        if kind == "sliver":
            c = a + (b - a) * rng.uniform(-0.5, 1.5, (n, 1)) + rng.normal(size=(n, 3)) * 10.0 ** rng.uniform(-8, -1, (n, 1))
        elif kind == "aligned":   # edges along an axis, or corners on the cells' grid
            b = a.copy()
            b[np.arange(n), rng.integers(0, 3, n)] += rng.normal(size=n)
        size = scale * 10.0 ** rng.uniform(-1.5, 1.5, (n, 1))
        at = rng.uniform(-1, 1, (n, 3)) * scale * 10.0 ** rng.uniform(0, 2, (n, 1))
        v = (np.stack([a, b, c], 1) * size[:, None] + at[:, None]).astype(F)
        h = (scale * 10.0 ** rng.uniform(-1, 0.5, n)).astype(F)
        if kind == "aligned":
            v[n // 2:] = (np.round(v[n // 2:] / h[n // 2:, None, None]) * h[n // 2:, None, None]).astype(F)
        eps = (np.abs(v).max((1, 2)) * F(2.0 ** -20)).astype(F)
        lo, hi = v.min(1), v.max(1)
        m = lo - h[:, None] + rng.uniform(0, 1, (n, 3)) * (hi - lo + 2 * h[:, None])
        near = (rng.dirichlet([0.4] * 3, n)[:, :, None] * v).sum(1) + h[:, None] * rng.choice([-1, 1, 1 - 1e-6, 0.3], (n, 3))
        m = np.where(rng.random((n, 1)) < 0.5, m, near)
        if kind == "aligned":
            m[n // 2:] = np.round(m[n // 2:] / h[n // 2:, None]) * h[n // 2:, None]
        reach = (h + eps)[:, None]
        m = np.ascontiguousarray(np.clip(m.astype(F), lo - reach, hi + reach).astype(F))
    full, gap, delta = np.zeros(n, np.uint8), np.zeros(n, F), np.zeros(n, F)
    lib.sat(ctypes.c_int64(n), _p(v), _p(m), _p(h), _p(eps), _p(full), _p(gap), _p(delta))
    full = full != 0
    assert not (full & (gap > delta)).any()
    assert not (~full & (gap < -delta)).any()
    decided = np.abs(gap) > delta
    if scale in (1e-16, 1e16):
        assert not decided.any()
    elif kind == "any":
        assert decided[np.isfinite(delta)].mean() > 0.5 and full.any() and not full.all()


@pytest.mark.parametrize("dim", [2, 3])
def test_own_bin_short_tests(lib, dim):
    rng = np.random.default_rng(3)
    n = 400000
    size = 10.0 ** rng.uniform(-4, 4, (n, 1))
    a = rng.normal(size=(n, dim))
    b = a + rng.normal(size=(n, dim))
    parts = [a, b]
    if dim == 3:   # third corner near the line a b, down to below the sliver limit, anywhere along it
        parts.append(a + (b - a) * rng.uniform(-0.2, 1.2, (n, 1)) + rng.normal(size=(n, 3)) * 10.0 ** rng.uniform(-3, 0, (n, 1)))
    at = rng.uniform(-1, 1, (n, dim)) * size * 10.0 ** rng.uniform(-1, 3, (n, 1))
    v = (np.stack(parts, 1) * size[:, None] + at[:, None]).astype(F)
    R = (size[:, 0] * 10.0 ** rng.uniform(-3, 2, n)).astype(F)
    # a point at about R from a point of the face (weights a little outside it too), or from the first corner
    w = rng.dirichlet(np.ones(dim), n) * 1.02 - 0.02 / dim
    d = rng.normal(size=(n, dim))
    if dim == 3:
        e = v.astype(float)
        across = np.cross(e[:, 1] - e[:, 0], e[:, 2] - e[:, 0])
        d = np.where((rng.random((n, 1)) < 0.5) & (np.abs(across).max(1) > 0)[:, None], across, d)
    d /= np.linalg.norm(d, axis=1)[:, None]
    p = (w[:, :, None] * v.astype(float)).sum(1) + d * R[:, None] * rng.uniform(0.97, 1.03, (n, 1))
    corner = v[:, 0] + d * R[:, None] * rng.uniform(0.999, 1.0, (n, 1))
    p = np.ascontiguousarray(np.where(rng.random((n, 1)) < 0.7, p, corner).astype(F))
    near, sure, maybe = (np.zeros(n, np.uint8) for _ in range(3))
    reach2 = np.zeros(n, F)
    lib.own(ctypes.c_int(dim), ctypes.c_int64(n), _p(v), _p(p), _p(R), _p(near), _p(reach2), _p(sure), _p(maybe))
    near, sure, maybe = near != 0, sure != 0, maybe != 0
    assert not (near & ~maybe).any()
    assert not (sure & ~near).any()
    assert sure.any() and (~maybe).any() and near.sum() > n // 10 and np.isfinite(reach2).mean() > 0.5
