"""The short test before the link step's FP32 filter, restated in FP32: a face's plane is followed over a block from the
value at its first cell.  Whatever the filter's own test of the plane (|T . n| <= |D . n| + margins, some direction D)
can pass for a cell of the block has to pass the short test too: over face shapes, sizes and offsets, unequal cell
sizes, and planes placed where the two bounds are met."""
import itertools

import numpy as np
import pytest

F = np.float32


def _centres(lo, g, dx):
    """(g + 1/2) dx + lo with one rounding after the product, each cell's own."""
    return (lo.astype(np.float64) + (g + 0.5) * dx.astype(np.float64)).astype(F)


@pytest.mark.parametrize("scale", [1e-14, 1e-6, 1.0, 1e5])
@pytest.mark.parametrize("seed", range(3))
def test_short_test_passes_all_that_the_filter_passes(scale, seed):
    rng = np.random.default_rng(seed)
    n = 4000
    dx = (scale * 10.0 ** rng.uniform(-1, 0.3, (n, 3))).astype(F)
    lo = (scale * rng.uniform(-100, 100, (n, 3)) * (rng.random((n, 1)) < 0.5)).astype(F)
    g0 = 4 * rng.integers(0, 1 << 10, (n, 3))
    # half a rounding of the largest coordinate, doubled twice: less than what the library takes
    top = np.maximum(np.abs(lo), np.abs(lo + dx * F(1 << 12)))
    eps = (top * F(2.0 ** -22)).astype(F)
    pos = np.array(list(itertools.product(range(4), repeat=3)))
    cells = rng.integers(0, 64, n)
    o_at = _centres(lo, g0 + pos[cells], dx)
    # a face whose plane is about S from that cell, corners in the plane up to a few cells or many away
    a = rng.normal(size=(n, 3))
    a[rng.random((n, 3)) < 0.2] = 0
    a[(a == 0).all(1)] = 1
    reach = (np.abs(a) * dx).sum(1) / (a * a).sum(1)
    shift = rng.choice([-1, 1], n) * reach * (1 + rng.choice([0, 1e-7, -1e-7, 1e-6, -1e-6, 1e-5, 1e-3, 0.2], n))
    base = o_at.astype(np.float64) + shift[:, None] * a
    w = np.cross(a, rng.normal(size=(n, 3)))
    w2 = np.cross(a, w)
    size = 10.0 ** rng.uniform(-1, 1.5, n)
    co = rng.normal(size=(n, 3, 2)) * (size * dx.mean(1))[:, None, None]
    un, wn = w / np.linalg.norm(w, axis=1)[:, None], w2 / np.linalg.norm(w2, axis=1)[:, None]
    v = (base[:, None] + co[..., :1] * un[:, None] + co[..., 1:] * wn[:, None]).astype(F)
    e1, e2 = v[:, 1] - v[:, 0], v[:, 2] - v[:, 0]
    nn = np.stack([e1[:, 1] * e2[:, 2] - e1[:, 2] * e2[:, 1], e1[:, 2] * e2[:, 0] - e1[:, 0] * e2[:, 2],
                   e1[:, 0] * e2[:, 1] - e1[:, 1] * e2[:, 0]], 1)
    assert nn.dtype == F

    def s3(x):
        return (x[:, 0] + x[:, 1]) + x[:, 2]
    n1, n2 = s3(np.abs(e1)), s3(np.abs(e2))
    c0 = _centres(lo, g0, dx)
    T = c0 - v[:, 0]
    mx = dx.max(1)
    sn, se = s3(np.abs(nn * dx)), s3(np.abs(nn * eps))
    slack = F(1.1920928955078125e-06) * (mx + F(2) * (s3(np.abs(T)) + F(3) * s3(dx))) * (n1 * n2)
    bound = ((sn * F(1.00001) + se) + slack) + F(1e-43)
    first = s3(T * nn)
    passed = 0
    for c in range(64):
        i = pos[c].astype(F)
        s = ((first + i[0] * (nn[:, 0] * dx[:, 0])) + i[1] * (nn[:, 1] * dx[:, 1])) + i[2] * (nn[:, 2] * dx[:, 2])
        short = ~(np.abs(s) > bound)
        To = _centres(lo, g0 + pos[c], dx) - v[:, 0]
        md = mx * F(2.0 ** -20) * n1 * n2
        mt = F(2.0 ** -20) * s3(np.abs(To)) * n1 * n2
        t_lo = np.abs(s3(To * nn)) - (md + mt)
        filt = t_lo <= sn * F(1 + 2.0 ** -22)   # the largest |D . n| that the filter's sums can give
        assert not (filt & ~short).any()
        passed += int(filt.sum())
    assert 64 * n // 20 < passed < 64 * n   # both answers of the filter's test occur
