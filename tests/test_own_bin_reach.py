"""The two short tests before the own-bin flag step's near test: a point that the FP32 near test accepts lies within
`reach` of the face's bounding box (reach restated here from its definition), and one within R of the first corner
by the FP32 squared distance against 0.9999 R^2 is accepted; over face shapes from regular to just above the sliver
limit, sizes and offsets over many orders of magnitude, and points placed around the distance R."""
import numpy as np
import pytest

import oracle


def _reach(f, dim, R):
    v = f.reshape(dim, dim).astype(np.float32)
    l2 = np.float32(0)
    for k in range(3 if dim == 3 else 1):
        e = v[(k + 1) % dim] - v[k]
        l2 = max(l2, np.float32((e * e).sum(dtype=np.float32)))
    fine = R <= 1e8 and 1e-10 <= l2 <= 1e10
    if dim == 3:
        n = np.cross(v[1] - v[0], v[2] - v[0]).astype(np.float32)
        fine = fine and np.float32((n * n).sum(dtype=np.float32)) >= np.float32(1e-4) * (l2 * l2)
    return np.float32(1.002) * np.float32(R) + np.float32(0.002) * np.sqrt(l2) if fine else np.inf


@pytest.mark.parametrize("dim", [2, 3])
def test_near_points_lie_within_reach_of_the_box(dim):
    rng = np.random.default_rng(3)
    near = bounded = sure = 0
    closest = 0.0   # largest box distance of an accepted point, as a share of the bound
    for _ in range(60000):
        size = 10.0 ** rng.uniform(-4, 4)
        offset = rng.uniform(-1, 1, dim) * size * 10.0 ** rng.uniform(-1, 3)
        a = rng.normal(size=dim)
        b = a + rng.normal(size=dim)
        if dim == 3:
            # third corner near the line a b, down to about the sliver limit, anywhere along it
            c = a + (b - a) * rng.uniform(-0.2, 1.2) + rng.normal(size=3) * 10.0 ** rng.uniform(-2.2, 0)
            v = np.stack([a, b, c])
        else:
            v = np.stack([a, b])
        v = (v * size + offset).astype(np.float32)
        R = np.float32(size * 10.0 ** rng.uniform(-3, 2))
        reach = _reach(v, dim, R)
        if not np.isfinite(reach):
            continue
        bounded += 1
        # a point at about R from a random point of the face (weights a little outside it too)
        w = rng.dirichlet(np.ones(dim)) * 1.02 - 0.02 / dim
        d = rng.normal(size=dim)
        if dim == 3 and rng.random() < 0.5:
            d = np.cross((v[1] - v[0]).astype(float), (v[2] - v[0]).astype(float))
        p = ((w[:, None] * v.astype(float)).sum(0) + d / np.linalg.norm(d) * R * rng.uniform(0.97, 1.03)).astype(np.float32)
        if oracle.near_l2_f32(dim, v, p, float(R)):
            near += 1
            g = np.maximum(np.maximum(v.min(0) - p, p - v.max(0)), 0).astype(np.float64)
            share = np.sqrt((g * g).sum()) / reach
            closest = max(closest, share)
            assert share <= 0.9995, (v, p, R)
        # around R from the first corner
        d = rng.normal(size=dim)
        p = (v[0] + d / np.linalg.norm(d) * R * rng.uniform(0.999, 1.0)).astype(np.float32)
        w = p - v[0]
        w2 = w[0] * w[0] + w[1] * w[1]
        w2 = w2 + w[2] * w[2] if dim == 3 else w2
        if w2 <= np.float32(0.9999) * (R * R):
            sure += 1
            assert oracle.near_l2_f32(dim, v, p, float(R)), (v, p, R)
    assert sure > 10000 and bounded > 30000 and near > 5000 and closest > 0.8
