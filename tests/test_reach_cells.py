"""The node pass's 64-bit cell masks, restated: a face's near code as the cells it covers, and the cells that pass the
short test of the face's plane, against the per-cell definitions the row pass uses."""
import itertools

import numpy as np

F = np.float32


def _code_cells(c):
    x, y, z = c & 15, (c >> 4) & 15, (c >> 8) & 15
    rows = ((y & 1) | (y & 2) << 3 | (y & 4) << 6 | (y & 8) << 9) * x
    lo = ((z & 1) | (z & 2) << 15) * rows
    hi = (((z >> 2) & 1) | ((z >> 2) & 2) << 15) * rows
    assert rows < 1 << 16 and lo < 1 << 32 and hi < 1 << 32
    return hi << 32 | lo


def test_code_cells():
    for c in range(1 << 12):
        want = 0
        for x, y, z in itertools.product(range(4), repeat=3):
            bits = 1 << x | 1 << (4 + y) | 1 << (8 + z)
            if c & bits == bits:
                want |= 1 << (x + 4 * y + 16 * z)
        assert _code_cells(c) == want


def test_shared_sums_are_the_pairs_sums():
    rng = np.random.default_rng(2)
    n = 20000
    base, a, b, c = (rng.normal(size=n).astype(F) for _ in range(4))
    bound = (np.abs(base) * rng.uniform(0, 2, n)).astype(F)
    base[:50], bound[50:100] = np.nan, np.inf
    for x, y, z in itertools.product(range(4), repeat=3):
        shared = ((base + F(x) * a) + F(y) * b) + F(z) * c
        pair = ((base + np.full(n, x, F) * a) + np.full(n, y, F) * b) + np.full(n, z, F) * c
        assert np.array_equal(shared, pair, equal_nan=True)
        assert not (np.abs(shared[:50]) > bound[:50]).any()   # a NaN stays for the filter
