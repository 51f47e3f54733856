"""The own-bin flag pass on both sides of its line between a cell per lane (at most as many faces in a bin as the wave
has cells there) and a face per lane: face counts around the cells of a wave in one bin, partial waves, bins of both
kinds in one wave, and faces on either side of the short tests (slivers, specks, large faces)."""
import numpy as np
import pytest

import geomgen
from test_gpu_own_bin import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,roots,faces", [(3, (1, 1, 1), [1, 2, 63, 64, 65, 129]), (3, (3, 2, 2), [5, 40, 64, 66]),
                                             (2, (1, 1, 1), [1, 15, 16, 17]), (2, (3, 2, 1), [3, 31, 33, 63, 64, 65])])
@pytest.mark.parametrize("B", [1, 2, 5])
def test_few_faces_in_a_bin(orc, dim, roots, faces, B):
    rng = np.random.default_rng(10 * dim + B)
    for n in faces:
        c = rng.uniform(0.1, 0.9, (n, 1, dim))
        v = c + rng.normal(size=(n, dim, dim)) * 10.0 ** rng.uniform(-4, -0.3, (n, 1, 1))
        thin = rng.random(n) < 0.3
        e = rng.normal(size=(n, 1, dim)) * 0.2
        v[thin] = (c + e * rng.uniform(-0.5, 0.5, (n, dim, 1)) + rng.normal(size=(n, dim, dim)) * 1e-5)[thin]
        v = v.reshape(-1, dim).astype(np.float32)
        f = np.arange(len(v), dtype=np.int32).reshape(n, dim)
        wl = geomgen.Workload(f"few{n}", dim, v, f, roots, 2, B, 19 if dim == 3 else 9)
        _check(orc, wl, B, [0.07, 0.03])
