"""The face-centric flag pass at the edges of its waves: face counts around the 4, 8 and 16 faces of a wave and the four
waves of a workgroup, faces from below a cell to most of the domain in one wave; forests (flags included) bit for bit
those of the oracle."""
import numpy as np
import pytest

import geomgen
from _parity import compare_forest, gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("faces", [1, 2, 3, 4, 5, 15, 16, 17, 65])
def test_few_faces(orc, dim, faces):
    rng = np.random.default_rng(100 * dim + faces)
    at = rng.uniform(0.2, 0.8, (faces, 1, dim))
    v = np.clip(at + rng.normal(size=(faces, dim, dim)) * 10.0 ** rng.uniform(-3, -0.5, (faces, 1, 1)), 0.02, 0.98)
    v = v.reshape(-1, dim).astype(np.float32)
    f = np.arange(faces * dim, dtype=np.int32).reshape(faces, dim)
    wl = geomgen.Workload("few", dim, v, f, (4, 3, 5 if dim == 3 else 1), 2, 8, 9 if dim == 2 else 19)
    g = gpu_run(wl, with_links=False)
    coords = orc.gather(dim, v, f)
    ob = orc.bin_faces(dim, coords, wl.lo[:dim], wl.hi[:dim], wl.bins)
    of = orc.refine(dim, coords, ob, wl.roots[:dim], wl.levels, wl.d_spec(), wl.lo[:dim], wl.hi[:dim])
    compare_forest(g, of, wl.levels)
    log(f"  {dim}D {faces} faces: {len(g['levels'])} levels compared")


def test_reciprocals_of_cell_counts():
    for n in list(range(1, 5000)) + [65535, 65536, 1 << 20, (1 << 31) - 1]:
        assert n == 1 or 0xFFFFFFFF // n + 1 == -(-(1 << 32) // n)
