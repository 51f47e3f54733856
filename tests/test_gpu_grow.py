"""Child generation where it rebuilds several levels in one pass: bodies far smaller than a root block under many
passes, so that every pass adds balance marks down a chain of levels (a level then is a parent and a child in the same
launch), on one root, few roots and a grid that is not a cube, and bodies that flag nothing or lie outside.  Every
level's keys, leaf bits, marks and cell flags must equal the oracle's."""
import numpy as np
import pytest

import geomgen
from _parity import compare_forest, gpu_run, log

pytestmark = pytest.mark.gpu


def _speck(dim, at, size):
    rng = np.random.default_rng(4)
    v = (np.asarray(at[:dim]) + rng.uniform(-size, size, (dim, dim))).astype(np.float32)
    return v, np.arange(dim, dtype=np.int32).reshape(1, dim)


CASES = [
    (2, (1, 1, 1), 7, (0.501, 0.499, 0.5), 1e-3),
    (2, (3, 2, 1), 6, (0.334, 0.5, 0.5), 1e-3),
    (2, (5, 5, 1), 5, (0.0, 0.0, 0.0), 1e-2),
    (3, (1, 1, 1), 6, (0.5, 0.5, 0.5), 1e-3),
    (3, (2, 3, 1), 5, (0.49, 0.34, 0.99), 1e-3),
    (3, (3, 3, 3), 4, (0.34, 0.66, 0.33), 5e-2),
    (3, (2, 2, 2), 3, (1.7, 0.5, 0.5), 1e-2),    # outside the domain: nothing is flagged
]


@pytest.mark.parametrize("own_bin", [False, True])
@pytest.mark.parametrize("dim,roots,levels,at,size", CASES)
def test_levels_rebuilt_in_one_pass(orc, dim, roots, levels, at, size, own_bin):
    v, f = _speck(dim, at, size)
    wl = geomgen.Workload("speck", dim, v, f, roots, levels, 2, 19 if dim == 3 else 9)
    # the distance, in cells, grows with the level: blocks at the edge of what exists are flagged and pull coarser ones
    d_spec = [float(max(wl.cell_size(l, a) for a in range(dim))) * (1 + 2 * l) for l in range(levels)]
    g = gpu_run(wl, d_spec=d_spec, own_bin=own_bin, n_prop=1 if own_bin else -1, with_links=False)
    coords = orc.gather(dim, v, f)
    ob = orc.bin_faces(dim, coords, wl.lo[:dim], wl.hi[:dim], wl.bins)
    of = orc.refine(dim, coords, ob, roots[:dim], levels, d_spec, wl.lo[:dim], wl.hi[:dim], own_bin=own_bin,
                    n_prop=1 if own_bin else -1)
    compare_forest(g, of, levels)
    marks = [np.bincount(l["mark"], minlength=4)[1:4].tolist() for l in g["levels"][:levels]]
    log(f"  {dim}D roots {roots[:dim]} L {levels} own_bin {own_bin}: blocks {[len(l['keys']) for l in g['levels']]}, "
        f"marks (flag, balance, propagation) {marks}")
