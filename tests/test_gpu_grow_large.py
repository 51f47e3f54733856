"""Child generation over root grids above the size from which a wave takes 64 parents and goes through the children of
the marked ones: few marks, marks everywhere, and levels of both forms in one launch; a number of parents that fills no
whole wave.  Every level equals the oracle's."""
import numpy as np
import pytest

import geomgen
from _parity import compare_forest, gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,roots,levels,body,d", [
    (2, (517, 509, 1), 3, "speck", 1.0),
    (2, (517, 509, 1), 2, "ring", 1.0),
    (2, (517, 509, 1), 1, "square", 60.0),   # blocks within 60 cells of four long segments
    (3, (67, 61, 65), 2, "speck", 1.0),
    (3, (67, 61, 65), 1, "ring", 1.0),
])
def test_large_root_grids(orc, dim, roots, levels, body, d):
    at = (0.37, 0.61) if dim == 2 else (0.37, 0.61, 0.5)
    if body == "square":
        v, f = geomgen.square_loop((0.1, 0.1), (0.9, 0.9))
    elif dim == 2:
        v, f = geomgen.circle(64, 0.4 if body == "ring" else 0.0005, (0.5, 0.5) if body == "ring" else at)
    else:
        v, f = geomgen.icosphere(2, 0.3 if body == "ring" else 0.002, (0.5, 0.5, 0.5) if body == "ring" else at)
    assert np.prod(roots) > 1 << 18 and np.prod(roots) % 64
    wl = geomgen.Workload(body, dim, v, f, roots, levels, 64, 19 if dim == 3 else 9)
    d_spec = [d * float(max(wl.cell_size(l, a) for a in range(dim))) for l in range(levels)]
    g = gpu_run(wl, d_spec=d_spec, with_links=False)
    coords = orc.gather(dim, v, f)
    ob = orc.bin_faces(dim, coords, wl.lo[:dim], wl.hi[:dim], wl.bins)
    of = orc.refine(dim, coords, ob, roots[:dim], levels, d_spec, wl.lo[:dim], wl.hi[:dim])
    compare_forest(g, of, levels)
    n = [len(l["keys"]) for l in g["levels"]]
    log(f"  {body} {dim}D: blocks {n}")
    assert n[1] > 0
