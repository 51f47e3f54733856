"""The link step's two ways to find a block (dense parent table, hash table of parents), on either side of the line
between them: a grid of parents just below and just above the dense table's limit, one level only, and parents with
odd counts per axis.  List mode must give the walk mode's links, and those the oracle's."""
import numpy as np
import pytest

import geomgen
from _parity import compare_links, gpu_run, log
from test_gpu_parity import _check_links

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,roots,levels", [(2, (32, 32, 1), 8), (2, (33, 32, 1), 8), (2, (5, 3, 1), 1), (3, (5, 3, 4), 1),
                                              (3, (3, 5, 2), 3), (3, (17, 1, 1), 4)])
def test_dense_and_hash_parent_tables(orc, dim, roots, levels):
    import paper_2502_16310_amd as agal
    # 2D, 8 passes: 4096^2 parents are the limit of 2^24, 4224 x 4096 are above it
    v, f = geomgen.circle(37, 0.003, (0.511, 0.497)) if levels == 8 else \
        (geomgen.circle(61, 0.3) if dim == 2 else geomgen.star(2))
    wl = geomgen.Workload("parents", dim, v, f, roots, levels, 16, 9 if dim == 2 else 27)
    d_spec = [float(max(wl.cell_size(l, a) for a in range(dim))) for l in range(levels)]
    walk, lists = agal.Context(), agal.Context()
    walk.set_link_list_limit(0)
    lists.set_link_list_limit(1 << 30)
    gw, gl = gpu_run(wl, ctx=walk, d_spec=d_spec), gpu_run(wl, ctx=lists, d_spec=d_spec)
    for k in ("key", "q", "face"):
        assert np.array_equal(gw[k], gl[k]), k
    coords = orc.gather(dim, v, f)
    ob = orc.bin_faces(dim, coords, wl.lo[:dim], wl.hi[:dim], wl.bins)
    of = orc.refine(dim, coords, ob, roots[:dim], levels, d_spec, wl.lo[:dim], wl.hi[:dim])
    rep, _ = compare_links(gl, orc.link_fractions(dim, coords, ob, of, wl.lattice), cells=4 ** dim)
    _check_links(rep)
    log(f"  {dim}D roots {roots[:dim]} L {levels}: {len(gl['key'])} nodes")
    assert len(gl["key"]) > 0
