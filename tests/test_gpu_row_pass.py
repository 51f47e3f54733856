"""The row pass's last wave: node counts with every remainder by the four elements of a 16-byte store, and waves of few
nodes, for each lattice.  List mode must write the walk mode's rows bit for bit (its kernel places them another way)."""
import numpy as np
import pytest

import geomgen
from _parity import gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,lattice", [(2, 9), (3, 19), (3, 27)])
def test_last_wave_of_rows(dim, lattice):
    import paper_2502_16310_amd as agal
    walk, lists = agal.Context(), agal.Context()
    walk.set_link_list_limit(0)
    lists.set_link_list_limit(1 << 30)
    rests, counts = set(), []
    for k in range(8):
        v, f = geomgen.circle(40 + 3 * k, 0.11 + 0.013 * k, (0.51, 0.47 + 0.003 * k)) if dim == 2 else geomgen.star(2)
        if dim == 3:
            v = (0.5 + (v - 0.5) * (0.2 + 0.07 * k)).astype(np.float32)   # from a few cells to much of the grid
        wl = geomgen.Workload("rows", dim, v, f, (4, 4, 4 if dim == 3 else 1), 2, 8, lattice)
        d_spec = [float(max(wl.cell_size(l, a) for a in range(dim))) for l in range(2)]
        gw, gl = gpu_run(wl, ctx=walk, d_spec=d_spec), gpu_run(wl, ctx=lists, d_spec=d_spec)
        assert len(gl["key"]) > 0
        assert np.array_equal(gw["key"], gl["key"]) and np.array_equal(gw["face"], gl["face"])
        assert np.array_equal(gw["q"].view(np.int32), gl["q"].view(np.int32))
        counts.append(len(gl["key"]))
        rests.add(len(gl["key"]) % 4)
    log(f"  D{dim}Q{lattice}: nodes {counts}")
    assert len(rests) >= 2


@pytest.mark.parametrize("dim,lattice,roots,levels", [(2, 9, (64, 64, 1), 4), (3, 19, (6, 6, 6), 3), (3, 27, (6, 6, 6), 3)])
def test_waves_in_runs_per_xcd(dim, lattice, roots, levels):
    """More than the 256 waves of one full group of runs, and a partial group behind it."""
    import paper_2502_16310_amd as agal
    walk, lists = agal.Context(), agal.Context()
    walk.set_link_list_limit(0)
    lists.set_link_list_limit(1 << 30)
    v, f = geomgen.circle(200, 0.4, (0.5, 0.5)) if dim == 2 else geomgen.star(4)
    wl = geomgen.Workload("rows", dim, v, f, roots, levels, 32, lattice)
    d_spec = [float(max(wl.cell_size(l, a) for a in range(dim))) for l in range(levels)]
    gw, gl = gpu_run(wl, ctx=walk, d_spec=d_spec), gpu_run(wl, ctx=lists, d_spec=d_spec)
    log(f"  D{dim}Q{lattice}: {len(gl['key'])} nodes")
    assert len(gl["key"]) > 256 * 32 + 1
    assert np.array_equal(gw["key"], gl["key"]) and np.array_equal(gw["face"], gl["face"])
    assert np.array_equal(gw["q"].view(np.int32), gl["q"].view(np.int32))
