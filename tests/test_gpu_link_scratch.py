"""Device memory that the list-mode link step takes unseen: candidate lists up to 512 MiB are allocated from the bound
(faces x blocks of the largest face), longer ones at their exact length after a host wait.  One face over the whole grid
among many small ones makes the bound a thousand times the lists."""
import numpy as np
import pytest

import geomgen
from _parity import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("faces", [20000, 24000, 30000])
def test_lists_allocated_from_the_bound(faces):
    import torch
    import paper_2502_16310_amd as agal
    v, f = geomgen.random_triangles(faces, 4, 0.1, 0.9, 0.005)
    v = v.copy()
    v[f[0]] = np.array([[0.01, 0.01, 0.01], [0.99, 0.99, 0.01], [0.99, 0.01, 0.99]], np.float32)
    ctx = agal.Context()
    ctx.set_link_list_limit(1 << 30)
    dev = torch.device("cuda", 0)
    geom = ctx.import_faces(torch.from_numpy(v).to(dev), torch.from_numpy(f).to(dev))
    lo, hi = (0.0,) * 3, (1.0,) * 3
    forest = agal.Forest(geom, geom.bin_faces(lo, hi, 10), 3, (10, 10, 10), 0, [], lo, hi)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    links = forest.link_fractions(19)
    peak = torch.cuda.max_memory_allocated() - before
    log(f"  {faces} faces: bound {faces * 2197 / 1e6:.0f} M entries, {links.n_nodes} nodes, peak {peak / 2 ** 20:.0f} MiB")
    assert 0 < links.n_nodes <= 64000
    # beside the lists: 160 B of results and 24 B of scratch for each of at most 64,000 cells
    assert peak <= (512 + 16) << 20
