"""A batched body whose face comes to span more bins than any face of the plan: the plan takes two faces per workgroup,
then one face is moved to cover every bin (more than 2^24 of them) while the others shrink to about a bin each, so that
the (face, bin) pairs stay within the plan's capacity.  Bin walks (flags and links) must still find the face everywhere:
identical to the single-body calls, before and after."""
import numpy as np
import pytest

import geomgen
from _parity import log
from test_gpu_batch import _cfg, _same_as_plain, _tensors

pytestmark = pytest.mark.gpu


def test_face_over_all_bins_of_a_planned_batch():
    import torch
    import paper_2502_16310_amd as agal
    B, n = 320, 10000
    assert B ** 3 > 1 << 24
    rng = np.random.default_rng(8)
    e = 5.9 / B   # boxes of up to 7 bins an axis
    c = rng.uniform(0.05, 0.93, (n, 1, 3))
    small = (c + e * np.array([[0, 0, 0], [1, 1, 0], [1, 0, 1]])).astype(np.float32)
    f = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    wl = geomgen.Workload("spread", 3, small.reshape(-1, 3), f, (8, 8, 8), 1, B, 19)
    moved = (small + (c - small) * 0.99).astype(np.float32)
    moved[0] = [[1e-4, 1e-4, 1e-4], [0.9999, 0.9999, 1e-4], [0.9999, 1e-4, 0.9999]]
    wide = geomgen.Workload("wide", 3, moved.reshape(-1, 3), f, (8, 8, 8), 1, B, 19)
    ctx = agal.Context()
    ctx.set_link_list_limit(0)
    ctx.set_flag_table_limit(0)
    v, ft = _tensors(wl)
    bt = agal.Batch([(v, ft, _cfg(wl, B))], tune_bins=False, tune_grid=False, capacity_margin=11.0, ctx=ctx)
    log(f"case wide face: {n} faces, {B}^3 bins")
    bt.run()
    bt.status()
    _same_as_plain(bt, 0, wl)
    v.copy_(torch.from_numpy(wide.vertices))
    for _ in range(2):
        bt.run()
        bt.status()
        _same_as_plain(bt, 0, wide)
