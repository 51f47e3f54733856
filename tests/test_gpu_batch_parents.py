"""The batched link step's two ways to find a block within one plan: a body whose parents' grid is above the dense
table's limit (hash table, cleared in every run) beside bodies below it, over several runs with the vertices moved
between them; identical to the single-body calls each time."""
import numpy as np
import pytest

import geomgen
from _parity import log
from test_gpu_batch import _cfg, _same_as_plain, _tensors

pytestmark = pytest.mark.gpu


def test_hash_and_dense_parents_in_one_batch():
    import torch
    import paper_2502_16310_amd as agal
    def bodies(shift):
        out = []
        for name, roots, levels, r in (("hash", (33, 32, 1), 8, 0.003), ("dense", (32, 32, 1), 8, 0.002), ("small", (5, 3, 1), 2, 0.2)):
            v, f = geomgen.circle(41, r, (0.511 + shift * r, 0.497))
            out.append(geomgen.Workload(name, 2, v, f, roots, levels, 16, 9))
        return out
    wls = bodies(0.0)
    assert 33 * 32 << 14 > 1 << 24 >= 32 * 32 << 14
    ts = [_tensors(w) for w in wls]
    ctx = agal.Context()
    ctx.set_link_list_limit(1 << 30)
    bt = agal.Batch([(v, f, _cfg(w, w.bins)) for w, (v, f) in zip(wls, ts)], tune_bins=False, tune_grid=False,
                    capacity_margin=1.0, ctx=ctx)
    for shift in (0.0, 0.3, -0.7, 0.0):
        now = bodies(shift)
        for w, (v, _) in zip(now, ts):
            v.copy_(torch.from_numpy(np.ascontiguousarray(w.vertices)))
        bt.run()
        bt.status()
        nodes = [len(_same_as_plain(bt, i, w)["key"]) for i, w in enumerate(now)]
        log(f"  shift {shift}: {nodes} nodes")
        assert all(nodes)
