"""Faces per workgroup of the bin count and scatter on both sides of the rule for few bins (at most 2,048, eight faces or
more to a bin): offsets and ids bit for bit those of the oracle, for faces of one bin and faces of up to 2^D bins, which
then fill more than one chunk of a workgroup."""
import numpy as np
import pytest

import geomgen
from _parity import compare_bins, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,B,faces", [(2, 1, (7, 8, 300, 5000)), (2, 45, (16199, 16200)), (2, 46, (16927, 16928)),
                                         (3, 1, (300, 5000)), (3, 2, (63, 64, 1000)), (3, 12, (13823, 13824)),
                                         (3, 13, (17575, 17576))])
@pytest.mark.parametrize("wide", [False, True])
def test_few_bins(orc, dim, B, faces, wide):
    import torch
    import paper_2502_16310_amd as agal
    dev = torch.device("cuda", 0)
    ctx = agal.Context()
    for n in faces:
        gen = geomgen.random_segments if dim == 2 else geomgen.random_triangles
        v, f = gen(n, 3, 0.1, 0.9, 0.45 / B if wide else 0.01 / B)
        geom = ctx.import_faces(torch.from_numpy(v).to(dev), torch.from_numpy(f).to(dev))
        off, ids = geom.bin_faces((0.0,) * dim, (1.0,) * dim, B).tensors()
        ob = orc.bin_faces(dim, orc.gather(dim, v, f), (0.0,) * dim, (1.0,) * dim, B)
        compare_bins({"offsets": off.cpu().numpy().view(np.uint32), "ids": ids.cpu().numpy()}, ob)
        log(f"  {dim}D {n} faces, {B}^{dim} bins: {ids.numel()} entries")
