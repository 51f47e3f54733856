"""Canonical order of the binning at the sizes where its sorts change.

Bins of 1, 2, 63..65 ids (rank sort | sorting network), around the network's
powers of two, and 2047..2049 ids (network | ordered sweep), placed so that
groups of 64 bins hold less and more than one LDS segment and, with many bins,
several groups per wave.  Offsets and ids must equal the oracle's exactly."""
import numpy as np
import pytest

import oracle
from _parity import log

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 63, 64, 65, 66, 127, 128, 129, 255, 257, 1000, 1024, 1025, 2047, 2048, 2049]


def _faces_in_bins(dim, B, bins, sizes, seed):
    """A coordinate list of tiny faces, sizes[i] of them strictly inside bin bins[i], in shuffled order."""
    rng = np.random.default_rng(seed)
    which = rng.permutation(np.repeat(bins, sizes))
    ix = np.stack([(which // B ** a) % B for a in range(dim)], 1)
    c = (ix + 0.5 + rng.uniform(-0.3, 0.3, ix.shape)) / B
    v = c[:, None, :] + rng.uniform(-0.05, 0.05, (len(which), dim, dim)) / B
    return v.astype(np.float32)


@pytest.mark.parametrize("dim,B,stride", [(2, 16, 1), (2, 16, 14), (3, 8, 27), (3, 96, 1), (3, 96, 48000), (2, 3, 1)])
def test_bins_at_the_sorts_edges(dim, B, stride):
    import torch
    import paper_2502_16310_amd as agal
    nb = B ** dim
    sizes = SIZES if nb >= len(SIZES) else SIZES[-nb:]
    bins = 1 + stride * np.arange(len(sizes)) if nb > len(SIZES) else np.arange(nb)
    assert bins.max() < nb
    v = _faces_in_bins(dim, B, bins, sizes, 11)
    log(f"dim {dim} B {B} stride {stride}: {len(v)} faces")
    coords = v.reshape(len(v), dim * dim)
    ref = oracle.bin_faces(dim, coords, (0.0,) * dim, (1.0,) * dim, B)
    ctx = agal.Context()
    g = ctx.import_faces(torch.from_numpy(v.reshape(-1, dim)).cuda())
    for kind in ("box", "sampled"):
        b = g.bin_faces([0.0] * dim, [1.0] * dim, B) if kind == "box" else \
            g.bin_faces_discrete([0.0] * dim, [1.0] * dim, B, spacing=1.0)
        off, ids = b.tensors()
        # the faces lie inside one bin each, so sampled points give the same bins
        assert np.array_equal(off.cpu().numpy().view(np.uint32), ref.offsets.astype(np.uint32)), kind
        assert np.array_equal(ids.cpu().numpy(), ref.ids.astype(np.int32)), kind


@pytest.mark.parametrize("what,B", [("box", 40), ("box", 1), ("wide", 16), ("wide", 33), ("many", 32), ("many", 1),
                                    ("many", 3), ("segments", 64), ("one", 12)])
def test_pairs_over_chunks_and_workgroups(what, B):
    """Count and scatter where a face has more pairs than one chunk, where a workgroup takes one face and where it
    takes many, with the last workgroup part full, and where every pair falls in few bins."""
    import geomgen
    import torch
    import paper_2502_16310_amd as agal
    if what == "box":
        v, f = geomgen.box_mesh()
    elif what == "wide":
        v, f = geomgen.random_triangles(1777, 5, size=0.25)
    elif what == "many":
        v, f = geomgen.random_triangles(150001, 6, size=0.004)
    elif what == "segments":
        v, f = geomgen.random_segments(5003, 7, size=0.1)
    else:
        v, f = np.array([[-0.2, 0.1, 0.1], [1.3, 0.2, 0.9], [0.4, 1.1, 0.3]], np.float32), np.array([[0, 1, 2]], np.int32)
    dim = v.shape[1]
    log(f"{what} B {B}: {len(f)} faces")
    ref = oracle.bin_faces(dim, oracle.gather(dim, v, f), (0.0,) * dim, (1.0,) * dim, B)
    g = agal.Context().import_faces(torch.from_numpy(v).cuda(), torch.from_numpy(f).cuda())
    off, ids = g.bin_faces([0.0] * dim, [1.0] * dim, B).tensors()
    assert np.array_equal(off.cpu().numpy().view(np.uint32), ref.offsets)
    assert np.array_equal(ids.cpu().numpy(), ref.ids)
