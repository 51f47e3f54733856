"""The paper's own form of near-wall refinement on the GPU (Euclidean point-face test against the faces of
the cell centre's own bin, then mark propagation over rings of blocks) against the oracle's
orc_refine_own_bin: keys, leaf bits, marks (1 flagged, 2 balance, 3 propagation) and cell flags bit for
bit, over bin densities from the naive single bin to fine bins, the propagation rule and overrides, 2D
and 3D, the paper's constant distance, a non-dyadic domain; and link fractions on such a forest."""
import numpy as np
import pytest

import geomgen
from _parity import compare_forest, compare_links, gpu_run, log
from test_gpu_parity import _check_links

pytestmark = pytest.mark.gpu


def _check(orc, wl, B, d_spec, n_prop=-1, with_links=False):
    g = gpu_run(wl, B=B, d_spec=d_spec, own_bin=True, n_prop=n_prop, with_links=with_links)
    coords = orc.gather(wl.dim, wl.vertices, wl.faces)
    ob = orc.bin_faces(wl.dim, coords, wl.lo[:wl.dim], wl.hi[:wl.dim], B)
    of = orc.refine(wl.dim, coords, ob, wl.roots[:wl.dim], wl.levels, d_spec, wl.lo[:wl.dim], wl.hi[:wl.dim],
                    own_bin=True, n_prop=n_prop)
    compare_forest(g, of, wl.levels)
    marks = [np.bincount(l["mark"], minlength=4)[1:4].tolist() for l in g["levels"][:wl.levels]]
    log(f"  {wl.name} B={B} n_prop={n_prop}: blocks per level {[len(l['keys']) for l in g['levels']]}, "
        f"marks (flag, balance, propagation) per level {marks}")
    return g, of, coords, ob


@pytest.mark.parametrize("B", [1, 2, 8, 32])
def test_own_bin_circle(orc, B):
    wl = geomgen.workload("C0")
    _check(orc, wl, B, list(wl.d_spec()))


@pytest.mark.parametrize("B,n_prop", [(1, -1), (4, -1), (16, -1), (16, 0), (16, 2)])
def test_own_bin_sphere(orc, B, n_prop):
    v, f = geomgen.icosphere(3, 0.2)
    wl = geomgen.Workload("ico3", 3, v, f, (8, 8, 8), 3, B, 19)
    _check(orc, wl, B, list(wl.d_spec()), n_prop)


@pytest.mark.parametrize("B", [2, 8])
def test_own_bin_star_constant_distance(orc, B):
    """The paper's setting at a small scale: a star body, constant d = 0.05 over two passes (several
    block lengths, so several propagation steps)."""
    v, f = geomgen.star(4)
    wl = geomgen.Workload("star4", 3, v, f, (8, 8, 8), 2, B, 19)
    _check(orc, wl, B, [0.05, 0.05])


def test_own_bin_non_dyadic_domain_and_links(orc):
    v, f = geomgen.icosphere(3, 0.2)
    wl = geomgen.Workload("ico3-nd", 3, v, f, (5, 6, 4), 2, 7, 27, lo=(0.05, -0.02, 0.1), hi=(0.97, 1.01, 0.9))
    g, of, coords, ob = _check(orc, wl, 7, list(wl.d_spec()), with_links=True)
    lk = orc.link_fractions(3, coords, ob, of, 27)
    rep, _ = compare_links(g, lk, cells=64)
    _check_links(rep)


def test_own_bin_segments_2d(orc):
    v, f = geomgen.random_segments(200, 10, 0.05, 0.95, 0.1)
    wl = geomgen.Workload("rseg", 2, v, f, (5, 3, 1), 3, 9, 9)
    _check(orc, wl, 9, [0.02, 0.01, 0.005])


@pytest.mark.parametrize("dim,kind,B", [(3, "needles", 2), (3, "needles", 5), (3, "dots", 3), (2, "needles", 3), (3, "mixed", 1)])
def test_own_bin_box_rejection(orc, dim, kind, B):
    """Faces on both sides of the box rejection's limits: needles (no bound is claimed for slivers), specks far below
    the distance, and a mix with degenerate faces; bins of more and fewer than 64 faces."""
    rng = np.random.default_rng(8)
    n = 333
    c = rng.uniform(0.25, 0.75, (n, 1, dim))
    e = rng.normal(size=(n, 1, dim)) * (0.15 if kind != "dots" else 1e-6)
    t = rng.uniform(-0.5, 0.5, (n, dim, 1)) if kind != "dots" else rng.normal(size=(n, dim, 1))
    wide = 10.0 ** rng.uniform(-7, -1, (n, 1, 1)) if kind == "mixed" else 1e-4
    v = c + e * t + rng.normal(size=(n, dim, dim)) * wide * (0.0 if kind == "dots" else 1.0)
    if kind == "mixed":
        v[::7, 1] = v[::7, 0]
        v[::11] = v[::11, :1]
    v = v.reshape(-1, dim).astype(np.float32)
    f = np.arange(len(v), dtype=np.int32).reshape(n, dim)
    roots = (6, 6, 6) if dim == 3 else (6, 6, 1)
    wl = geomgen.Workload(f"{kind}{dim}d", dim, v, f, roots, 2, B, 19 if dim == 3 else 9)
    _check(orc, wl, B, [0.04, 0.015])
