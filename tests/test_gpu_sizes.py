"""Sizes at which a launch changes its path or fills its last tile: the
tessellation of every such size against the oracle's."""
from __future__ import annotations

import pytest

import workloads as W
from gpu_common import compare_mesh, mesh_pair

pytestmark = pytest.mark.gpu


# One block's scan covers 4,096 cells, one block's sort 8,192 points; a scan
# tile holds 2,048 items, a list slice 64 cells.
@pytest.mark.parametrize("n", [127, 2047, 2049, 4096, 4097, 8191, 8192, 8193])
def test_tessellation_at_path_edges(orc, n):
    box = (1.0, 1.0, 1.0)
    mm, info, om = mesh_pair(orc, W.poisson_points(n, box, seed=n), box)
    assert om.status == 0 and om.delta_min > 1e-12
    assert 2 * info["n_faces"] == len(om.j)
    # Poisson points have sliver faces, whose centroids carry rounding
    # amplified by nearly co-spherical generators (1e-9 of the cell scale, as
    # in the full-size samples).
    compare_mesh(mm, om, ftol=1e-9)


# Cells started from their six nearest sector neighbours: nearly exact
# lattices (all of them, bitwise as from the box), jittered ones (some, in
# rank order), a long box (tilted planes meet inside it), and points so
# irregular that most start from the box.
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape,jitter", [((12, 11, 10), 1e-3), ((11, 12, 13), 0.1), ((13, 10, 11), 0.3),
                                          ((48, 6, 6), 0.05), ((48, 6, 7), 0.25), ((9, 9, 9), 0.5)])
def test_lattice_starts(orc, shape, jitter, precision):
    box = tuple(s / shape[1] for s in shape)
    pos = W.jittered_lattice(shape, box, jitter=jitter, seed=31)
    mm, info, om = mesh_pair(orc, pos, box, precision=precision)
    assert om.status == 0 and om.delta_min > 1e-12
    compare_mesh(mm, om, ftol=1e-9)
