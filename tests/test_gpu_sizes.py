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
