"""Which passes build a cell may follow from the lists of the tessellation
before and from the other simulations of a batch; its results may not.  Irregular
points throughout: clusters hundreds of times denser than the mean, with
thousands of cells for the dense passes and cells handed from pass to pass."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from gpu_common import dev

pytestmark = pytest.mark.gpu

BOX = (1.0, 1.0, 1.0)


def _case(what, **kw):
    print(f"[case] {what} {kw}", flush=True)


def _cluster(n, n_in, seed, width=0.03):
    rng = np.random.default_rng(seed)
    pos = W.poisson_points(n, BOX, seed=seed)
    pos[:n_in] = 0.5 + width * rng.standard_normal((n_in, 3)).clip(-4, 4)
    prim = np.ones((n, 5))
    prim[:, 1:4] = 0.1 * rng.standard_normal((n, 3))
    return pos, prim


def _mesh(mm):
    ex = mm.mesh_export()
    return [ex.V, ex.centroid, ex.face_i, ex.face_j, ex.face_code, ex.face_A, ex.face_f]


def _unlike(a, b):
    """Which of two lists of arrays differ."""
    import torch
    return [k for k, (x, y) in enumerate(zip(a, b)) if not torch.equal(x, y)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_dense_cells_do_not_follow_from_their_order(precision):
    # The dense buckets join their list in any order, so two tessellations pair
    # other cells in one wavefront.  The cells are bitwise the same, and built by
    # the same passes.
    import paper_1707_05333_amd as M
    pos, _ = _cluster(20000, 12000, seed=3)
    _case("order of the dense cells", n=len(pos), precision=precision)
    mm = M.MovingMesh(len(pos), M.make_params(box=BOX, precision=precision))
    info = mm.tessellate(dev(pos))
    mesh = _mesh(mm)
    for _ in range(5):
        assert mm.tessellate(dev(pos)) == info
        assert _unlike(_mesh(mm), mesh) == []


def test_lists_survive_the_component_calls():
    # The list lengths that size the next tessellation's passes are those of
    # the last tessellation, whatever calls come between: the same cells are
    # handed on, by the same passes.
    import paper_1707_05333_amd as M
    pos, prim = _cluster(20000, 12000, seed=3)
    _case("tessellate, cell_state, tessellate", n=len(pos))
    mm = M.MovingMesh(len(pos), M.make_params(box=BOX))
    first = mm.tessellate(dev(pos))
    mesh = _mesh(mm)
    Q = mm.init_charges(dev(prim))
    for _ in range(2):
        mm.cell_state(Q)
        assert mm.tessellate(dev(pos)) == first
        assert _unlike(_mesh(mm), mesh) == []
