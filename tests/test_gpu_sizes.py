"""Sizes at which a launch changes its path or fills its last tile: the
tessellation of every such size against the oracle's."""
from __future__ import annotations

import ctypes

import numpy as np
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


# The component calls write the caller's rows directly, unless an output lies
# over an input (or over the other output): the results are the same bits.
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_component_outputs_over_inputs(orc, precision):
    torch = pytest.importorskip("torch")
    shape, box = (11, 9, 10), (1.0, 1.0, 1.0)
    mm, _, _ = mesh_pair(orc, W.jittered_lattice(shape, box, jitter=0.2, seed=5), box, precision=precision)
    n = mm.n
    rng = torch.Generator().manual_seed(3)
    prim = torch.rand(n, 5, generator=rng, dtype=torch.float64).add(0.5).to(mm.device)
    Q = mm.init_charges(prim)
    U, w, dt, _ = mm.cell_state(Q)
    G = mm.gradients(U)
    Uh = mm.predict(U, G, w, dt)
    rs, dptr = U.element_size(), lambda t, at=0: ctypes.c_void_p(t.data_ptr() + at)

    def state(buf, u_at, w_at, q):
        d = ctypes.c_double()
        mm._check(mm.lib.mm_cell_state(mm.ctx, dptr(q), dptr(buf, u_at), dptr(buf, w_at), ctypes.byref(d), None))
        assert d.value == dt
        return buf

    # U over the charges, w behind them; then w over the charges.
    for u_at, w_at in ((0, 40 * n), (40 * n, 0)):
        buf = torch.zeros(80 * n, dtype=torch.uint8, device=mm.device)
        buf[:40 * n].view(torch.float64).copy_(Q.view(-1))
        state(buf, u_at, w_at, buf)
        assert torch.equal(buf[u_at:u_at + 5 * rs * n].view(U.dtype).view(n, 5), U)
        assert torch.equal(buf[w_at:w_at + 24 * n].view(torch.float64).view(n, 3), w)
    # The half-step state over the state, and over the gradients.
    for over in (U, G):
        a = [t.clone() for t in (U, G)]
        out = a[0] if over is U else a[1]
        mm._check(mm.lib.mm_predict(mm.ctx, dptr(a[0]), dptr(a[1]), dptr(w), float(dt), dptr(out)))
        assert torch.equal(out.view(-1)[:5 * n].view(n, 5), Uh)


# Cells that go on after their first radius take only the points near their
# farthest vertices: irregular points in few buckets a side, in a long box, and
# a cluster of dense buckets on a thin background.
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,box,cluster", [(130, (1.0, 1.0, 1.0), 0), (700, (3.0, 1.0, 1.0), 0),
                                           (2500, (1.0, 1.5, 1.0), 0), (2400, (1.0, 1.0, 1.0), 1400)])
def test_shells_after_the_first(orc, n, box, cluster, precision):
    pos = W.poisson_points(n, box, seed=17 + n)
    if cluster:
        rng = np.random.default_rng(n)
        pos[:cluster] = 0.5 + 0.03 * rng.standard_normal((cluster, 3)).clip(-4, 4)
    mm, info, om = mesh_pair(orc, pos, box, precision=precision)
    assert om.status == 0 and om.delta_min > 1e-12
    compare_mesh(mm, om, ftol=1e-9)
