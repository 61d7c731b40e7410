"""Which passes build a cell may follow from the lists of the tessellation
before and from the other simulations of a batch; its results may not.  Irregular
points throughout: clusters hundreds of times denser than the mean, with
thousands of cells for the dense passes and cells handed from pass to pass."""
from __future__ import annotations

import time

import numpy as np
import pytest

import workloads as W
from gpu_common import compare_mesh, dev

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


@pytest.mark.parametrize("n,n_in", [(6000, 4500), (20000, 12000)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_mesh_does_not_follow_from_the_one_before(orc, precision, n, n_in):
    # A new context takes every dense cell in the two-cell pass; one whose last
    # mesh had none takes all lists in one launch, cell by cell; one whose last
    # mesh had a few dense cells takes most of them beyond the two-cell pass's
    # grid.  (What the passes hand on, which the call reports, may differ.)
    import paper_1707_05333_amd as M
    pos, _ = _cluster(n, n_in, seed=n)
    _case("mesh after others", n=n, precision=precision)
    p = M.make_params(box=BOX, precision=precision)
    mm = M.MovingMesh(n, p)
    mm.tessellate(dev(pos))
    mesh = _mesh(mm)
    om = orc.tessellate(pos, BOX, certificate=True)
    assert om.status == 0 and om.delta_min > 1e-12
    compare_mesh(mm, om, ftol=1e-9)
    few = W.jittered_lattice((17, 18, 17), BOX, jitter=0.2, seed=2)
    for dense in (0, 12):
        other = few.copy()
        other[:dense] = 0.52 + 1e-3 * (few[:dense] - 0.5)   # within one bucket
        mm = M.MovingMesh(n, p)
        mm.tessellate(dev(other))
        mm.tessellate(dev(pos))
        assert _unlike(_mesh(mm), mesh) == [], f"after {dense} dense cells"


@pytest.mark.parametrize("n,n_in", [(2400, 1400), (3600, 300), (6000, 4500)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_clustered_simulation_alone_and_in_a_mix(precision, n, n_in):
    import paper_1707_05333_amd as M
    pos, prim = _cluster(n, n_in, seed=n + 1)
    big = W.c1_uniform_random_velocity(n_side=17)   # 4,913 cells: an odd offset, other cells share a wavefront
    _case("clustered simulation", n=n, precision=precision)
    p = M.make_params(box=BOX, precision=precision)
    pb = M.make_params(box=big.box, precision=precision, **big.params)

    def run(before, beside):
        B = M.Batch(M.batch_footprint(20000, precision), max_sims=4, precision=precision)
        if before or beside:
            other = B.admit(pb, dev(big.pos), dev(big.prim))
        if before:
            B.step()
        if before and not beside:
            B.evict(other)
        s = B.admit(p, dev(pos), dev(prim))
        for _ in range(3):
            assert all(r["status"] == 0 for r in B.step())
        return B.read(s)

    alone = run(False, False)
    for before, beside in ((False, True), (True, True), (True, False)):
        assert _unlike(run(before, beside), alone) == [], (before, beside)


def test_many_small_simulations():
    # The table of the simulations and their reports go to the device and back
    # in many blocks.
    import paper_1707_05333_amd as M
    wl = W.c1_uniform_random_velocity(n_side=4)
    count, precision = 3000, "mixed"
    _case("many simulations", n=wl.n, count=count)
    B = M.Batch(M.batch_footprint(wl.n, precision) * count, max_sims=count, precision=precision)
    pos, prim = dev(wl.pos), dev(wl.prim)
    ids = [B.admit(M.make_params(box=wl.box, precision=precision, **{**wl.params, "cfl": 0.2 + 1e-5 * k}), pos, prim)
           for k in range(count)]
    for _ in range(2):
        rep = B.step()
    assert [r["sim"] for r in rep] == ids and all(r["status"] == 0 and r["steps"] == 2 for r in rep)
    for k in (0, 1, 255, 256, 1023, 1500, count - 1):
        A = M.Batch(M.batch_footprint(wl.n, precision) * 2, max_sims=1, precision=precision)
        s = A.admit(M.make_params(box=wl.box, precision=precision, **{**wl.params, "cfl": 0.2 + 1e-5 * k}), pos, prim)
        for _ in range(2):
            r, = A.step()
        assert rep[k]["dt"] == r["dt"] and rep[k]["t"] == r["t"]
        assert _unlike(A.read(s), B.read(ids[k])) == []


@pytest.mark.parametrize("fill", ["one spot", "nan"])
def test_refusal_of_an_overfull_bucket_is_quick(fill):
    # Every point in one bucket (a blown-up state: every position not a
    # number): refused, in a time of the order of a tessellation of as many
    # uniform points (2 ms; one thread that copied the bucket took 66 ms).
    import torch
    import paper_1707_05333_amd as M
    n = 262144
    _case("overfull bucket", n=n, fill=fill)
    mm = M.MovingMesh(n, M.make_params(box=BOX))

    def best(pos, fails):
        t = []
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            if fails:
                with pytest.raises(M.MMError) as e:
                    mm.tessellate(pos)
                assert e.value.name == ("MM_EINVAL" if fill == "nan" else "MM_ECAPACITY")
            else:
                mm.tessellate(pos)
            t.append(time.perf_counter() - t0)
        return min(t)

    if fill == "nan":
        bad = torch.full((n, 3), float("nan"), dtype=torch.float64, device="cuda")
    else:
        bad = dev(0.52 + 1e-5 * np.random.default_rng(1).uniform(-1, 1, (n, 3)))
    uniform = best(dev(W.poisson_points(n, BOX, seed=1)), False)
    refused = best(bad, True)
    print(f"uniform {1e3 * uniform:.2f} ms, refused {1e3 * refused:.2f} ms", flush=True)
    assert refused < 12 * uniform
