"""Steps that fail in their update: a start state that is finite, with one
cell so hot that its fluxes overflow (pressure times velocity beyond the type's
range), or an entropy charge that is not a number.  The update has then written
the caller's arrays, and the call puts them back: positions, charges and
entropy charges are bitwise those before the call, and so are the Mach numbers
of the call before.  The mesh velocities of a single simulation, which may hold
partial results after an error, show that the update ran."""
import numpy as np
import pytest

import workloads as W
from gpu_common import dev, host

pytestmark = pytest.mark.gpu

MM_ENONFINITE = -5   # mm_status of include/mm.h
HOT = {"fp64": 1e230, "mixed": 1e30}   # pressure whose 3/2 power overflows
UNSET = -7.0


def _case(what, **kw):
    print(f"[case] {what} {kw}", flush=True)


def _hot(wl, P, cell=37):
    prim = wl.prim.copy()
    prim[cell, 4] = P
    return prim


def _start(M, wl, prec, P, **params):
    """A context, positions, charges (one cell hot) and unset velocities."""
    import torch
    mm = M.MovingMesh(wl.n, M.make_params(box=wl.box, precision=prec, **{**wl.params, **params}))
    pos = dev(wl.pos)
    mm.tessellate(pos)
    prim = dev(_hot(wl, P))
    Q = mm.init_charges(prim)
    assert bool(torch.isfinite(Q).all())
    return mm, pos, Q, torch.full_like(pos, UNSET), prim


def _fails_in_update(M, call, keep, w):
    """call() fails as non-finite, after its update wrote some of w; the
    arrays in keep hold the bits they held."""
    before = [host(t).copy() for t in keep]
    with pytest.raises(M.MMError) as e:
        call()
    assert e.value.name == "MM_ENONFINITE"
    assert bool((w != UNSET).any())
    for t, b in zip(keep, before):
        assert np.array_equal(host(t).view(np.uint8), b.view(np.uint8))


@pytest.mark.parametrize("half_step_mesh", [0, 1])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_step_is_undone(prec, half_step_mesh):
    import paper_1707_05333_amd as M
    wl = W.c1_uniform_random_velocity(n_side=9)
    _case("step", prec=prec, half=half_step_mesh, n=wl.n)
    mm, pos, Q, w, _ = _start(M, wl, prec, HOT[prec], half_step_mesh=half_step_mesh)
    _fails_in_update(M, lambda: mm.step(pos, w, Q), [pos, Q], w)
    Q[37] = Q[38]   # repaired, it steps
    mm.step(pos, w, Q)
    assert np.isfinite(host(Q)).all()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_static_step_is_undone(prec):
    import paper_1707_05333_amd as M
    wl = W.c1_uniform_random_velocity(n_side=9)
    _case("static step", prec=prec, n=wl.n)
    mm, pos, Q, w, _ = _start(M, wl, prec, HOT[prec])
    _fails_in_update(M, lambda: M.step_static(mm.params, pos, w, Q), [pos, Q], w)


@pytest.mark.parametrize("what", ["flux", "entropy"])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_entropy_step_is_undone(prec, what):
    import paper_1707_05333_amd as M
    import torch
    wl = W.c1_uniform_random_velocity(n_side=9)
    _case("entropy step", prec=prec, n=wl.n, overflow=what)
    mm, pos, Q, w, prim = _start(M, wl, prec, HOT[prec] if what == "flux" else 1.0, mach_threshold=1.1)
    S = mm.init_entropy(prim)
    if what == "entropy":
        S[37] = float("nan")
    mach = torch.full((wl.n,), -3.0, dtype=torch.float32, device="cuda")
    _fails_in_update(M, lambda: mm.step_entropy(pos, w, Q, S, mach), [pos, Q, S, mach], w)
