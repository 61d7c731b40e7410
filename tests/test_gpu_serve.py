"""The serving loop's count of resident simulations, with arrivals that overlap,
or do not, by construction (all at the start, or far apart against a step)."""
import pytest

import workloads as W
from gpu_common import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_sims,arrivals,resident,batch_steps", [
    (8, [0.0] * 6, 6, 3),                  # room for all: every one in each step
    (2, [0.0] * 6, 2, 9),                  # two at a time
    (1, [0.0] * 3, 1, 9),
    (8, [0.0, 0.2, 0.4], 1, 9),            # each gone long before the next arrives
    (8, [0.0, 0.0, 0.2, 0.2, 0.2], 3, 6),
])
def test_resident_simulations(max_sims, arrivals, resident, batch_steps):
    import paper_1707_05333_amd as M
    prec, wl = "mixed", W.c1_uniform_random_velocity(n_side=8)
    print(f"[case] serve max_sims {max_sims} arrivals {arrivals}", flush=True)
    B = M.Batch(M.batch_footprint(wl.n, prec) * 8, max_sims=max_sims, precision=prec)
    p, pos, prim = M.make_params(box=wl.box, precision=prec, **wl.params), dev(wl.pos), dev(wl.prim)
    B.serve([dict(arrival=0.0, params=p, pos=pos, prim=prim, steps=1)])   # (kernels loaded)
    res, stats = B.serve([dict(arrival=t, params=p, pos=pos, prim=prim, steps=3) for t in arrivals])
    assert all(r["status"] == 0 and r["steps"] == 3 for r in res)
    assert stats["max_resident"] == resident and stats["batch_steps"] == batch_steps
    assert B.usage()["sims"] == 0
