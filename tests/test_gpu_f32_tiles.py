"""The 2D FP32-compute step against the CPU oracle on grids at the edges of its
tiles (32 x 8, 32 x 4; 64 x 4 in 16-bit storage): smaller than a tile, one node
more, whole tiles only (each of them on the domain's edge and wholly inside),
and large enough for an interior tile.  Three steps: FP32 values come of some
1e2 dependent operations a step at 6e-8, so 2e-5 of the largest state value; a
16-bit population is off by at most 2^-11 of the largest deviation (about 1) a
step and a moment by at most nine of them, so 3 * 9 / 2048 = 1.3e-2."""
import pytest

import workloads
from parity_util import oracle_run, oracle_state, rel_err

pytestmark = pytest.mark.gpu

FIELDS = [("ns", "phi", "psi", "c", "theta"), ("psi", "c"), ("ns", "psi", "theta"), ("phi", "psi", "c", "theta")]
SYM = dict(periodic=(False, False, False), symmetric=("lo", True, False), farfield=("hi", False, False))
BOUND = {"f32": 2e-5, "f16": 1.4e-2}


@pytest.mark.parametrize("store", ["f32", "f16"])
@pytest.mark.parametrize("over", [{}, dict(periodic=(True, False, True)), SYM], ids=["periodic", "walls", "sym"])
@pytest.mark.parametrize("fields", FIELDS, ids="-".join)
@pytest.mark.parametrize("nx,ny", [(5, 4), (33, 9), (64, 16), (130, 26)])
def test_tiles(nx, ny, fields, over, store):
    import paper_2407_01651_amd as pfl
    if "theta" not in fields and "c" in fields:
        over = dict(over, Le=float("inf"), U0=-0.4, theta0=0.0)
    w = workloads.small(dim=2, nx=nx, ny=ny, nz=1, fields=fields, seed=31, **over)
    sim = pfl.Sim(w, store=store)
    sim.init_fields()
    sim.step(3)
    got = sim.get_state().cpu().double()
    ref = oracle_run(w, 3)
    sim.close()
    assert rel_err(got, oracle_state(ref, w["fields"])) < BOUND[store]
