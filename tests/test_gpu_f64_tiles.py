"""The FP64 step kernels against the CPU oracle on grids at the edges of their
tiles (2D 32 x 8 and 32 x 4, 3D 32 x 8 columns): smaller than a tile, one node
less and more, and large enough for an interior tile with the fast addressing,
for every field combination they are built for.  Three steps of both sides in
FP64 differ by rounding alone: some 1e3 operations a step at 1.1e-16, so 1e-12
of the largest state value."""
import pytest
import torch

import workloads
from parity_util import oracle_run, oracle_state, rel_err

pytestmark = pytest.mark.gpu

F2 = [("ns", "phi", "psi", "c", "theta"), ("psi", "c"), ("psi", "c", "theta"), ("ns", "phi"),
      ("phi", "psi", "c", "theta"), ("psi",), ("phi",), ("ns", "psi", "theta"), ("ns", "psi", "c", "theta"),
      ("psi", "theta")]
F3 = [F2[0], F2[1], F2[2], F2[3], F2[5], F2[6], F2[7]]
SYM = dict(periodic=(False, False, False), symmetric=("lo", True, "lo"), farfield=("hi", False, "hi"))


def _check(w):
    import paper_2407_01651_amd as pfl
    sim = pfl.Sim(w, store="f64")
    sim.init_fields()
    sim.step(3)
    got = sim.get_state().cpu()
    ref = oracle_run(w, 3)
    sim.close()
    assert rel_err(got, oracle_state(ref, w["fields"])) < 1e-12


def _workload(dim, nx, ny, nz, fields, seed, **over):
    if "theta" not in fields and "c" in fields:
        over.update(Le=float("inf"), U0=-0.4, theta0=0.0)
    w = workloads.small(dim=dim, nx=nx, ny=ny, nz=nz, fields=fields, seed=seed, **over)
    if "psi" not in fields:
        w["seeds"] = []
    return w


@pytest.mark.parametrize("fields", F2, ids="-".join)
@pytest.mark.parametrize("nx,ny", [(4, 4), (31, 7), (33, 9), (70, 26)])
def test_2d_tiles(nx, ny, fields):
    _check(_workload(2, nx, ny, 1, fields, 21))


@pytest.mark.parametrize("nx,ny,over", [(33, 9, dict(phi_q=9)), (70, 26, dict(phi_q=9)), (33, 9, SYM),
                                        (70, 26, dict(SYM, phi_q=9)), (70, 26, dict(aac_form="le1")),
                                        (40, 30, dict(th_rho_g=0.7, th_cp_g=0.9, th_k_g=0.5))])
def test_2d_forms(nx, ny, over):
    _check(_workload(2, nx, ny, 1, F2[0], 22, **over))


@pytest.mark.parametrize("fields", F3, ids="-".join)
@pytest.mark.parametrize("nx,ny,nz", [(4, 4, 4), (33, 9, 5), (70, 22, 6)])
def test_3d_tiles(nx, ny, nz, fields):
    _check(_workload(3, nx, ny, nz, fields, 23))


@pytest.mark.parametrize("nx,ny,nz,over", [(33, 9, 5, dict(periodic=(True, True, False))), (33, 9, 5, SYM), (70, 22, 6, SYM),
                                           (70, 22, 6, dict(aac_form="le1")),
                                           (30, 12, 6, dict(th_rho_g=0.7, th_cp_g=0.9, th_k_g=0.5))])
def test_3d_forms(nx, ny, nz, over):
    _check(_workload(3, nx, ny, nz, F3[0], 24, **over))
