"""The sums over nodes: the FP64 reduction against torch sums of the exported
state, and the initial-state gradient's sums against the oracle, on grids with
fewer nodes than a block, ragged ones, and more than one pass or stretch.

Both sides add the same FP64 values in another order: n terms of one sign agree
to n eps at worst, sqrt(n) eps in practice; the bars are 1e-12 of the sum of
magnitudes (n up to 2e6) and 1e-9 for the gradient."""
import pytest
import torch

import workloads
from adjoint_ref import flatten, init_vjp
from oracle import OracleParams, OracleSim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("dim,nx,ny,nz,over", [
    (2, 4, 4, 1, {}), (2, 33, 31, 1, {}), (2, 1000, 333, 1, {}), (2, 64, 50, 1, dict(phi_q=9)),
    (2, 60, 44, 1, dict(periodic=(False, False, True), symmetric=("lo", True, False), farfield=("hi", False, False))),
    (3, 5, 4, 6, {}), (3, 70, 41, 33, {}),
    (3, 30, 20, 18, dict(periodic=(False, False, False), symmetric=("lo", "lo", True), farfield=("hi", False, False))),
])
def test_reduction_matches_the_exported_state(dim, nx, ny, nz, over, store):
    import paper_2407_01651_amd as pfl
    w = workloads.small(dim=dim, nx=nx, ny=ny, nz=nz, seed=11, **over)
    sim = pfl.Sim(w, store=store)
    sim.init_fields()
    sim.step(2)
    st = sim.get_state()
    r = sim.reduce()
    sim.close()
    qn, qp, qs = (9, w["phi_q"], 5) if dim == 2 else (19, 7, 7)
    phi, psi, C = st[qn:qn + qp].sum(0), st[qn + qp:qn + qp + qs].sum(0), st[qn + qp + qs:qn + qp + 2 * qs].sum(0)
    gas = 1.0 - phi
    vol = float(gas.sum())

    def close(a, b, scale):
        assert abs(a - b) <= 1e-12 * max(float(scale), 1.0), (a, b)
    close(r["sum_phi"], float(phi.sum()), phi.abs().sum())
    close(r["gas_volume"], vol, phi.abs().sum())
    close(r["sum_C"], float(C.sum()), C.abs().sum())
    close(r["solid_fraction"], float(((psi + 1) / 2).mean()), 1.0)
    grid = torch.meshgrid(*[torch.arange(n, dtype=torch.float64, device="cuda") for n in gas.shape], indexing="ij")
    for a in range(dim):
        x = grid[dim - 1 - a]
        assert abs(r["gas_centroid"][a] * vol - float((gas * x).sum())) <= 1e-12 * float((phi.abs() * x).sum() + 1)
    assert not r["nonfinite"]


@pytest.mark.parametrize("nx,ny,store", [(64, 64, "f64"), (65, 64, "f64"), (300, 410, "f64"), (515, 512, "f32")])
def test_initial_gradient_sums(nx, ny, store):
    import paper_2407_01651_amd as pfl
    w = workloads.small(nx=nx, ny=ny, seed=12)
    w["bubbles"].append(dict(x=5.0, y=20.0, z=0.0, r=3.5))
    osim = OracleSim(OracleParams.from_workload(w))
    osim.init_fields()
    g = torch.Generator().manual_seed(5)
    lam0 = torch.rand(flatten(osim.state, workloads.FIELDS_ALL).shape, generator=g, dtype=torch.float64)
    if store == "f32":
        lam0 = lam0.float().double()
    ref = torch.tensor([float(v) for v in init_vjp(w, lam0)], dtype=torch.float64)
    sim = pfl.Sim(w, store=store, adjoint=True)
    sim.init_fields()
    dp = torch.zeros(3 + len(w["bubbles"]), dtype=torch.float64, device="cuda")
    sim.init_backward(lam0.to("cuda", sim.adj_dtype), dp)
    sim.close()
    assert float((dp[1:].cpu() - ref).abs().max()) <= 1e-9 * float(ref.abs().max())
