"""The checkpointed gradient, whose forward keeps its last segments' images and
tapes, equals the resident one bit for bit for one to five segments, a short
last one, with and without the second stream, and again when the backward is
repeated with nothing kept."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["f64", "f32"])
@pytest.mark.parametrize("steps,K", [(5, 8), (8, 8), (9, 8), (16, 8), (17, 8), (20, 8), (37, 8), (3, 1)])
@pytest.mark.parametrize("overlap", [True, False])
def test_kept_segments(steps, K, overlap, store):
    from paper_2407_01651_amd.adjoint import CheckpointedRun, ResidentRun
    w = workloads.small(nx=45, ny=33, seed=31)
    res = ResidentRun(w, store=store, steps=steps)
    m = res.forward(steps)
    lam = res.lam_from_macros(m["phi"], m["psi"] ** 3)
    ref, phi = res.backward(lam), m["phi"].clone()
    res.close()
    run = CheckpointedRun(w, store=store, K=K, overlap=overlap)
    for _ in range(2):
        m = run.forward(steps)
        assert torch.equal(m["phi"], phi) and run.sim.steps == steps
        assert torch.equal(run.backward(lam), ref)
    assert torch.equal(run.backward(lam), ref)
    run.close()
