"""The 3D step's own choice of z planes per workgroup gives the state of one
chunk per column, bit for bit: chunks of one plane, chunks with a remainder,
more chunks than one round of workgroups holds, and walls, symmetry planes and
far-field sides in z."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("store", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny,nz,over", [
    (18, 12, 4, {}),                                    # one plane a chunk
    (33, 17, 131, {}),                                  # a remainder
    (180, 170, 24, {}),                                 # several planes, a remainder
    (40, 20, 50, dict(periodic=(True, False, False))),  # walls in z
    (40, 20, 50, dict(periodic=(False, False, False), symmetric=("lo", "lo", "lo"), farfield=("hi", "hi", "hi"),
                      fields=("psi", "c", "theta"), bubbles=[])),
])
def test_chosen_chunks_give_the_state_of_one_chunk(nx, ny, nz, over, store, monkeypatch):
    import paper_2407_01651_amd as pfl
    w = workloads.small(dim=3, nx=nx, ny=ny, nz=nz, seed=7, **over)
    states = []
    for chunk in (None, str(nz)):
        if chunk is None:
            monkeypatch.delenv("PFL_ZCHUNK", raising=False)
        else:
            monkeypatch.setenv("PFL_ZCHUNK", chunk)
        sim = pfl.Sim(w, store=store)
        sim.init_fields()
        sim.step(5)
        states.append((sim.get_state().cpu(), sim.macros()["vx"].cpu()))
        sim.close()
    assert all(torch.equal(a, b) for a, b in zip(*states))


@pytest.mark.parametrize("store", ["f16", "bf16"])
def test_chunks_agree_on_a_state_beyond_the_last_level_cache(store, monkeypatch):
    """The step touches the next plane's rows ahead on such a state (2 x 159 MB): ragged
    tiles, chunks with a remainder and the last planes of a chunk and of the grid."""
    import paper_2407_01651_amd as pfl
    w = workloads.small(dim=3, nx=131, ny=133, nz=67, seed=8)
    states = []
    for chunk in (None, "67", "9"):
        if chunk is None:
            monkeypatch.delenv("PFL_ZCHUNK", raising=False)
        else:
            monkeypatch.setenv("PFL_ZCHUNK", chunk)
        sim = pfl.Sim(w, store=store)
        assert 2 * (sim.sizes.pops_bytes + sim.sizes.hist_bytes) > 256 << 20
        sim.init_fields()
        sim.step(3)
        states.append(sim.get_state())
        sim.close()
    assert torch.equal(states[0], states[1]) and torch.equal(states[0], states[2])
