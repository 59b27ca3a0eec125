"""Contexts freed while a stream is being captured: the page-locked block that contexts share is
given back with the last of them, and must not spoil a graph that is being captured then."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_28534_amd as P

    P.load_library()
    return P


# beyond 64 contexts each locks a page of its own
@pytest.mark.parametrize("contexts", [1, 2, 66])
def test_free_during_capture(pic, contexts):
    import gc

    import torch

    gc.collect()
    e = synth.ensemble(64, 20, collisions=True, seed=4)
    w = {"name": "t", "steps": 1, "precision": "fp32", "ensembles": [e]}
    sims = [pic.Sim(w) for _ in range(contexts)]
    for s in sims[:2]:
        s.step(2)
    x = torch.zeros(1000, device="cuda")
    x += 1.0
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x += 1.0
        for s in reversed(sims):
            s.close()
        x *= 2.0
    want = 1.0
    for _ in range(3):
        g.replay()
        want = (want + 1.0) * 2.0
        assert torch.equal(x, torch.full_like(x, want))
    # and a context made afterwards works
    sim = pic.Sim(w)
    sim.step(2)
    assert sim.diag()["step"] == 2
    sim.close()
