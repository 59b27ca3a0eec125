"""The autotuner's candidates differ from one another: streaming always is tried only where the option
changes the launch (a fused collisional pass with its candidates in a launch of their own), and the
shape it reports runs as the tuned run does."""
import re

import numpy as np
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


# slots above 16384 tiles with four particles a thread, above and below with eight
@pytest.mark.parametrize("slots,collisions,fused,want", [
    (100_000, True, True, {(4, 0), (8, 0)}),
    (20_000_000, True, True, {(4, 0), (4, 1), (8, 0)}),
    (40_000_000, True, True, {(4, 0), (4, 1), (8, 0), (8, 1)}),
    (40_000_000, False, True, {(4, 0), (8, 0)}),
    (40_000_000, True, False, {(4, 0), (8, 0)}),
])
def test_candidates(pic, capfd, monkeypatch, slots, collisions, fused, want):
    monkeypatch.setenv("PIC_AUTOTUNE_VERBOSE", "1")
    e = synth.ensemble(500, 20, collisions=collisions, seed=3, sort_every=5, extra=slots // 2)
    w = {"name": "t", "steps": 1, "precision": "fp32", "ensembles": [e]}
    a = pic.Sim(w, fused=fused)
    shape = a.autotune(2)
    tried = re.findall(r"ppt (\d) window (\d+) nt (\d) round", capfd.readouterr().err)
    assert {(int(p), int(nt)) for p, _, nt in tried} == want
    assert len(tried) == 2 * 3 * len(want)  # both rounds, three windows
    # a run of the reported shape goes on as the tuned one
    b = pic.Sim(w, fused=fused, **shape)
    b.load(a.save())
    a.step(7), b.step(7)
    for k in ("rho", "phi", "E"):
        assert np.array_equal(a.grid()[k], b.grid()[k]), k
    assert a.diag()["count"] == b.diag()["count"]
    a.close(), b.close()
