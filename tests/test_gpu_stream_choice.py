"""The pass's choice between cached and non-temporal particle streams changes no result: a run on
either side of 1e7 slots in use (and one that crosses it by injection and by a restart) against
the same run with non-temporal streams asked for."""
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


def same(a, b):
    da, db = a.diag(), b.diag()
    for q in ("count", "coll", "created", "wall_count", "pushes", "numax", "emax", "step"):
        assert da[q] == db[q], q
    ga, gb = a.grid(), b.grid()
    for q in ("rho", "phi", "E"):
        assert np.array_equal(ga[q], gb[q]), q
    for s in range(2):
        assert np.array_equal(ga["Q"][s], gb["Q"][s]), s


@pytest.mark.parametrize("ppc,collisions,fused", [(100, True, True), (126, True, True), (126, False, True),
                                                  (126, True, False)])
def test_stream_choice_changes_nothing(pic, ppc, collisions, fused):
    e = synth.ensemble(40_000, ppc, collisions=collisions, seed=5, sort_every=3, cap_factor=3.0)
    w = {"name": "t", "steps": 1, "precision": "fp32", "ensembles": [e]}
    a, b = pic.Sim(w, fused=fused), pic.Sim(w, fused=fused, nontemporal=1)
    for n in (2, 6):
        a.step(n), b.step(n)
        same(a, b)
    c = pic.Sim(w, fused=fused)
    c.load(a.save())
    for x in (b, c):
        x.step(4)
    same(b, c)
    # few particles in the same capacity
    st = synth.random_state(e, [30_000, 20_000], seed=8)
    for x in (b, c):
        x.set_state(st)
        x.deposit()
        x.step(4)
    same(b, c)
    for x in (a, b, c):
        x.close()
