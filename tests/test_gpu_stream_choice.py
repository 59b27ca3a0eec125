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


@pytest.mark.parametrize("fused", [False, True])
def test_fp64_push_on_either_side(pic, fused):
    """The FP64 push streams by itself from 1e7 slots in use, as counted by the sort and where state
    is set: one push of the same particles in a run that streams (filled to the line by a second
    ensemble) and in one that does not is the same to the last bit."""
    e = synth.ensemble(20_000, 100, collisions=True, seed=5, sort_every=3, cap_factor=1.25)
    big = synth.ensemble(20_000, 160, collisions=True, seed=6, sort_every=3, cap_factor=1.25)
    a = pic.Sim({"name": "t", "steps": 1, "precision": "fp64", "ensembles": [e]}, fused=fused)
    b = pic.Sim({"name": "t", "steps": 1, "precision": "fp64", "ensembles": [e, big]}, fused=fused)
    E = synth.random_field(e, seed=3)
    st = synth.random_state(e, [2_000_001, 1_999_999], seed=8)
    for rep in range(2):
        for x in (a, b):
            if rep:
                x.sort()  # counts the slots in use itself
            else:
                x.set_state(st)
            x.set_fields(E)
            x.push()
        for s in range(2):
            pa, pb = (x.particles(0, s) for x in (a, b))
            ia, ib = np.argsort(pa["id"]), np.argsort(pb["id"])
            for q in ("id", "x", "vx", "vy", "vz"):
                assert np.array_equal(pa[q][ia], pb[q][ib]), (rep, s, q)
    a.close(), b.close()
