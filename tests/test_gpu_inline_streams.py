"""Collisions inside the particle pass at the edge of that path (16384 tiles of slot capacity, with four
and with eight particles a thread) and over particles that the pass streams non-temporally: the
same run with one aligned slot range more of capacity collides its candidates in their own launch,
and with the non-temporal option asked for, and all of them agree to the last bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

TILES, ALIGN = 16384, 4096


@pytest.fixture(scope="module")
def pic():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_28534_amd as P

    P.load_library()
    return P


@pytest.mark.parametrize("ppt,cx_relative", [(4, False), (4, True), (8, False)])
@pytest.mark.parametrize("use", [9_000_000, 15_600_000, 25_000_000])
def test_edge_and_streams(pic, ppt, cx_relative, use):
    slots = TILES * 256 * ppt
    if use > slots:
        pytest.skip("more than the capacity at the edge")
    ppc = use // 2 // 40_000
    e = synth.ensemble(40_000, ppc, collisions=True, seed=6, sort_every=3, cx_relative=cx_relative)
    caps = [slots // 2, slots // 2 + ALIGN, slots // 2]
    ens = [{**e, "species": [{**sp, "capacity": c} for sp in e["species"]]} for c in caps]
    runs = [pic.Sim({"name": "t", "steps": 1, "precision": "fp32", "ensembles": [x]}, ppt=ppt, nontemporal=nt)
            for x, nt in zip(ens, (0, 0, 1))]
    for steps in (2, 5):  # a sorting pass and more
        for r in runs:
            r.step(steps)
        d = [r.diag() for r in runs]
        g = [r.grid() for r in runs]
        for k in (1, 2):
            for q in ("count", "coll", "created", "wall_count", "pushes", "numax", "emax"):
                assert d[0][q] == d[k][q], (k, q)
            for q in ("rho", "phi", "E"):
                assert np.array_equal(g[0][q], g[k][q]), (k, q)
            for s in range(2):
                assert np.array_equal(g[0]["Q"][s], g[k]["Q"][s]), (k, s)
    assert sum(d[0]["coll"]) > 0
    for r in runs:
        r.close()
