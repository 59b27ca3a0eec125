"""The sort's one-block scan of the cell counts (up to 32768 cells in all, rounds of 16384, a
thread's run of 16): totals at the edges of a run, a round and the path, several segments whose
first cells fall inside runs, and the second sort, which needs the counts cleared by the first."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import by_id

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_28534_amd as P

    P.load_library()
    return P


# cells of each one-species ensemble
CELLS = [[2], [15], [16], [17], [16383], [16384], [16385], [32767], [32768], [32769],
         [7, 1000, 3], [16385, 5, 16377], [16384, 16384], [20011, 12757, 2]]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("cells", CELLS, ids=lambda c: "-".join(map(str, c)))
def test_sort_scan_sizes(pic, prec, cells):
    ens = [synth.ensemble(N, 4, periodic=True, nspecies=1, collisions=False, seed=1 + k, extra=600)
           for k, N in enumerate(cells)]
    sim = pic.Sim({"name": "t", "steps": 1, "precision": prec, "ensembles": ens}, fused=False)
    states = [synth.random_state(e, [500 + 3 * e["ncells"]], seed=5 + k) for k, e in enumerate(ens)]
    for k, st in enumerate(states):
        sim.set_state(st, k)
    for _ in range(2):
        sim.sort()
        for k, (e, st) in enumerate(zip(ens, states)):
            o = oracle.Oracle(e, init=False)
            o.set_state(st)
            o.sort()
            g, r = sim.particles(k, 0), o.particles(0)
            gc, rc = (np.floor(p["x"] / e["dx"]).astype(np.int64) for p in (g, r))
            assert np.all(np.diff(gc) >= 0)
            assert np.array_equal(gc, rc)
            G, R = by_id(g), by_id(r)
            assert np.array_equal(G["id"], R["id"])
            assert np.array_equal(np.floor(G["x"] / e["dx"]), np.floor(R["x"] / e["dx"]))
    sim.close()
