"""The sort's scan on either side of the number of tiles (2048 of 4096 cells) up to which each block
adds up the tiles before its own: after a sort every particle is there once and the slots are in
the order of the cells."""
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


@pytest.mark.parametrize("N", [2048 * 4096 - 1, 2048 * 4096, 2048 * 4096 + 1, 2049 * 4096 + 1])
def test_sort_of_many_cells(pic, N):
    e = synth.ensemble(N, 1, nspecies=1, collisions=False, periodic=True, seed=2)
    sim = pic.Sim({"name": "t", "steps": 1, "precision": "fp32", "ensembles": [e]}, fused=False)
    sim.push()  # (the field is zero: the particles move by their own velocities)
    before = sim.slots(0, 0, 0, N)
    assert np.any(np.diff(np.floor(before["x"] / e["dx"])) < 0)
    sim.sort()
    after = sim.slots(0, 0, 0, N)
    assert np.all(np.diff(np.floor(after["x"] / e["dx"])) >= 0)
    order = np.argsort(after["id"], kind="stable")
    for k in ("id", "x", "vx", "vy", "vz"):
        assert np.array_equal(after[k][order], before[k]), k  # (the load numbers its slots by id)
    sim.close()
