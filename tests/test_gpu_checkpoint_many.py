"""Checkpoint and restart of many ensembles of one species each: the loaded run goes on bit for bit
as the saved one (the slot counts of the segments go to the device, and nothing beyond them)."""
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


@pytest.mark.parametrize("nens", [64, 65, 100, 256])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_restart_of_one_species_ensembles(pic, nens, precision):
    ens = [synth.ensemble(100 + k % 7, 10, nspecies=1, collisions=False, periodic=True, seed=k + 1) for k in range(nens)]
    w = {"name": "t", "steps": 1, "precision": precision, "ensembles": ens}
    a, b = pic.Sim(w, fused=False), pic.Sim(w, fused=False)
    a.step(2)
    b.load(a.save())
    for k in (0, 1, nens // 2, nens - 1):
        assert np.array_equal(a.grid(k)["Q"][0], b.grid(k)["Q"][0]), k
    a.step(3), b.step(3)
    for k in range(nens):
        ga, gb = a.grid(k), b.grid(k)
        for q in ("rho", "phi", "E"):
            if precision == "fp32":
                assert np.array_equal(ga[q], gb[q]), (k, q)
            else:  # the FP64 deposit's atomics have no order
                assert np.allclose(ga[q], gb[q], rtol=0, atol=1e-12 * max(1.0, np.abs(ga[q]).max())), (k, q)
    a.close(), b.close()
