"""The adjoint window at its limits: particles whose motion is no valid state, which the push drops
(their slots hold no cell, so the reverse sweep has to leave them out)."""
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


# the one-launch steps of a small grid and the general sweep; the first and the last slot of a
# thread's run, and a whole run
@pytest.mark.parametrize("N", [300, 5000])
@pytest.mark.parametrize("fast", [[0], [3, 4, 5, 6, 7, 8], [-1]])
def test_dropped_particles_are_reported(pic, N, fast):
    e = synth.c4_langmuir(ncells=N, ppc=3)["ensembles"][0]
    st = synth.quiet_start_state(e)[0]
    v = np.array(st["vx"])
    v[fast] = 1e30  # more than a period in one step
    sim = pic.Sim({"name": "w", "steps": 6, "precision": "fp32", "ensembles": [e]}, fused=True)
    sim.set_particles(0, 0, st["x"], v, st["vy"], st["vz"], st["id"], st["next_id"])
    with pytest.raises(pic.PicError) as ei:
        sim.adjoint_window(6, 4)
    assert ei.value.code == pic.PIC_ENONFINITE
    sim.close()
