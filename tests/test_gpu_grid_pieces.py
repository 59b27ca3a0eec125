"""Node arrays read back in pieces: the sizes at which fewer arrays are joined in one copy (1 MiB holds
five arrays of 26214 nodes, two of 65536) and beyond which each is copied from where it lies.  A field
set from the host comes back as it was, and arrays read together are those read one by one."""
import ctypes as C

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


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nspecies", [1, 2])
@pytest.mark.parametrize("nn", [26214, 26215, 43690, 43691, 65536, 65537])
def test_pieces(pic, prec, nspecies, nn):
    ens = [synth.ensemble(n, 2, collisions=False, nspecies=nspecies, seed=5, periodic=True) for n in (11, nn)]
    sim = pic.Sim({"name": "t", "steps": 1, "precision": prec, "ensembles": ens}, fused=False)
    sim.step(1)
    E = np.random.default_rng(nn).standard_normal(nn)
    sim.set_fields(E, 1)
    g = sim.grid(1)
    assert np.array_equal(g["E"], E)
    rows = g["Q"] + ([np.zeros(nn)] if nspecies == 1 else []) + [g["rho"], g["phi"], g["E"]]
    assert all(abs(q.sum() - 2 * nn) <= 1e-9 * nn for q in g["Q"])  # 2^-24 shares, FP64 sums
    assert np.any(rows[2] != 0.0) and np.any(rows[3] != 0.0)
    one = np.full(nn + 2, np.nan)
    for k in range(5):
        one[:] = np.nan
        ptr = [C.c_void_p(one.ctypes.data) if i == k else None for i in range(5)]
        assert sim.L.pic_get_grid(sim.h, 1, *ptr, sim._s()) == 0
        assert np.array_equal(one[:nn], rows[k]) and np.isnan(one[nn:]).all(), k
    sim.close()
