"""Read-back of the grid and the scalars: the node arrays in one piece, one by one and some only,
for one and two species; the fused step's tallied scalars of each of several ensembles against
a recount of the same state."""
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


def work_of(ens, precision="fp32"):
    return {"name": "t", "steps": 1, "precision": precision, "ensembles": ens}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nspecies", [1, 2])
@pytest.mark.parametrize("N", [2, 255, 300_001])
def test_grid_arrays_in_any_host_layout(pic, prec, nspecies, N):
    ens = [synth.ensemble(n, 3, collisions=False, nspecies=nspecies, seed=4, extra=64) for n in (7, N)]
    sim = pic.Sim(work_of(ens, prec), fused=False)
    sim.step(2)
    g = sim.grid(1)
    nn = N + 1
    assert sum(q.sum() for q in g["Q"]) == pytest.approx(sum(sim.diag(1)["count"]), rel=1e-12)
    rows = g["Q"] + ([np.zeros(nn)] if nspecies == 1 else []) + [g["rho"], g["phi"], g["E"]]
    gap = np.full((5, nn + 3), np.nan)  # arrays apart from one another, padding untouched
    for want in ([0, 1, 2, 3, 4], [0, 4], [2, 3], [1]):
        gap[:] = np.nan
        ptr = [C.c_void_p(gap[k].ctypes.data) if k in want else None for k in range(5)]
        assert sim.L.pic_get_grid(sim.h, 1, *ptr, sim._s()) == 0
        for k in range(5):
            assert np.array_equal(gap[k, :nn], rows[k]) if k in want else np.isnan(gap[k]).all(), k
        assert np.isnan(gap[:, nn:]).all()
    sim.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_scalars_of_every_ensemble(pic, prec):
    """After a fused step the scalars come from its tallies; a sort leaves the particles as they
    are and makes the next read a recount.  Counts are exact; the tallied energies sum |v|^2
    per thread in binary32 (relative 8 x 2^-24)."""
    ens = [synth.ensemble(40 + 300 * k, 30, collisions=True, seed=k + 1, sort_every=5, extra=4000) for k in range(11)]
    for e in ens:
        e["ngs_el"], e["ngs_iz"] = 0.1, 0.3
    sim = pic.Sim(work_of(ens, prec), fused=True)
    sim.step(7)
    a = [sim.diag(k) for k in range(len(ens))]
    sim.sort()
    for k, d in enumerate(a):
        r = sim.diag(k)
        for q in ("count", "wall_count", "wall_charge", "wall_ke", "coll", "created", "pushes", "step", "numax", "emax",
                  "charge"):
            assert d[q] == r[q], (k, q)
        assert d["ke"] == pytest.approx(r["ke"], rel=8 * 2.0**-24)
        assert d["field_energy"] == pytest.approx(r["field_energy"], rel=1e-12)
        p = [sim.particles(k, s) for s in range(2)]
        assert d["count"] == [len(x["id"]) for x in p]
        for s in range(2):
            sp = ens[k]["species"][s]
            v2 = sum(np.square(p[s][c]).sum() for c in ("vx", "vy", "vz"))
            assert r["ke"][s] == pytest.approx(0.5 * sp["m"] * sp["w"] * v2, rel=1e-12)
    sim.close()


def test_contexts_share_the_read_back_block(pic):
    """More contexts than the shared page-locked block has pages (64), closed out of order, then
    one after the block was given back: each reads its own scalars."""
    def one(k):
        e = synth.ensemble(5 + k, 3, collisions=False, nspecies=1, seed=1 + k, extra=64)
        return pic.Sim({"name": "t", "steps": 1, "precision": "fp32", "ensembles": [e]}, fused=True)

    sims = [one(k) for k in range(67)]
    for k, s in enumerate(sims):
        assert s.diag()["count"][0] == 3 * (5 + k)
    for s in sims[::2] + sims[1::2]:
        s.close()
    s = one(70)
    s.step(1)
    assert s.diag()["step"] == 1 and s.diag()["count"][0] <= 3 * 75
    s.close()
