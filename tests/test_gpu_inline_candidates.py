"""Collisions inside the particle pass (runs of at most 1024 tiles of slot capacity) against the
kernel of their own that larger runs use: the same run with a larger capacity takes the other
path, and particles, fields, counts and bounds have to be the same to the last bit.  Collision
rates up to every particle a candidate fill the tile's LDS records and spill beyond them."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("ppt", [4, 8])
@pytest.mark.parametrize("rate", [1.0, 30.0, 3000.0])
@pytest.mark.parametrize("cx_relative,nspecies", [(False, 2), (True, 2), (False, 1)])
def test_inline_candidates_match_their_kernel(pic, fused, ppt, rate, cx_relative, nspecies):
    e = synth.ensemble(700, 40, collisions=True, nspecies=nspecies, seed=9, sort_every=4, extra=300_000,
                       cx_relative=cx_relative)
    e["ngs_el"], e["ngs_iz"], e["ngs_cx"] = 0.05 * rate, 0.01 * rate, 2.0 * rate
    big = {**e, "species": [{**sp, "capacity": sp["capacity"] + 16384 * 256 * ppt} for sp in e["species"]]}
    runs = [pic.Sim({"name": "t", "steps": 1, "precision": "fp32", "ensembles": [x]}, fused=fused, ppt=ppt)
            for x in (e, big)]
    for steps in (4, 7):  # through a replayed sort cycle and past it
        for r in runs:
            r.step(steps)
        da, db = (r.diag() for r in runs)
        for q in ("count", "coll", "created", "wall_count", "pushes", "numax", "emax"):
            assert da[q] == db[q], q
        assert da["created"][0] > 0 and sum(da["coll"]) > 0
        # the tallied energy groups particles per thread in binary32
        assert da["ke"] == pytest.approx(db["ke"], rel=8 * 2.0**-24)
        ga, gb = (r.grid() for r in runs)
        for q in ("rho", "phi", "E"):
            assert np.array_equal(ga[q], gb[q]), q
        for s in range(nspecies):
            assert np.array_equal(ga["Q"][s], gb["Q"][s])
            sa, sb = (by_id(r.particles(0, s)) for r in runs)
            for q in ("id", "x", "vx", "vy", "vz"):
                assert np.array_equal(sa[q], sb[q]), (s, q)
    # the stage verb
    for r in runs:
        r.solve(), r.push(), r.collide(), r.deposit()
    da, db = (r.diag() for r in runs)
    for q in ("count", "coll", "created", "numax"):
        assert da[q] == db[q], q
    for s in range(nspecies):
        sa, sb = (by_id(r.particles(0, s)) for r in runs)
        for q in ("id", "x", "vx", "vy", "vz"):
            assert np.array_equal(sa[q], sb[q]), (s, q)
    for r in runs:
        r.close()
