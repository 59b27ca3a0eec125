"""The separate stages, stepped: in a call of several steps a step's births are placed beside the
next step's solve, in calls of one step at its end.  Both have to give the same run: FP32 to
the last bit, FP64 within its reordered sums (1e-9 over these steps)."""
import numpy as np
import pytest

import synth
from parity_util import by_id, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_28534_amd as P

    P.load_library()
    return P


# the one-launch solve, the chunked solve, and more ensembles than the former takes; inline
# candidates, and with the large capacity (past 16384 tiles) candidates in a launch of their own
CASES = [([2], {}), ([256], {}), ([5000], {}), ([4097], {"floating": True, "recycle": True}),
         ([300], {"floating": True, "recycle": True, "src_pairs": 40}), ([700], {"periodic": True}),
         ([64 + 50 * k for k in range(9)], {}), ([3000], {"cap": 8_500_000})]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("K", [1, 5, 20])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_one_call_is_many(pic, case, K, prec):
    cells, opt = CASES[case]
    opt = dict(opt)
    if prec == "fp64" and opt.get("recycle"):
        pytest.skip("recycling is an FP32 form")
    cap = opt.pop("cap", 0)
    ens = []
    for k, N in enumerate(cells):
        e = synth.ensemble(N, 12 if N > 100 else 60, collisions=True, sort_every=K, seed=2 + k, extra=4000,
                           neutral_capacity=65536 if opt.get("recycle") else 0, **opt)
        e["ngs_el"], e["ngs_iz"] = 0.1, 0.2
        if cap:
            for sp in e["species"]:
                sp["capacity"] = cap
        ens.append(e)
    work = {"name": "t", "steps": 1, "precision": prec, "ensembles": ens}
    a, b = pic.Sim(work, fused=False), pic.Sim(work, fused=False)
    for n in (13, 2, 1, 7):
        a.step(n)
        for _ in range(n):
            b.step(1)
    born = 0
    for k in range(len(ens)):
        da, db = a.diag(k), b.diag(k)
        for q in ("count", "coll", "created", "wall_count", "pushes", "step", "recycled", "sourced", "neutral_count"):
            assert da[q] == db[q], (k, q)
        born += sum(da["created"])
        ga, gb = a.grid(k), b.grid(k)
        for q in ("rho", "phi", "E"):
            if prec == "fp32":
                assert np.array_equal(ga[q], gb[q]), (k, q)
            else:
                assert rel(ga[q], gb[q]) <= 1e-9, (k, q)
        for s in range(2):
            sa, sb = by_id(a.particles(k, s)), by_id(b.particles(k, s))
            assert np.array_equal(sa["id"], sb["id"]), (k, s)
            for q in ("x", "vx", "vy", "vz"):
                if prec == "fp32":
                    assert np.array_equal(sa[q], sb[q]), (k, s, q)
                else:
                    assert rel(sa[q], sb[q]) <= 1e-9, (k, s, q)
    assert born > 0 or cells == [2]
    a.close(), b.close()
