"""The one-launch step of small periodic collisionless runs (taken in replayed windows, whole turns
of three steps) against the two launches of single steps: fields, particles and tallies have
to be the same to the last bit."""
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


def same(a, b, nens, nsp):
    for k in range(nens):
        ga, gb, da, db = a.grid(k), b.grid(k), a.diag(k), b.diag(k)
        for q in ("rho", "phi", "E"):
            assert np.array_equal(ga[q], gb[q]), (k, q)
        for q in ("count", "pushes", "step", "emax", "field_energy"):
            assert da[q] == db[q], (k, q)
        for s in range(nsp):
            assert np.array_equal(ga["Q"][s], gb["Q"][s]), (k, s)
            sa, sb = by_id(a.particles(k, s)), by_id(b.particles(k, s))
            for q in ("id", "x", "vx", "vy", "vz"):
                assert np.array_equal(sa[q], sb[q]), (k, s, q)


# one, two and four groups of 1024 nodes and their edges
SIZES = [[2], [255], [1024], [1025], [2048], [2049], [4096], [3, 1024, 700], [4095, 5, 2048, 64]]


@pytest.mark.parametrize("cells", SIZES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("nsp", [1, 2])
@pytest.mark.parametrize("K", [4, 5, 20])
def test_window_is_single_steps(pic, cells, nsp, K):
    """Windows with none (K = 4), one and six turns; the calls in between leave a charge, a field
    and a step phase of their own."""
    ens = [synth.ensemble(N, 9 if N > 64 else 500, periodic=True, nspecies=nsp, collisions=False, sort_every=K,
                          seed=3 + k, B=[0.3, 0.4, 0.5] if nsp == 2 else None, E_ext=0.05 * (nsp - 1),
                          smooth=N % 3, extra=37) for k, N in enumerate(cells)]
    work = {"name": "t", "steps": 1, "precision": "fp32", "ensembles": ens}
    a, b = pic.Sim(work, fused=True), pic.Sim(work, fused=True)
    for n in (2 * K + 3, K, 3 * K - 1):
        a.step(n)
        for _ in range(n):
            b.step(1)
        same(a, b, len(ens), nsp)
        for x in (a, b):
            x.deposit()
            x.solve()
    assert a.graph_launches() > 0 and b.graph_launches() == 0
    a.close(), b.close()


@pytest.mark.parametrize("extra", [0, 1])
def test_both_sides_of_the_slot_line(pic, extra):
    e = synth.ensemble(1024, 1000, periodic=True, nspecies=1, collisions=False, sort_every=20, seed=5)
    e["species"][0]["capacity"] = (1 << 20) + extra
    work = {"name": "t", "steps": 1, "precision": "fp32", "ensembles": [e]}
    a, b = pic.Sim(work, fused=True), pic.Sim(work, fused=True)
    a.step(40)
    for _ in range(40):
        b.step(1)
    same(a, b, 1, 1)
    a.close(), b.close()
