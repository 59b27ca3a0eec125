"""The one-launch solve of small runs against the FP64 oracle and against the chunked solve: a
ninth ensemble (a copy of the first) takes a run off the small path, whose fields, particles
and counts have to be the same to the last bit."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import TOL_FIELD, by_id, rel

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


# one chunk of 1024 nodes, its edges, the edges of two and of four chunks (the most the small
# path takes), and the first size beyond it
SIZES = [2, 256, 1023, 1024, 2047, 2048, 3071, 4095, 4096]


@pytest.mark.parametrize("N", SIZES)
@pytest.mark.parametrize("boundary", ["absorbing", "floating", "periodic"])
@pytest.mark.parametrize("fused", [False, True])
def test_small_solve_is_the_chunked_solve(pic, N, boundary, fused):
    """22 collisional steps (births placed by the solve's launch in the replayed cycle), with and
    without smoothing: bit for bit, and the field of a first step against the oracle."""
    ens = []
    for k in range(9):
        e = synth.ensemble(N if k in (0, 8) else 5 + k, 12 if N > 100 else 60, collisions=True, seed=1 + k % 8,
                           sort_every=20, periodic=boundary == "periodic", floating=boundary == "floating",
                           smooth=2 if N % 2 else 0, extra=4000)
        e["ngs_el"], e["ngs_iz"] = 0.1, 0.2
        ens.append(e)
    one = pic.Sim(work_of(ens[:1]), fused=fused)
    o = oracle.Oracle(ens[0])
    one.step(1)
    o.step(1)
    g, r = one.grid(), o.grid()
    for k in ("rho", "phi", "E"):
        assert rel(g[k], r[k]) <= TOL_FIELD, k
    a, b = pic.Sim(work_of(ens[:8]), fused=fused), pic.Sim(work_of(ens), fused=fused)
    for x in (a, b):
        x.step(22)
    one.step(21)
    for x, k in ((a, 0), (one, 0), (b, 8)):
        ga, gb = x.grid(k), b.grid(0)
        for q in ("rho", "phi", "E"):
            assert np.array_equal(ga[q], gb[q]), (k, q)
        da, db = x.diag(k), b.diag(0)
        for q in ("count", "coll", "created", "wall_count", "pushes", "step", "numax", "emax"):
            assert da[q] == db[q], (k, q)
        assert sum(da["created"]) > 0 or N == 2
        for s in range(2):
            sa, sb = by_id(x.particles(k, s)), by_id(b.particles(0, s))
            for q in ("id", "x", "vx", "vy", "vz"):
                assert np.array_equal(sa[q], sb[q]), (k, s, q)
    for x in (one, a, b):
        x.close()


@pytest.mark.parametrize("N", [256, 2048, 4096])
def test_small_solve_fp64(pic, N):
    """The FP64 form (its deposit's atomics reorder sums: 1e-9 over 22 steps) and the
    collisionless periodic run, whose step counter the solve advances."""
    e = synth.ensemble(N, 12, collisions=True, seed=3, sort_every=20, extra=4000)
    sim, o = pic.Sim(work_of([e], "fp64"), fused=False), oracle.Oracle(e)
    sim.step(22)
    o.step(22)
    g, r = sim.grid(), o.grid()
    for k in ("rho", "phi", "E"):
        assert rel(g[k], r[k]) <= 1e-9, k
    assert sim.diag()["coll"] == o.diag()["coll"] and sim.diag()["step"] == 22
    sim.close()
    e = synth.ensemble(N, 12, periodic=True, nspecies=1, collisions=False, seed=3, cap_factor=1.0)
    sim, o = pic.Sim(work_of([e], "fp64"), fused=True), oracle.Oracle(e)
    sim.step(22)
    o.step(22)
    g, r = sim.grid(), o.grid()
    for k in ("rho", "phi", "E"):
        assert rel(g[k], r[k]) <= 1e-9, k
    assert sim.diag()["step"] == 22
    sim.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n_ens", [1, 3])
def test_births_on_either_side_of_the_ranking_line(pic, precision, n_ens):
    """Up to 256 births of a step are ranked by comparison, more through the group counts and the
    bitmap: runs whose steps make from none to several thousand, against the chunked path."""
    per_step = []
    for rate in (0.0, 0.002, 0.02, 0.06, 0.1, 0.3, 3.0):
        ens = []
        for k in range(9):
            e = synth.ensemble(900 + 50 * k if k < n_ens else 3, 60, collisions=True, seed=1 + k, sort_every=5,
                               extra=200_000)
            e["ngs_iz"] = rate
            ens.append(e)
        a, b = (pic.Sim(work_of(x, precision), fused=precision == "fp32") for x in (ens[:n_ens], ens))
        last = 0
        for _ in range(4):
            a.step(1), b.step(1)
            made = sum(a.diag(k)["created"][0] for k in range(n_ens))
            per_step.append(made - last)
            last = made
        for x in (a, b):
            x.step(7)
        for k in range(n_ens):
            da, db = a.diag(k), b.diag(k)
            for q in ("count", "coll", "created", "step"):
                assert da[q] == db[q], (rate, k, q)
            for s in range(2):
                sa, sb = by_id(a.particles(k, s)), by_id(b.particles(k, s))
                assert np.array_equal(sa["id"], sb["id"])
                for q in ("x", "vx", "vy", "vz"):
                    if precision == "fp32":
                        assert np.array_equal(sa[q], sb[q]), (rate, k, s, q)
                    else:  # the FP64 deposit's atomics reorder sums
                        assert np.max(np.abs(sa[q] - sb[q])) <= 1e-9 * np.max(np.abs(sb[q])), (rate, k, s, q)
        a.close(), b.close()
    per_step.sort()
    assert per_step[0] == 0 and any(0 < m <= 256 for m in per_step) and per_step[-1] > 512
