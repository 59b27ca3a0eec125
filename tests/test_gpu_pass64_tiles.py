"""The FP64 pass at the edges of its tiles (thread blocks of 64 and 256 threads, four slots a
thread in two runs of two) and of its LDS deposit window (1024 nodes, shared out as copies of
the tile's nodes): deposit, push, collide and sort from injected states against the FP64
oracle, with dead slots in odd places from the push's absorptions."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import cell_counts, compare_particles, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2606_28534_amd as P

    P.load_library()
    return P


@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1023, 1024, 1025, 2051])
def test_fp64_stages_at_tile_edges(pic, block, periodic, n):
    """FP64 on both sides: a node sums at most 2 n < 2^13 shares (rel 2^-40 of the largest), a
    push differs by a few roundings, collision decisions take the same FP64 comparisons."""
    N = 1500
    e = synth.ensemble(N, 1, periodic=periodic, collisions=True, seed=3 + n, cap_factor=1.0, extra=4 * n + 64)
    e["ngs_el"], e["ngs_iz"], e["ngs_cx"] = 0.3, 0.5, 300.0
    # spans of 2, 17, 1023, 1024 and 1025 nodes, and the whole grid
    for width in (1, 16, 1022, 1023, 1024, N):
        lo = N - width if periodic else 0  # the periodic window wraps to node 0
        st = synth.random_state(e, [n, n], seed=n + width, vscale=[2.0, 0.5], cell_range=(lo, lo + width))
        for s in st:  # both ends of the range are occupied, so the span is the one meant
            s["cell"][0], s["cell"][-1] = lo, lo + width - 1
            s["x"] = (s["cell"].astype(np.float64) + s["off"].astype(np.float64)) * e["dx"]
        sim = pic.Sim({"name": "t", "steps": 1, "precision": "fp64", "ensembles": [e]}, fused=False, block=block)
        sim.set_state(st)
        o = oracle.Oracle(e, init=False)
        o.set_state(st)
        for x in (sim, o):
            x.deposit()
            x.solve()
            x.push()
        o.walls()
        sim.collide()
        o.collide()
        sim.deposit()
        o.deposit()
        g, r = sim.grid(), o.grid()
        gd, od = sim.diag(), o.diag()
        for k in ("count", "wall_count", "coll", "created", "pushes"):
            assert gd[k] == od[k], (width, k)
        for s in range(2):
            assert rel(g["Q"][s], r["Q"][s]) <= 1e-11, (width, s)
            assert gd["ke"][s] == pytest.approx(od["ke"][s], rel=1e-11)
            compare_particles(sim.particles(0, s), o.particles(s), e["dx"], True, vtol=1e-10)
        sim.sort()
        for s in range(2):
            c = np.floor(sim.particles(0, s)["x"] / e["dx"]).astype(np.int64)
            assert np.all(np.diff(c) >= 0), (width, s)
            assert np.array_equal(np.bincount(c, minlength=N), cell_counts(o.particles(s)["x"], e["dx"], N))
            compare_particles(sim.particles(0, s), o.particles(s), e["dx"], True, vtol=1e-10)
        sim.close()
