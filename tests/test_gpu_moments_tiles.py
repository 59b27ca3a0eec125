"""Node moments at the edges of their tiles: slot counts around the 2048-slot tile and its
runs of four, and tile spans on either side of each size of the LDS window's node copies
(512 slots shared out as copies x nodes) and of the window itself, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
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
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("n", [1, 3, 1023, 2047, 2048, 2049, 4099])
def test_moments_tile_edges(pic, prec, periodic, n):
    """Both sides sum at most n < 2^13 terms in FP64 from the same binary32-exact inputs (dx is
    a power of two, so the oracle's x / dx is exact), so they differ by at most about
    2 n 2^-53 < 2e-12 of the largest term: of the density, of the largest speed, and for the
    temperature (a difference of two such sums) of m max|v|^2."""
    N = 1200
    e = synth.ensemble(N, 8, periodic=periodic, collisions=False, cap_factor=1.0)
    # cells per tile: spans of 2, 8, 9, 16, 17, 257, 511, 512 and 513 nodes, and the whole grid
    for width in (1, 7, 8, 15, 16, 256, 510, 511, 512, N):
        lo = N - width if periodic else 0  # the periodic window wraps to node 0
        st = synth.random_state(e, [n, n], seed=n + width, vscale=[1.0, 0.5], cell_range=(lo, lo + width))
        for s in st:  # both ends of the range are occupied, so the span is the one meant
            s["cell"][0], s["cell"][-1] = lo, lo + width - 1
            s["x"] = (s["cell"].astype(np.float64) + s["off"].astype(np.float64)) * e["dx"]
        sim = pic.Sim({"name": "t", "steps": 1, "precision": prec, "ensembles": [e]}, fused=False)
        sim.set_state(st)
        o = oracle.Oracle(e, init=False)
        o.set_state(st)
        got = sim.moments()
        for s in range(2):
            want = o.moments(s)
            vmax = max(float(np.abs(st[s][k]).max()) for k in ("vx", "vy", "vz"))
            scale = {"n": want["n"].max(), "ux": vmax, "uy": vmax, "uz": vmax,
                     "T": 3.0 * e["species"][s]["m"] * vmax**2}
            for k, sc in scale.items():
                assert np.abs(got[s][k] - want[k]).max() <= 2e-12 * sc, (width, s, k)
        sim.close()
