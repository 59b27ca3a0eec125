"""The adjoint window at its limits: particles whose motion is no valid state, which the push drops
(their slots hold no cell, so the reverse sweep has to leave them out), and scratch that holds the
general sweep but not the one-launch steps of a small grid, or that starts at any byte."""
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


def window(pic, sim, steps, ckpt, scratch, offset, size):
    """pic_adjoint_window on bytes [offset, offset + size) of a device tensor."""
    n = int(sim.work["ensembles"][0]["species"][0]["capacity"])
    g, W, gE = np.zeros(n), C.c_double(0), C.c_double(0)
    rc = sim.L.pic_adjoint_window(sim.h, steps, ckpt, C.c_void_p(scratch.data_ptr() + offset), size, C.byref(W),
                                  C.c_void_p(g.ctypes.data), n, C.byref(gE), sim._s())
    return rc, W.value, g, gE.value


def query(sim, steps, ckpt):
    nb = C.c_size_t(0)
    assert sim.L.pic_adjoint_query(sim.h, steps, ckpt, C.byref(nb)) == 0
    return nb.value


def general_bytes(slots, nodes, steps, ckpt):
    """The general sweep's scratch: a state per checkpoint, the recorded positions and fields of a
    segment, the adjoint arrays and the final state."""
    segs = -(-steps // ckpt)
    parts = [4 * segs * slots] * 3 + [4 * ckpt * slots] * 2 + [8 * ckpt * nodes] + [8 * slots] * 2 + [64]
    parts += [8 * nodes] * 3 + [20 * slots]
    return sum((p + 255) // 256 * 256 for p in parts)


# The routes sum the same terms in another order: each step's field adjoint has up to 4096 terms a
# node, 4096 2^-53 of its size, and the steps add up.
def close(a, b, steps):
    scale = np.abs(a[1]).max()
    assert a[0] == pytest.approx(b[0], rel=1e-12)
    assert np.abs(a[1] - b[1]).max() <= 4096 * 2.0**-53 * steps**2 * scale
    assert abs(a[2] - b[2]) <= 4096 * 2.0**-53 * steps**2 * scale * len(a[1])


@pytest.mark.parametrize("N,ppc,steps,ckpt", [(4096, 1, 12, 1), (1024, 4, 9, 2), (250, 40, 8, 4)])
def test_scratch_of_any_size_and_alignment(pic, N, ppc, steps, ckpt):
    import torch

    e = synth.c4_langmuir(ncells=N, ppc=ppc)["ensembles"][0]
    sim = pic.Sim({"name": "w", "steps": steps, "precision": "fp32", "ensembles": [e]}, fused=True)
    start = sim.save()
    want = sim.adjoint_window(steps, ckpt)
    end = sim.particles()
    full = query(sim, steps, ckpt)
    general = general_bytes(-(-N * ppc // 4096) * 4096, N, steps, ckpt)
    scratch = torch.empty(max(full, general) + 256, dtype=torch.uint8, device="cuda")
    for offset, size, fits in [(0, full, True), (4, full, True), (8, full, True), (0, general, True), (8, general, True),
                               (0, min(full - 16, general) - 1, False)]:
        sim.load(start)
        rc, *got = window(pic, sim, steps, ckpt, scratch, offset, size)
        assert rc == (pic.PIC_OK if fits else pic.PIC_EINVAL), (offset, size)
        if not fits:
            continue
        close(got, want, steps)
        now = sim.particles()
        a, b = np.argsort(now["id"]), np.argsort(end["id"])
        for k in ("id", "x", "vx", "vy", "vz"):
            assert np.array_equal(now[k][a], end[k][b]), (offset, size, k)
    sim.close()


def test_noalloc_takes_what_the_general_sweep_fits(pic):
    """2500 checkpoints of 4096 cells with a particle each: 117 MiB for the general sweep, 195 MiB for
    the one-launch steps; the static array has 160."""
    e = synth.c4_langmuir(ncells=4096, ppc=1)["ensembles"][0]
    w = {"name": "w", "steps": 2500, "precision": "fp32", "ensembles": [e]}
    assert general_bytes(4096, 4096, 2500, 1) < 160 << 20 < query(pic.Sim(w, fused=True), 2500, 1)
    a, b = pic.Sim(w, fused=True), pic.Sim(w, fused=True)
    ra, rb = a.adjoint_window(2500, 1), b.adjoint_window_noalloc(2500, 1)
    close(ra, rb, 2500)
    pa, pb = a.particles(), b.particles()
    oa, ob = np.argsort(pa["id"]), np.argsort(pb["id"])
    for k in ("id", "x", "vx"):
        assert np.array_equal(pa[k][oa], pb[k][ob]), k
    a.close(), b.close()
