"""The adjoint window at the edges of its one-launch steps (1024 nodes per group of threads, up
to four groups; larger grids take the general path) and of its particle tiles, for checkpoint
spacings that divide the window, leave a short last segment, or make every step a segment:
objective, gradients, final state and counters against FP64 autograd of the same discrete
forward, the C oracle and the stepped run."""
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


@pytest.mark.parametrize("N,ppc", [(2, 500), (64, 33), (1023, 5), (1024, 4), (1025, 5), (2048, 3), (2049, 3), (4096, 2),
                                   (4097, 2)])
@pytest.mark.parametrize("steps,ckpt", [(1, 1), (7, 3), (6, 6), (4, 1), (5, 20)])
def test_window_matches_autograd(pic, N, ppc, steps, ckpt):
    """Few steps of a thermal state, so that hardly a particle sits within the FP32 rounding of a
    node when it is read: the gradient differs by the FP32 forward's rounding (2^-24 a step of
    field and position, against the FP64 reference) apart from particles whose cell differs."""
    import torch

    from oracle import adjoint_torch

    e = synth.c4_langmuir(ncells=N, ppc=ppc)["ensembles"][0]
    e["perturb_amp"] = 0.05
    st = synth.quiet_start_state(e)[0]
    n = len(st["x"])
    rng = np.random.default_rng(N + steps)
    vx = (0.3 * rng.standard_normal(n)).astype(np.float32).astype(np.float64)
    w = {"name": "w", "steps": steps, "precision": "fp32", "ensembles": [e]}

    def fresh():
        sim = pic.Sim(w, fused=True)
        sim.set_particles(0, 0, st["x"], vx, st["vy"], st["vz"], st["id"], st["next_id"])
        sim.deposit()
        return sim

    sim, ref = fresh(), fresh()
    W, g, gE = sim.adjoint_window(steps, ckpt)
    v0 = torch.tensor(vx, requires_grad=True)
    Ee = torch.tensor(0.0, dtype=torch.float64, requires_grad=True)
    Wt = adjoint_torch.window_energy(e, torch.tensor(st["x"]), v0, Ee, steps)
    gt, gEt = (t.numpy() for t in torch.autograd.grad(Wt, (v0, Ee)))
    assert W == pytest.approx(Wt.item(), rel=1e-4)
    scale = np.abs(gt).sum()
    assert np.mean(np.abs(g[:n] - gt) > 1e-3 * np.abs(gt).max()) <= 2e-3
    assert np.abs(g[:n] - gt).sum() <= 1e-3 * scale
    assert abs(gE - gEt) <= 1e-3 * scale * e["dt"] * steps
    # the run is left in the window's final state, as the same steps leave it
    ref.step(steps)
    a, b = sim.particles(), ref.particles()
    oa, ob = np.argsort(a["id"]), np.argsort(b["id"])
    for k in ("id", "x", "vx", "vy", "vz"):
        assert np.array_equal(a[k][oa], b[k][ob]), k
    assert np.array_equal(sim.grid()["Q"][0], ref.grid()["Q"][0])
    sim.solve(), ref.solve()
    for k in ("rho", "phi", "E"):
        assert np.array_equal(sim.grid()[k], ref.grid()[k]), k
    da, db = sim.diag(), ref.diag()
    assert da["count"] == db["count"] and da["step"] == db["step"] == steps
    assert da["pushes"] == 2 * db["pushes"]  # every step is pushed forward and recomputed
    assert da["field_energy"] == pytest.approx(W, rel=1e-12)
    # and goes on from there
    sim.step(3), ref.step(3)
    for k in ("rho", "E"):
        assert np.array_equal(sim.grid()[k], ref.grid()[k]), k
    sim.close()
    ref.close()
