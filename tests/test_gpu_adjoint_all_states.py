"""Adjoint of a run that keeps every state (checkpoint interval 1): its reverse
launches take several steps and read the states from the checkpoints.  Bitwise
the gradients of runs that recompute their segments."""
import numpy as np
import pytest

from paper_2404_03399_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 13, 27])
@pytest.mark.parametrize("kw", [
    {}, dict(speed=-0.75, degree=4, rk="lsrk4"), dict(flux="central", pe=1, degree=1, rk="heun"),
    dict(equation="burgers", flux="llf", degree=2, rk="ssprk3"), dict(equation="burgers", flux="llf", pe=25, rk="rk4")],
    ids=lambda k: "-".join(f"{a}{b}" for a, b in k.items()) or "upwind")
def test_every_state_kept(kw, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_03399_amd.solver import Solver
    kw = dict(kw)
    pe = kw.pop("pe", 32)
    ne = 1600
    w = W.Workload(name="kept", scheme="adg_at", n_elem=ne, pe_size=pe, probs=W.DELAYS_C2, seed=8,
                   dt=0.0005 * W.TWO_PI / ne, ic=W.MultiSine((1, 3), (1.0, 0.5), (0.3, 1.9), 0.5),
                   **{**dict(rk="rk4", degree=3), **kw})
    print(f"[gpu-case] adjoint, every state kept: {w.equation} {w.flux} PE={pe} {w.rk} n={n}", flush=True)
    out = []
    for ck in (1, 5, 64):
        s = Solver(w, n_steps_record=n + 3, ckpt_every=ck)
        u = s.initial_state()
        s.run(u, n, record=True)
        g, gs = s.adjoint(u)
        g2, _ = s.adjoint(u)  # the recording stays valid
        assert torch.equal(s.view(g), s.view(g2))
        out.append((s.unpack(u)[0], s.unpack(g)[0], gs))
        s.close()
    for u, g, gs in out[1:]:
        assert np.array_equal(u, out[0][0]) and np.array_equal(g, out[0][1]) and gs == out[0][2]
