"""Calls of few steps: every number of steps has a work list of its own and a call
whose launches would end in the other buffer halves its first one.  Bitwise the
run of one step per launch, whatever the calls."""
import numpy as np
import pytest

from paper_2404_03399_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(ne=(1 << 18) + 256), dict(ne=1 << 18, speed=-1.0, rk="heun", degree=1),
    dict(ne=(1 << 18) + 6, pe=25, flux="central", degree=1, rk="ssprk3"),
    dict(ne=1 << 18, equation="burgers", flux="llf", degree=2, rk="lsrk3"),
    dict(ne=1 << 18, equation="viscous_burgers", flux="llf", degree=1, rk="heun", viscosity=0.1, at_levels=2),
    dict(ne=1024, degree=2), dict(ne=320, pe=64, degree=2)], ids=lambda k: "-".join(f"{a}{b}" for a, b in k.items()))
@pytest.mark.parametrize("opt", [{}, dict(lane_elems=4), dict(record=True)], ids=["default", "R4", "record"])
def test_any_calls_give_the_same_states(kw, opt):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2404_03399_amd.solver import Solver
    kw, opt = dict(kw), dict(opt)
    ne, pe = kw.pop("ne"), kw.pop("pe", 256 if kw.get("ne", 1 << 18) > 2048 else 64)
    pe = pe if ne % pe == 0 else 2
    if opt.get("lane_elems", 1) > pe or (opt.get("record") and kw.get("equation") == "viscous_burgers"):
        pytest.skip("not a valid option")
    w = W.Workload(name="short", scheme="adg_at", n_elem=ne, pe_size=pe, probs=W.DELAYS_C2, seed=4,
                   dt=0.001 * (2e-6 if kw.get("viscosity") else 1.0) * W.TWO_PI / ne,
                   ic=W.MultiSine((1, 3), (1.0, 0.5), (0.3, 1.9)), **{**dict(rk="rk4", degree=3), **kw})
    print(f"[gpu-case] short calls {w.equation} N={ne} PE={pe} {w.rk} {opt}", flush=True)
    rec = opt.pop("record", False)
    calls = [4, 7, 1, 8, 2, 14, 3, 16, 24, 5, 6]
    n = sum(calls)
    ref = Solver(w, fused_steps=1, lane_elems=1, n_steps_record=n if rec else 0)
    s = Solver(w, n_steps_record=n if rec else 0, **opt)
    u, v = s.initial_state(), ref.initial_state()
    assert torch.equal(u, v)
    for i, c in enumerate(calls):
        s.run(u, c, graph=i % 3 == 2)
        ref.run(v, c, graph=False)
        assert torch.equal(s.view(u), ref.view(v)), (c, calls[:i])  # a padded plane's end is nobody's
    assert bool(torch.isfinite(s.view(u)).all())
    if rec:
        for ck in (4, 7, 12):  # segments of so many steps each, the states kept of any
            t = Solver(w, n_steps_record=n, ckpt_every=ck)
            x = t.initial_state()
            t.run(x, n, record=True)
            assert torch.equal(t.view(x), s.view(u)), ck
            t.close()
    s.close()
    ref.close()
