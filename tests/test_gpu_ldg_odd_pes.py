"""Viscous Burgers (local DG) on odd PE sizes with two elements per lane, whose
faces lie left of either element of a lane: bitwise one element per lane and one
step per launch, and the oracle's run.  Odd meshes, whose lanes straddle the
periodic wrap, meshes within the halo, PEs of three, and a batch of odd and even
PEs."""
import numpy as np
import pytest


from paper_2404_03399_amd import workloads as W
from oracle import stats, stepper
from parity_bars import derived_bars

pytestmark = pytest.mark.gpu


def _w(p, rk, scheme, q, ne, pe):
    dx = W.TWO_PI / ne
    return W.Workload(name=f"ldg_odd_{p}_{rk}_{ne}_{pe}", equation="viscous_burgers", scheme=scheme, flux="llf", rk=rk,
                      degree=p, n_elem=ne, pe_size=pe, probs=W.DELAYS_C2, seed=5, per_stage=False, at_levels=q,
                      viscosity=0.1, dt=min(0.0005 * dx, 0.0004 * dx * dx / 0.1), ic=W.PAPER_MULTISINE)


def _run(ws, u0s, n, **kw):
    from paper_2404_03399_amd.solver import Solver
    s = Solver(ws, kernel="fused", **kw)
    u = s.pack(u0s)
    s.run(u, n, graph=kw.get("lane_elems") == 2)
    out = s.unpack(u)
    s.close()
    return out


@pytest.mark.parametrize("p,rk,scheme,q,ne,pe", [
    (2, "heun", "adg_at", 2, 375, 25), (2, "ssprk3", "adg_at", 2, 405, 15), (3, "rk4", "adg_at", 2, 129, 3),
    (1, "heun", "adg_at", 3, 9, 3), (4, "lsrk4", "adg", 0, 210, 35), (2, "heun", "dg", 0, 375, 25)])
def test_odd_pes(p, rk, scheme, q, ne, pe):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = _w(p, rk, scheme, q, ne, pe)
    print(f"[gpu-case] local DG, odd PEs {w.name}", flush=True)
    u0 = stepper.initial_state(w)
    n = 21
    out = {(R, K): _run(w, u0, n, lane_elems=R, fused_steps=K)[0] for R in (1, 2, 0) for K in (1, 2, 0)}
    for key, v in out.items():
        assert np.array_equal(v, out[1, 1]), key
    ref = stepper.Stepper(w).run(u0, n)
    assert stats.rel_l2(out[2, 0], ref) <= derived_bars(w, u0, n, ref)[0]


def test_batch_of_odd_and_even_pes():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ws = [_w(2, "heun", "adg_at", 2, 375, 25), _w(2, "heun", "adg_at", 2, 512, 64), _w(3, "heun", "adg_at", 2, 99, 33),
          _w(2, "heun", "adg_at", 2, 64, 2)]
    print("[gpu-case] local DG, batch of odd and even PEs", flush=True)
    u0s = [stepper.initial_state(w) for w in ws]
    alone = [_run(w, u0, 19, lane_elems=1, fused_steps=1)[0] for w, u0 in zip(ws, u0s)]
    for kw in ({}, dict(lane_elems=2)):
        for w, a, b in zip(ws, alone, _run(ws, u0s, 19, **kw)):
            assert np.array_equal(a, b), (w.name, kw)


