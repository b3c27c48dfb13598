"""The fused step's linear form (upwind advection with a > 0): at the edges of
its tiles and launches against the oracle, and every launch shape bitwise.

Bars as everywhere (parity_bars.py), taken from the oracle's own rounding
response where that is larger than 1e-12."""
import sys

import numpy as np
import pytest

from paper_2404_03399_amd import workloads as W
from oracle import stats, stepper
from parity_bars import derived_bars, pe_max_rel

pytestmark = pytest.mark.gpu

FORCED_LATE = ("0", "0", "0", "0", "0", "0", "0", "1")  # every face 7 levels late: L at its maximum


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _w(ne, pe, p=3, rk="rk4", probs=W.DELAYS_C2, scheme="adg_at", **kw):
    sig = {1: 0.05, 2: 0.01, 3: 0.005, 4: 0.001}[p]
    return W.Workload(name=f"lin_{ne}_{pe}_p{p}_{rk}_{scheme}", rk=rk, scheme=scheme, degree=p, n_elem=ne, pe_size=pe,
                      probs=probs, seed=31 + ne, dt=sig * W.TWO_PI / ne, ic=W.MultiSine((1, 3), (1.0, 0.5), (0.3, 1.9)),
                      **kw)


def _run(ws, u0s, n, **kw):
    from paper_2404_03399_amd.solver import Solver
    s = Solver(ws, **kw)
    u = s.pack(u0s)
    s.run(u, n, graph=False)
    s.run(u, 16, graph=True)
    out = s.unpack(u)
    s.close()
    return out


# owned elements of a tile (S = 4, PE faces): R = 4: 220, 236, 244 or 248 at
# 8, 4, 2 or 1 steps per launch; R = 2: 94, 110, 118, 122; R = 1: 31, 47, 55, 59
CASES = [
    (1024, 16, {}),                                    # the smallest mesh of the form, 16 faces per wave
    (1100, 1100, {}),                                  # five whole tiles, one PE: no face
    (1120, 20, {}),                                    # a ragged last tile
    (1199, 109, {}),                                   # odd PE size: one element per lane, no grouped loads
    (1085, 31, dict(rk="lsrk4", p=4)),                 # one element per lane, five stages
    (1100, 22, dict(p=2)),                             # two elements per lane
    (1099, 157, dict(p=1, rk="heun")),
    (1026, 2, dict(p=1)),                              # 64 faces per wave, job lanes in many passes
    (1025, 1, dict(rk="heun", p=2)),                   # every face a PE face
    (1760, 4, dict(p=4)),
    (1760, 16, dict(rk="ssprk3", per_stage=False)),
    (2640, 220, dict(rk="lsrk3", p=2, scheme="adg")),
    (1250, 250, dict(scheme="dg", rk="lsrk4")),        # synchronous
    (1152, 48, dict(probs=FORCED_LATE, at_levels=5)),  # L = 8, q = 5: the longest windows
    (1152, 48, dict(probs=FORCED_LATE, at_levels=1)),
    (1024, 64, dict(probs=("1/3", "1/3", "1/3"), caa=True, per_stage=False)),
    (70000, 35000, dict(p=2, rk="ssprk3")),            # two elements per lane by the library's choice
]


@pytest.mark.parametrize("ne,pe,kw", CASES, ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(
    f"{k}{v[k]}" if k != "probs" else f"L{len(v[k])}" for k in v) or "default")
def test_linear_form_edges(torch_cuda, ne, pe, kw):
    """Steps 15 and 16: launches of 8, 4, 2 and 1 steps, then a graph."""
    w = _w(ne, pe, **kw)
    print(f"[gpu-case] linear form {w.name} {kw}", flush=True)
    u0 = stepper.initial_state(w)
    n = 15
    ref = stepper.Stepper(w).run(u0, n + 16)
    tol, tol_pe = derived_bars(w, u0, n + 16, ref)
    outs = {(R, K): _run(w, u0, n, lane_elems=R, fused_steps=K)[0] for R in (0, 1, 2, 4) if R <= pe for K in (0, 1, 2)}
    first = outs[0, 0]
    assert stats.rel_l2(first, ref) <= tol
    assert pe_max_rel(first, ref, w) <= tol_pe
    for key, o in outs.items():
        assert np.array_equal(o, first), key
    sys.stdout.flush()


def test_linear_form_in_a_batch(torch_cuda):
    """A batch of both upwind forms (meshes below 1024 elements step stage by
    stage), degrees and signs of the speed: each problem bitwise as alone, in
    one launch per range and in one launch over all."""
    ws = [_w(1280, 64), _w(640, 8), _w(1536, 16, p=1), _w(1300, 25, p=4), _w(1280, 64, speed=-1.0), _w(1024, 1024, p=2),
          _w(640, 64, p=3)]
    print("[gpu-case] linear form in a batch", flush=True)
    u0s = [stepper.initial_state(w) for w in ws]
    alone = [_run(w, u0, 7)[0] for w, u0 in zip(ws, u0s)]
    for kw in ({}, dict(one_launch=True)):
        for w, a, b in zip(ws, alone, _run(ws, u0s, 7, **kw)):
            assert np.array_equal(a, b), (w.name, kw)


@pytest.mark.parametrize("ne,n", [(1280, 3), (1280, 1), (320, 11)])
def test_steps_in_a_callers_graph(torch_cuda, ne, n):
    """A caller's capture of adg_run: its replays, the library's own graph and
    direct steps in any order advance one step counter."""
    from paper_2404_03399_amd.solver import Solver
    torch = torch_cuda
    w = _w(ne, 64)
    print(f"[gpu-case] captured run of {n} steps, N={ne}", flush=True)
    u0 = stepper.initial_state(w)
    st = torch.cuda.Stream()
    s = Solver(w, stream=st)
    total = 2 + 4 * n + 16 + 5
    ref = Solver(w)
    v = ref.pack(u0)
    ref.run(v, total, graph=False)
    with torch.cuda.stream(st):
        u = s.pack(u0)
        s.run(u, 2, graph=False)
        s.capture_graph(u)
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            s.run(u, n, graph=False)
        for i in range(4):
            g.replay()
            if i == 1:
                s.run(u, 16)
                float(u.sum())
            if i == 2:
                s.run(u, 5, graph=False)
                float(u.sum())
    st.synchronize()
    assert np.array_equal(s.unpack(u)[0], ref.unpack(v)[0])
    s.close()
    ref.close()


@pytest.mark.parametrize("eq,flux,rk,p,speed,ne,pe", [
    ("advection", "upwind", "lsrk4", 4, -0.75, 405, 15), ("advection", "central", "rk4", 3, 1.3, 129, 3),
    ("burgers", "llf", "ssprk3", 2, 1.0, 125, 125), ("advection", "central", "heun", 1, 1.3, 9, 3)])
def test_general_form_with_odd_pes(torch_cuda, eq, flux, rk, p, speed, ne, pe):
    """Two elements per lane on odd PEs, whose faces lie left of either element
    of a lane (odd meshes, whose lanes straddle the periodic wrap, and one
    within the halo): bitwise one element per lane at one and at the library's
    steps per launch, and the oracle's run."""
    from paper_2404_03399_amd.solver import Solver
    dt = {1: 0.05, 2: 0.02, 3: 0.005, 4: 0.001}[p] * W.TWO_PI / ne * (0.2 if eq == "burgers" else 1.0)
    w = W.Workload(name="odd", scheme="adg_at", rk=rk, degree=p, n_elem=ne, pe_size=pe, equation=eq, flux=flux,
                   probs=W.DELAYS_C2, seed=3, dt=dt, speed=speed, ic=W.PAPER_MULTISINE)
    n = 21
    u0 = stepper.initial_state(w)
    out = {}
    for R in (1, 2, 0):
        for K in (1, 0):
            s = Solver(w, kernel="fused", lane_elems=R, fused_steps=K)
            u = s.pack(u0)
            s.run(u, n, graph=R == 2)
            torch_cuda.cuda.synchronize()
            out[R, K] = s.unpack(u)[0]
            s.close()
    for key, v in out.items():
        assert np.array_equal(v, out[1, 1]), key
    assert stats.rel_l2(out[2, 0], stepper.Stepper(w).run(u0, n)) <= 1e-12
