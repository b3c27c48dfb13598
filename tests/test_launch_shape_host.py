"""The launch shape that the library reports (adg_launch_shape), which callers
that count launches go by; no GPU needed."""
import itertools
import os
import sys

import pytest

from paper_2404_03399_amd import adg, solver
from paper_2404_03399_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def _w(ne, pe, **kw):
    kw = dict(dict(rk="rk4", degree=3), **kw)
    if kw.get("equation", "advection") != "advection":
        kw["flux"] = "llf"
    return W.Workload(name="shape", n_elem=ne, pe_size=pe, probs=W.DELAYS_C2, seed=1, dt=1e-9, **kw)


def _shape(ws, n, n_rec=0, **opt):
    ws = ws if isinstance(ws, list) else [ws]
    o = adg.adg_options(**opt)
    return adg.adg_launch_shape([solver.to_problem(w) for w in ws], o, n_rec, n)


@pytest.mark.parametrize("kw", [{}, dict(speed=-1.0), dict(flux="central"), dict(equation="burgers"),
                                dict(equation="viscous_burgers", viscosity=0.1, rk="heun", degree=2)],
                         ids=["upwind", "downwind", "central", "burgers", "viscous"])
@pytest.mark.parametrize("ne,pe", [(64, 16), (1 << 14, 256), (1 << 23, 256), (25 * 40000, 25), (1 << 12, 1), (1 << 12, 2)])
def test_reported_shape_is_one_that_runs(kw, ne, pe):
    w = _w(ne, pe, **kw)
    for n, R, K in itertools.product((1, 2, 3, 5, 16, 1000), (0, 1, 2, 4), (0, 1, 2)):
        if R > pe:
            continue
        r, k = _shape(w, n, lane_elems=R, fused_steps=K)
        assert r in (1, 2, 4) and k in (1, 2, 4, 8) and k <= n
        assert r <= (R or 4) and k <= (K or 8)
    assert _shape(w, 16, kernel=adg.KERNEL["stage"]) == (1, 1)


def test_one_step_launches_take_two_elements():
    """A launch of one step is bound by HBM and keeps two elements per lane where
    longer ones take four."""
    w = _w(1 << 23, 256)
    assert _shape(w, 16) == (4, 8)
    assert _shape(w, 1) == (2, 1)
    assert _shape(w, 16, fused_steps=1) == (2, 1)


def test_calls_of_few_steps():
    """Each number of steps has a list of its own, so that a launch of two steps
    takes two elements per lane where eight take four; a call whose launches
    would end in the other buffer halves its first one from 2^18 elements on."""
    w = _w(1 << 20, 256, flux="central")
    assert [_shape(w, n)[1] for n in (1, 2, 3, 4, 5, 6, 7, 8, 9, 14, 15, 16, 100)] == [
        1, 2, 2, 2, 4, 4, 2, 4, 8, 4, 8, 8, 8]
    assert _shape(w, 2) == (2, 2) and _shape(w, 16) == (4, 8)
    assert _shape(_w(1 << 17, 256), 8)[1] == 8 and _shape(_w(1 << 18, 256), 8)[1] == 4
    assert _shape(_w(1 << 22, 256), 4)[1] == 4 and _shape(_w(1 << 22, 256), 8)[1] == 4
    assert _shape(w, 16, lane_elems=4) == (4, 8) and _shape(w, 2, lane_elems=4, fused_steps=2) == (4, 2)
    assert _shape(w, 2, lane_elems=4) == (2, 2) and _shape(w, 1, lane_elems=4) == (2, 1)


def test_bad_arguments():
    with pytest.raises(adg.AdgError):
        _shape(_w(64, 16), 0)
    with pytest.raises(adg.AdgError):
        _shape(_w(64, 2), 1, lane_elems=4)


def test_bench_asks_the_library():
    """bench.py's rooflines describe the shape that runs: it holds no rule of its
    own, and a solver's shape follows its options, odd PE sizes among them."""
    import bench
    assert not hasattr(bench, "launch_shape")
    s = solver.Solver.__new__(solver.Solver)
    s.ctx, s.n_steps_record = None, 0
    for w, opt in ((_w(1 << 23, 256), dict(fused_steps=1)), (_w(25 * 160000, 25), {}),
                   (_w(25 * 160000, 25, speed=-1.0, rk="lsrk4"), {}), (_w(1 << 20, 4), {})):
        s.probs, s.opt = [solver.to_problem(w)], adg.adg_options(**opt)
        assert s.launch_shape(100) == _shape(w, 100, **opt)


def test_odd_pes_of_local_dg_take_two_elements():
    """One element per lane leaves Heun and eight steps 31 of 64 lanes."""
    kw = dict(equation="viscous_burgers", viscosity=0.1, rk="heun", degree=2)
    odd, even = _w(25 * 40000, 25, **kw), _w(1 << 20, 256, **kw)
    assert _shape(odd, 16) == (2, 8)
    assert _shape([odd, even], 16) == (2, 8)
