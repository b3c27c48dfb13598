"""The work that a user of this library has it do, as cases to be timed and
compared: forward runs of the stepper from one small mesh to 2^24 elements,
single steps in a caller's own loop, batched ensembles with their statistics,
and the discrete adjoint, each through the public entry points (Solver,
solve_with_grad) at the library's default launch shape.

`exact` steps the same problems in plain torch FP64, written from the scheme
itself, with gradients by automatic differentiation.
"""
from __future__ import annotations

import math
from fractions import Fraction

import numpy as np
import torch

from paper_2404_03399_amd import workloads as W
from paper_2404_03399_amd.autograd import solve_with_grad
from paper_2404_03399_amd.solver import Solver

DELAYS = {"c2": W.DELAYS_C2, "uniform3": W.DELAYS_UNIFORM3, "fig9": W.DELAYS_FIG9, "uniform2": ("1/2", "1/2")}
STAGES = {"heun": 2, "ssprk3": 3, "rk4": 4, "lsrk3": 3, "lsrk4": 5}


def _case(name, kind, **kw):
    """A case: advection upwind RK4 ADG-AT with the delays {0..3} per stage
    unless told otherwise."""
    c = dict(kind=kind, equation="advection", flux="upwind", rk="rk4", scheme="adg_at", degree=3, at_levels=0,
             n_elem=1 << 20, pe_size=256, delays="c2", per_stage=True, sigma=0.005, speed=1.0, n_steps=64,
             n_meshes=1, n_real=1)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest problem of the tests and the smoke run: 64 elements to T = 1
        _case("small_run", "run", degree=2, n_elem=64, pe_size=16, delays="uniform3", sigma=0.04, n_steps=255),
        # a caller's own time loop (output or coupling after every step) on a modest mesh
        _case("step_loop", "step", n_elem=1 << 14, n_steps=32),
        # the headline run: 2^20 elements, 4096 PEs
        _case("advection_2p20", "run", n_steps=64),
        # the same at a size that lives in HBM
        _case("advection_2p24", "run", n_elem=1 << 24, n_steps=32),
        # ragged mesh, small PEs, central flux, five-stage low-storage integrator, degree 4
        _case("central_ragged", "run", flux="central", rk="lsrk4", degree=4, n_elem=99990, pe_size=30, delays="fig9",
              sigma=0.001, n_steps=48),
        # inviscid Burgers with SSP-RK3
        _case("burgers_2p22", "run", equation="burgers", flux="llf", rk="ssprk3", degree=2, n_elem=1 << 22, sigma=0.01,
              n_steps=32),
        # viscous Burgers in local DG form, AT2, Heun, one delay per step
        _case("viscous_2p20", "run", equation="viscous_burgers", flux="llf", rk="heun", degree=2, at_levels=2,
              delays="fig9", per_stage=False, sigma=0.0005, n_steps=64),
        # batched ensemble: meshes of 2^10 to 2^16 elements and degrees 1 to 4, many delay realizations of each
        _case("ensemble_c4", "ensemble", pe_size=64, n_meshes=12, n_real=64, n_steps=16),
        # the scaling experiment: one mesh, P = 2..32, delay realizations of each, then the group statistics
        _case("scaling_at2", "scaling", rk="heun", degree=1, n_elem=512, delays="fig9", per_stage=False, sigma=0.1,
              n_real=32, n_steps=200),
        # recorded run and its adjoint with the gradient of the speed, checkpoints every 64 steps
        _case("adjoint_2p20", "adjoint", n_steps=128),
        # gradient of the initial state through torch.autograd
        _case("grad_u0_2p17", "grad", n_elem=1 << 17, n_steps=64),
        # the nonlinear adjoint
        _case("adjoint_burgers_2p18", "adjoint", equation="burgers", flux="llf", rk="ssprk3", degree=2,
              n_elem=1 << 18, sigma=0.01, n_steps=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any equation, flux, integrator, degree, mesh (ragged
    ones among them), PE size, delay set and length of run, so that a pass
    costs no more than the largest listed one."""
    kind = rng.choice(["run", "run", "run", "run", "step", "ensemble", "scaling", "adjoint", "adjoint", "grad"])
    delays = rng.choice(["c2", "uniform3", "fig9", "uniform2"])
    if kind == "ensemble":
        return _case(None, kind, pe_size=rng.choice([16, 32, 64]), delays=delays, n_meshes=rng.randint(2, 12),
                     n_real=_log_int(rng, 2, 64), n_steps=rng.randint(4, 32), sigma=0.004)
    if kind == "scaling":
        if rng.random() < 0.5:
            return _case(None, kind, rk="heun", degree=1, n_elem=64 * _log_int(rng, 1, 16), delays=delays,
                         per_stage=False, sigma=0.05, n_real=rng.randint(8, 64), n_steps=_log_int(rng, 20, 300))
        return _case(None, kind, rk="rk4", degree=3, n_elem=64 * _log_int(rng, 1, 16), delays=delays, per_stage=False,
                     sigma=0.005, n_real=rng.randint(8, 64), n_steps=_log_int(rng, 20, 300))
    back = kind in ("adjoint", "grad")
    eq = rng.choice(["advection", "advection", "advection", "burgers"] + ([] if back else ["viscous_burgers"]))
    degree = rng.choice([1, 2, 3, 4])
    rk = rng.choice(["heun", "ssprk3", "rk4", "rk4", "lsrk3", "lsrk4"])
    pe = rng.choice([16, 25, 32, 48, 64, 100, 128, 256, 256, 1000])
    total = _log_int(rng, 64, (1 << 20) if back else (1 << 23))
    n_pe = max(2, total // pe)
    n_steps = _log_int(rng, 4, 64) if total > (1 << 20) else _log_int(rng, 8, 128)
    c = dict(equation=eq, degree=degree, rk=rk, n_elem=n_pe * pe, pe_size=pe, delays=delays, n_steps=n_steps,
             per_stage=rng.random() < 0.5, scheme=rng.choice(["adg_at", "adg_at", "adg_at", "adg", "dg"]),
             speed=rng.choice([1.0, 1.0, 1.5, -0.75]), sigma={1: 0.02, 2: 0.005, 3: 0.003, 4: 0.001}[degree])
    if eq == "advection":
        c["flux"] = rng.choice(["upwind", "upwind", "upwind", "central"])
    else:
        c.update(flux="llf", speed=1.0)
    if eq == "viscous_burgers":
        c.update(sigma=0.0005, at_levels=2 if c["scheme"] == "adg_at" else 0, per_stage=False)
    return _case(None, kind, **c)


# ---- problems ----------------------------------------------------------------
def _viscosity(case):
    return 0.1 if case["equation"] == "viscous_burgers" else 0.0


def problems(case, seed):
    """The problems of a case (parameters only; every draw from the seed)."""
    rng = np.random.default_rng([seed, 17])
    probs = DELAYS[case["delays"]]

    def one(n_elem, pe_size, degree, sigma, delay_seed, ic, a_max, rk=case["rk"]):
        dx = W.TWO_PI / n_elem
        nu = _viscosity(case)
        if nu:
            sigma = min(sigma, 0.002 * dx * a_max / nu)  # explicit diffusive limit
        return W.Workload(name="case", equation=case["equation"], scheme=case["scheme"], flux=case["flux"], rk=rk,
                          degree=degree, n_elem=n_elem, pe_size=pe_size, probs=probs, seed=int(delay_seed),
                          per_stage=case["per_stage"], at_levels=case["at_levels"], speed=case["speed"],
                          viscosity=nu, dt=sigma * dx / a_max, n_steps=case["n_steps"], ic=ic)

    if case["kind"] == "ensemble":
        # meshes of the paper's shapes: the sizes and degrees are the case's, the delays and phases the seed's
        shape = np.random.default_rng([case["n_meshes"], 4])
        us = shape.uniform(10.0, 16.0, size=case["n_meshes"])
        ps = shape.integers(1, 5, size=case["n_meshes"])
        out = []
        for m in range(case["n_meshes"]):
            ne = 64 * max(1, round(2.0 ** us[m] / 64.0))
            sigma = {1: 0.05, 2: 0.01, 3: 0.005, 4: 0.001}[int(ps[m])]
            ic = W.MultiSine((2, 3, 5), (3.0, 2.0, 1.0), tuple(float(x) for x in rng.uniform(0, W.TWO_PI, 3)))
            out += [one(ne, case["pe_size"], int(ps[m]), sigma, (seed << 32) | (m << 16) | r, ic, 1.0)
                    for r in range(case["n_real"])]
        return out
    if case["kind"] == "scaling":
        ic = W.MultiSine((2, 3), (2.0, 1.0), tuple(float(x) for x in rng.uniform(0, W.TWO_PI, 2)))
        return [one(case["n_elem"], case["n_elem"] // npe, case["degree"], case["sigma"],
                    (seed << 32) | (npe << 16) | r, ic, 1.0)
                for npe in (2, 4, 8, 16, 32) for r in range(case["n_real"])]
    if case["equation"] == "burgers":
        ic, a_max = W.MultiSine((1,), (1.0,), (float(rng.uniform(0, W.TWO_PI)),), 0.5), 1.5
    elif case["equation"] == "viscous_burgers":
        ic = W.MultiSine((2, 3, 5), (3.0, 2.0, 1.0), tuple(float(x) for x in rng.uniform(0, W.TWO_PI, 3)))
        a_max = 6.0
    else:
        kmax = 32 if case["n_elem"] >= 512 else 4
        ic, a_max = W.MultiSine(tuple(int(k) for k in rng.integers(1, kmax + 1, 8)),
                                tuple(float(x) for x in rng.standard_normal(8)),
                                tuple(float(x) for x in rng.uniform(0, W.TWO_PI, 8))), abs(case["speed"])
    return [one(case["n_elem"], case["pe_size"], case["degree"], case["sigma"], seed, ic, a_max)]


def _target_modes(seed):
    """Modes of the target state u_ref of the misfit 1/2 |u(T) - u_ref|^2."""
    rng = np.random.default_rng([seed, 23])
    return rng.integers(1, 9, 4), rng.standard_normal(4), rng.uniform(0, W.TWO_PI, 4)


def _target(x, seed):
    v = torch.zeros_like(x)
    for k, a, ph in zip(*_target_modes(seed)):
        v = v + float(a) * torch.sin(int(k) * x + float(ph))
    return v


# ---- the framework's side ------------------------------------------------------
def prepare(case, seed):
    ws = problems(case, seed)
    st = {"case": case, "ws": ws}
    if case["kind"] == "grad":
        # the initial state that the program differentiates by, and the target
        s = Solver(ws[0])
        st["u0"] = s.initial_state().requires_grad_(True)
        ref = s.empty_state()
        s.view(ref).copy_(_target(s.nodes(), seed))
        st["ref"], st["speed"], st["view"] = ref, torch.tensor(ws[0].speed, dtype=torch.float64), s
        return st
    rec = case["n_steps"] if case["kind"] == "adjoint" else 0
    s = Solver(ws, n_steps_record=rec, ckpt_every=64 if rec else 0)
    st["solver"], st["u"] = s, s.initial_state()
    if case["kind"] == "adjoint":
        st["u0"], st["ref"] = st["u"].clone(), s.empty_state()
        s.view(st["ref"]).copy_(_target(s.nodes(), seed))
    if case["kind"] == "scaling":
        st["ref"] = s.exact_advection_state(ws[0].dt * case["n_steps"])
        st["group"] = [i // case["n_real"] for i in range(len(ws))]
    return st


def run(st):
    case, n = st["case"], st["case"]["n_steps"]
    if case["kind"] == "grad":
        u0 = st["u0"]
        u0.grad = None
        u = solve_with_grad(u0, st["speed"], st["ws"][0], n)
        loss = 0.5 * (u - st["ref"]).square().sum()
        loss.backward()
        return st["view"].view(u.detach()), st["view"].view(u0.grad)
    s, u = st["solver"], st["u"]
    if case["kind"] == "step":
        for _ in range(n):
            s.step(u)
        return s.view(u)
    if case["kind"] == "adjoint":
        s.reset()
        u.copy_(st["u0"])
        s.run(u, n, record=True)
        g, gs = s.adjoint(u - st["ref"])
        return (s.view(u), s.view(g)) + ((float(gs[0]),) if case["equation"] == "advection" else ())
    s.run(u, n)
    if case["kind"] == "scaling":
        return u, [float(x) for row in s.ensemble_stats(u, st["ref"], st["group"], 5) for x in row[0::2]]
    return u if case["kind"] == "ensemble" else s.view(u)  # the ensemble's meshes have no padding


def work(case):
    """Bytes: the initial state read and the final one written, and for the
    adjoint the cotangent and the gradient too.  Flops: the element operator
    (volume term and two lifts), the flux and the update of every stage."""
    dofs = flops = 0
    for w in problems(case, 0):
        n = w.degree + 1
        per = 2 * n * n + 4 * n + 4 + 4 * n + (2 * n * n + 4 * n if _viscosity(case) else 0)
        dofs += w.n_elem * n
        flops += w.n_elem * STAGES[w.rk] * per * case["n_steps"]
    back = case["kind"] in ("adjoint", "grad")
    return {"bytes": 8.0 * dofs * (4 if back else 2 if case["kind"] != "scaling" else 3),
            "flops": float(flops) * (2 if back else 1)}


# ---- the same in plain torch, 64 bits ------------------------------------------
def _operators(p):
    """GLL nodes and D = M^-1 S, M^-1 phi(-1), M^-1 phi(1) with exact M and S."""
    x = {1: [-1.0, 1.0], 2: [-1.0, 0.0, 1.0], 3: [-1.0, -math.sqrt(0.2), math.sqrt(0.2), 1.0],
         4: [-1.0, -math.sqrt(3.0 / 7.0), 0.0, math.sqrt(3.0 / 7.0), 1.0]}[p]
    qx, qw = np.polynomial.legendre.leggauss(p + 2)
    phi = np.ones((p + 1, len(qx)))
    dphi = np.zeros((p + 1, len(qx)))
    for j in range(p + 1):
        poly = np.poly1d([1.0])
        for m in range(p + 1):
            if m != j:
                poly = poly * np.poly1d([1.0, -x[m]]) / (x[j] - x[m])
        phi[j], dphi[j] = poly(qx), poly.deriv()(qx)
    M, S = (phi * qw) @ phi.T, (dphi * qw) @ phi.T
    e0, ep = np.eye(p + 1)[0], np.eye(p + 1)[p]
    return np.array(x), np.linalg.solve(M, S), np.linalg.solve(M, e0), np.linalg.solve(M, ep)


def _mix(x):
    """SplitMix64 on uint64 arrays."""
    with np.errstate(over="ignore"):
        z = x + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


LOW = {"lsrk3": (("0", "-5/9", "-153/128"), ("1/3", "15/16", "8/15")),
       "lsrk4": (("0", "-567301805773/1357537059087", "-2404267990393/2016746695238",
                  "-3550918686646/2091501179385", "-1275806237668/842570457699"),
                 ("1432997174477/9575080441755", "5161836677717/13612068292357", "1720146321549/2090206949498",
                  "3134564353537/4481467310338", "2277821191437/14882151754819"))}


class _Plain:
    """Problems of one shape (they differ in their delay seeds), stepped as
    tensors (problem, node, element)."""

    def __init__(self, ws, device):
        w = ws[0]
        self.w, self.p, self.N = w, w.degree, w.n_elem
        self.x, self.D, self.ll, self.lr = _operators(w.degree)
        self.two_dx = 2.0 * w.n_elem / w.length
        self.seeds = np.array([v.seed for v in ws], dtype=np.uint64)
        self.P = w.n_elem // w.pe_size
        self.async_ = w.scheme != "dg" and self.P > 1
        self.q = (w.at_levels or w.degree + 1) if w.scheme == "adg_at" else 1
        self.dev = device
        self.idx = torch.arange(self.P, device=device) * w.pe_size
        acc, self.edges = Fraction(0), []
        for pr in w.probs[:-1]:
            acc += Fraction(pr)
            self.edges.append(np.uint64(math.floor(acc * (1 << 53))))
        L = len(w.probs)
        c = np.zeros((L, self.q))
        for k in range(L):
            for j in range(self.q):
                f = Fraction(1)
                for m in range(self.q):
                    if m != j:
                        f *= Fraction(k + m, m - j)
                c[k, j] = float(f)
        self.c = torch.tensor(c, device=device)
        self.keep = L + self.q
        self.hist = {}
        self.a = torch.tensor(w.speed, dtype=torch.float64, device=device)

    def nodes(self):
        e = torch.arange(self.N, dtype=torch.float64, device=self.dev)
        dx = self.w.length / self.N
        xi = torch.tensor(self.x, device=self.dev)
        return self.w.x_left + e[None] * dx + (xi[:, None] + 1.0) * (dx / 2.0)

    def start(self):
        x, ic = self.nodes(), self.w.ic
        v = torch.full_like(x, ic.offset)
        for k, a, ph in zip(ic.kappa, ic.amp, ic.phase):
            v = v + a * torch.sin(k * x + ph)
        return v[None].repeat(len(self.seeds), 1, 1)

    def delays(self, n, s):
        h = _mix(self.seeds)
        h = _mix(h ^ np.uint64(n))
        h = _mix(h ^ np.uint64(s if self.w.per_stage else 0))
        u = _mix(h[:, None] ^ np.arange(self.P, dtype=np.uint64)[None]) >> np.uint64(11)
        k = sum((u >= t).astype(np.int64) for t in self.edges) if self.edges else np.zeros(u.shape, np.int64)
        return torch.from_numpy(np.minimum(k, max(0, n - self.q + 1))).to(self.dev)

    def face(self, F, n, s, which):
        """PE faces: keep the level-n values, take the AT combination."""
        if not self.async_:
            return F
        raw = F[:, self.idx]
        past = [raw] + self.hist.get((which, s), [])[: self.keep]
        self.hist[(which, s)] = past
        H, k = torch.stack(past), self.delays(n, s)
        at = torch.zeros_like(raw)
        for j in range(self.q):
            lev = torch.clamp(k + j, max=len(past) - 1)
            at = at + self.c[:, j][k] * torch.gather(H, 0, lev[None])[0]
        F = F.clone()
        F[:, self.idx] = torch.where(k == 0, raw, at)
        return F

    @staticmethod
    def mul(A, y):
        return torch.stack([sum(float(A[i, j]) * y[:, j] for j in range(A.shape[1])) for i in range(A.shape[0])], 1)

    def lift(self, v, F):
        return torch.stack([float(x) * F for x in v], 1)

    def operator(self, y, n, s):
        w = self.w
        um, up = torch.roll(y[:, -1], 1, -1), y[:, 0]
        if w.equation == "advection":
            F = 0.5 * (um + up) if w.flux == "central" else (um if w.speed > 0 else up)
            F = self.face(F, n, s, "f")
            r = self.mul(self.D, y) + self.lift(self.ll, F) - self.lift(self.lr, torch.roll(F, -1, -1))
            return self.two_dx * self.a * r
        lam = torch.maximum(um.abs(), up.abs())
        F = 0.25 * (um * um + up * up) - 0.5 * lam * (up - um)
        g = 0.5 * y * y
        if w.equation == "viscous_burgers":
            h = self.face(um, n, s, "u")
            q = self.two_dx * (self.lift(self.lr, torch.roll(h, -1, -1)) - self.lift(self.ll, h) - self.mul(self.D, y))
            F, g = F - w.viscosity * q[:, 0], g - w.viscosity * q
        F = self.face(F, n, s, "f")
        r = self.mul(self.D, g) + self.lift(self.ll, F) - self.lift(self.lr, torch.roll(F, -1, -1))
        return self.two_dx * r

    def step(self, u, n):
        dt, L, rk = self.w.dt, self.operator, self.w.rk
        if rk == "heun":
            k1 = dt * L(u, n, 0)
            return u + 0.5 * (k1 + dt * L(u + k1, n, 1))
        if rk == "ssprk3":
            u1 = u + dt * L(u, n, 0)
            u2 = 0.75 * u + 0.25 * (u1 + dt * L(u1, n, 1))
            return u / 3.0 + (2.0 / 3.0) * (u2 + dt * L(u2, n, 2))
        if rk == "rk4":
            k1 = L(u, n, 0)
            k2 = L(u + 0.5 * dt * k1, n, 1)
            k3 = L(u + 0.5 * dt * k2, n, 2)
            return u + (dt / 6.0) * (k1 + 2.0 * k2 + 2.0 * k3 + L(u + dt * k3, n, 3))
        d, y = 0.0, u
        for s, (a, b) in enumerate(zip(*LOW[rk])):
            d = float(Fraction(a)) * d + dt * L(y, n, s)
            y = y + float(Fraction(b)) * d
        return y

    def evolve(self, u, n_steps):
        for n in range(n_steps):
            u = self.step(u, n)
        return u


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    ws, n = problems(case, seed), case["n_steps"]
    if case["kind"] in ("adjoint", "grad"):
        # what automatic differentiation keeps of every stage has to fit the card
        kept = 3 if case["equation"] == "advection" else 12
        if 8.0 * kept * ws[0].n_elem * (ws[0].degree + 1) * STAGES[ws[0].rk] * n > 100e9:
            return None
        P = _Plain(ws, dev)
        want_speed = case["kind"] == "adjoint" and case["equation"] == "advection"
        u0 = P.start().requires_grad_(True)
        P.a.requires_grad_(want_speed)
        u = P.evolve(u0, n)
        J = 0.5 * (u - _target(P.nodes(), seed)).square().sum()
        J.backward()
        return (u.detach()[0], u0.grad[0]) + ((float(P.a.grad),) if want_speed else ())
    with torch.no_grad():
        out, groups = [], {}
        for w in ws:
            groups.setdefault((w.n_elem, w.degree, w.pe_size, w.ic), []).append(w)
        plain = [_Plain(g, dev) for g in groups.values()]
        for P in plain:
            u = P.start()
            # the step loop and the runs start at step 0
            out.append(P.evolve(u, n))
        if case["kind"] == "scaling":
            stats = []
            for P, u in zip(plain, out):
                x, ic = P.nodes() - P.w.speed * (P.w.dt * n), P.w.ic
                v = torch.full_like(x, ic.offset)
                for k, a, ph in zip(ic.kappa, ic.amp, ic.phase):
                    v = v + a * torch.sin(k * x + ph)
                d = (u - v[None]).abs().flatten(1)
                stats += [float(d.mean(1).mean()), float(d.amax(1).mean())]
            return torch.cat([u.reshape(-1) for u in out]), stats
        if case["kind"] == "ensemble":
            return torch.cat([u.reshape(-1) for u in out])
        return out[0][0]
