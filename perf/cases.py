"""What a user of this library has it do, as cases that can be timed and checked.

A program holds a `Solver` (one problem on one grid) and a state on the GPU and
calls one of the public entry points over and over:

* ``step``      one CFL-limited SSP-RK3 step in place (the production loop),
* ``rhs``       one right-hand side (a program with its own time integrator),
* ``rhs_vjp``   the adjoint of one right-hand side,
* ``step_vjp``  the adjoint of one fixed-dt step from its input state,
* ``rollout``   the checkpointed gradient of the wall-pressure objective: forward
                run and backward sweep.

Inputs are synthetic flows made on the GPU from the seed: ``tube`` (a shock tube
of one gas), ``mixture`` (a smooth air-water mixture, nowhere uniform, which
stays finite over any number of in-place steps), ``bubbles`` (air bubbles in
water hit by a pressure pulse) and ``slab`` (an air-water slab in a random
velocity field).
"""
import math

import numpy as np
import torch

from paper_2503_07953_amd import autograd as AG
from paper_2503_07953_amd.solver import Solver

PERIODIC, EXTRAP, WALL = 0, 1, 2
WATER, AIR = (6.12, 3.43e8, 1000.0), (1.4, 0.0, 1.0)  # gamma, pi_inf, density
FLOOR = 1e-6
CFL = 0.5


def _case(name, op, n, flow, nf=2, prec="fp64", bc="EEE", weno=0, riemann=0, low_mach=0, model=0, stretch=0.0, steps=0):
    n = tuple(n) + (1,) * (3 - len(n))
    c = dict(op=op, nx=n[0], ny=n[1], nz=n[2], flow=flow, nf=nf, prec=prec, bc=bc, weno=weno, riemann=riemann,
             low_mach=low_mach, model=model, stretch=stretch, steps=steps)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the 200-cell shock tube of every first session: launch latency
        _case("tube_200_step_fp64", "step", (200,), "tube", nf=1, bc="E"),
        # the 2D configuration (512^2) and a ragged 2D channel with walls in the FP32 form
        _case("mixture_512x512_step_fp64", "step", (512, 512), "mixture", bc="PP"),
        _case("channel_701x293_step_fp32", "step", (701, 293), "mixture", prec="fp32", bc="PW"),
        # a small 3D problem under a program's own integrator
        _case("bubbles_64_rhs_fp64", "rhs", (64, 64, 64), "bubbles"),
        # the benchmark shapes: 200^3, and the 256^3 bubble cloud in both precisions
        _case("bubbles_200_step_fp64", "step", (200, 200, 200), "bubbles"),
        _case("bubbles_256_step_fp64", "step", (256, 256, 256), "bubbles"),
        _case("bubbles_256_step_fp32", "step", (256, 256, 256), "bubbles", prec="fp32"),
        # the largest configuration: the periodic slab at 512^3 in the FP32 form
        _case("slab_512_step_fp32", "step", (512, 512, 512), "slab", prec="fp32", bc="PPP"),
        # the other reconstruction and face solver on a ragged box
        _case("mixture_150x98x61_wenoz_hll_rhs_fp64", "rhs", (150, 98, 61), "mixture", bc="PEW", weno=1, riemann=1),
        # a grid stretched along every axis
        _case("bubbles_128x96x80_stretched_rhs_fp64", "rhs", (128, 96, 80), "bubbles", stretch=0.3),
        # gradients: the 256^2 configuration's rollout over one checkpointed stretch, and one 3D adjoint
        _case("mixture_256x256_rollout_fp64", "rollout", (256, 256), "mixture", bc="EE", steps=20),
        _case("mixture_96x80x72_rhs_vjp_fp64", "rhs_vjp", (96, 80, 72), "mixture", bc="PEW"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    nd = rng.choice((1, 2, 2, 3, 3, 3, 3))
    op = rng.choice(("step", "step", "step", "rhs", "rhs", "rhs_vjp", "step_vjp"))
    adj = op.endswith("vjp")
    nf = 2 if nd > 1 and rng.random() < 0.8 else rng.choice((1, 2))
    if nd == 1:
        n = (_log(rng, 50, 100000),)
    elif nd == 2:
        n = (_log(rng, 24, 1200), _log(rng, 24, 700 if adj else 1200))
    else:
        top = 70 if op == "step_vjp" else 110 if adj else 260
        n = tuple(_log(rng, 14, top) for _ in range(3))
    if nf == 1:
        flow = "tube" if nd == 1 else "gas"
    else:
        flow = rng.choice(("mixture", "bubbles")) if op == "rhs" and nd == 3 else "mixture"
    bc = "".join(rng.choice("PEW") for _ in range(nd)) if flow != "tube" else "E"
    weno = rng.choice((0, 0, 0, 0, 1, 3))
    riemann = rng.choice((0, 0, 0, 1))
    low = rng.choice((0, 0, 0, 1, 2)) if riemann == 0 else 0
    model = 1 if nf == 2 and flow == "mixture" and rng.random() < 0.15 else 0
    stretch = 0.3 if weno == 0 and not adj and rng.random() < 0.15 else 0.0
    prec = "fp64" if adj else rng.choice(("fp64", "fp64", "fp32"))
    return _case("", op, n, flow, nf, prec, bc, weno, riemann, low, model, stretch)


# ---------------------------------------------------------------------------
# the problem and its inputs
# ---------------------------------------------------------------------------
def _shape(c):
    n = (c["nx"], c["ny"], c["nz"])
    return n, len(c["bc"])


def _neq(c):
    return c["nf"] + _shape(c)[1] + 1 + (2 if c["nf"] == 2 else 0)


def _problem(c):
    n, nd = _shape(c)
    fluids = (WATER, AIR) if c["nf"] == 2 else (AIR, AIR)
    bc = tuple({"P": PERIODIC, "E": EXTRAP, "W": WALL}[b] for b in c["bc"]) + (EXTRAP,) * (3 - nd)
    dx = tuple(1.0 / n[0] if d < nd else 1.0 for d in range(3))
    faces = None
    if c["stretch"]:
        # widths vary smoothly by (1 + a)/(1 - a) along every axis
        faces = []
        for d in range(nd):
            xi = np.arange(n[d] + 1) / n[d]
            faces.append(dx[d] * n[d] * (xi - c["stretch"] * np.sin(2 * np.pi * xi) / (2 * np.pi)))
        faces = tuple(faces) + (None,) * (3 - nd)
    return dict(ndim=nd, n=n, num_fluids=c["nf"], dx=dx, gamma=tuple(f[0] for f in fluids),
                pi_inf=tuple(f[1] for f in fluids), bc_lo=bc, bc_hi=bc, weno_variant=c["weno"], riemann=c["riemann"],
                low_mach=c["low_mach"], model=c["model"], faces=faces)


def _grids(n, nd):
    ax = [(torch.arange(n[d], dtype=torch.float64, device="cuda") + 0.5) / n[d] for d in range(3)]
    return ax[0][None, None, :], ax[1][None, :, None] if nd > 1 else None, ax[2][:, None, None] if nd > 2 else None


def _smooth(rng, n, nd, modes=4, kmax=3):
    """A sum of `modes` separable cosines, scaled to [-1, 1]; periodic on every axis."""
    f = torch.zeros(n[::-1], dtype=torch.float64, device="cuda")
    for _ in range(modes):
        t = rng.uniform(0.3, 1.0)
        for x in _grids(n, nd):
            if x is not None:
                t = t * torch.cos(2 * math.pi * (int(rng.integers(0, kmax + 1)) * x) + rng.uniform(0, 2 * math.pi))
        f += t
    return f / f.abs().max().clamp_min(1e-3)


def _two_fluids(aw, rho_w, rho_a, vel, p, dtype):
    w = torch.empty((5 + len(vel),) + tuple(aw.shape), dtype=dtype, device="cuda")
    w[0] = aw * rho_w
    w[1] = (1.0 - aw) * rho_a
    for d, v in enumerate(vel):
        w[2 + d] = v
    w[2 + len(vel)] = p
    w[3 + len(vel)] = aw
    w[4 + len(vel)] = 1.0 - aw
    return w


def _primitive(c, seed):
    n, nd = _shape(c)
    rng = np.random.default_rng(seed)
    dtype = torch.float64 if c["prec"] == "fp64" else torch.float32
    if c["flow"] in ("tube", "gas"):
        w = torch.empty((nd + 2,) + n[::-1], dtype=torch.float64, device="cuda")
        if c["flow"] == "tube":
            left = (_grids(n, 1)[0] < rng.uniform(0.4, 0.6)).double()
            f = _smooth(rng, n, nd)
            w[0] = (0.125 + 0.875 * left) * (1 + 0.02 * f)
            w[1] = 0.01 * f
            w[2] = (0.1 + 0.9 * left) * (1 + 0.02 * f)
        else:
            w[0] = 1.2 * (1 + 0.3 * _smooth(rng, n, nd))
            for d in range(nd):
                w[1 + d] = 80.0 * _smooth(rng, n, nd)
            w[1 + nd] = 1e5 * (1 + 0.3 * _smooth(rng, n, nd))
        return w.to(dtype)
    if c["flow"] == "mixture":
        aw = 0.5 + 0.3 * _smooth(rng, n, nd)
        vel = [30.0 * _smooth(rng, n, nd) for _ in range(nd)]
        return _two_fluids(aw, WATER[2] * (1 + 0.02 * _smooth(rng, n, nd)), AIR[2] * (1 + 0.25 * _smooth(rng, n, nd)),
                           vel, 1e6 * (1 + 0.3 * _smooth(rng, n, nd)), dtype)
    X, Y, Z = _grids(n, nd)
    if c["flow"] == "bubbles":
        # in cells: radii 3 to 6 % of the shortest edge, six cells apart, interfaces a cell wide; a 100 bar pulse enters along x
        dist = torch.full(n[::-1], 1e3, dtype=torch.float64, device="cuda")
        placed = []
        for _ in range(48):
            r = max(2.0, rng.uniform(0.03, 0.06) * min(n))
            x, y, z = (n[d] * rng.uniform(0.2 if d == 0 else 0.1, 0.9) for d in range(3))
            if any(math.dist((x, y, z), b[:3]) < r + b[3] + 6.0 for b in placed):
                continue
            placed.append((x, y, z, r))
            d2 = (X * n[0] - x) ** 2 + (Y * n[1] - y) ** 2 + (Z * n[2] - z) ** 2
            dist = torch.minimum(dist, torch.sqrt(d2) - r)
        aa = FLOOR + (1 - 2 * FLOOR) * 0.5 * (1 - torch.tanh(dist))
        pulse = 0.5 * (1 - torch.tanh((X - 16.0 / 256) * n[0])) + 0 * aa
        cw = math.sqrt(WATER[0] * (1e5 + WATER[1]) / WATER[2])
        vel = [0.2 * _smooth(rng, n, nd) for _ in range(nd)]
        vel[0] = vel[0] + pulse * ((1e7 - 1e5) / (WATER[2] * cw))
        return _two_fluids(1 - aa, WATER[2], AIR[2], vel, 1e5 * (1 + 0.05 * _smooth(rng, n, nd)) + 1e7 * pulse, dtype)
    zlo = 0.25 + 0.01 * _smooth(rng, (n[0], n[1], 1), 2, kmax=16)
    zhi = 0.75 + 0.01 * _smooth(rng, (n[0], n[1], 1), 2, kmax=16)
    aw = FLOOR + (1 - 2 * FLOOR) * 0.5 * (torch.tanh((Z - zlo) * n[0]) - torch.tanh((Z - zhi) * n[0]))
    vel = [112.0 * _smooth(rng, n, nd, modes=6, kmax=8) for _ in range(nd)]
    return _two_fluids(aw.clamp(FLOOR, 1 - FLOOR), WATER[2], AIR[2], vel, 1e5, dtype)


def _inputs(c, seed):
    """Conservative state and, for the adjoints, the incoming cotangent (each row on the scale of its field)."""
    P = _Exact(c)
    w = _primitive(c, seed)
    q = torch.empty_like(w)
    step = max(1, 2 ** 22 // (w.shape[2] * w.shape[3]))
    for k in range(0, w.shape[1], step):
        q[:, k:k + step] = P.cons(w[:, k:k + step].double())
    del w
    bar = None
    if c["op"].endswith("vjp"):
        g = torch.Generator(device="cuda").manual_seed(seed + 1)
        bar = torch.randn(q.shape, generator=g, dtype=torch.float64, device="cuda")
        bar /= q.flatten(1).std(dim=1).clamp_min(1e-12)[:, None, None, None]
    return q, bar


def _frozen_dt(c):
    """A stable time step that needs no look at the state: 0.3 dx over D times a bound of |u| + c."""
    return 0.3 / c["nx"] / (_shape(c)[1] * (3000.0 if c["nf"] == 2 else 700.0 if c["flow"] == "gas" else 3.0))


def prepare(case, seed):
    S = Solver(precision=case["prec"], **_problem(case))
    q, bar = _inputs(case, seed)
    st = dict(S=S, q=q, bar=bar, op=case["op"], case=case)
    if case["op"] == "step":
        st["dt"] = torch.zeros(1, dtype=torch.float64, device="cuda")
    else:
        st["out"] = S.empty() if case["op"] != "rollout" else None
        st["frozen"] = _frozen_dt(case)
    return st


def run(st):
    S, q, op = st["S"], st["q"], st["op"]
    if op == "step":
        return S.step(q, cfl=CFL, dt_out=st["dt"]), st["dt"]
    if op == "rhs":
        return S.rhs(q, out=st["out"])
    if op == "rhs_vjp":
        return S.rhs_vjp(q, st["bar"], out=st["out"])
    if op == "step_vjp":
        return S.step_vjp(q, st["frozen"], st["bar"], out=st["out"])
    q0 = q.detach().requires_grad_(True)
    q0.grad = None
    J = AG.rollout_objective(q0, S, st["case"]["steps"], st["frozen"], every=10)
    J.backward()
    return J.detach(), q0.grad


def work(case):
    n, nd = _shape(case)
    cells, neq = n[0] * n[1] * n[2], _neq(case)
    size = 8 if case["prec"] == "fp64" else 4
    # one axis of one right-hand side: conversion 21, reconstruction 97 a row, face solver 106, difference and source 30
    rhs = nd * (21 + 97 * neq + 106 + 30) * cells
    state = neq * size * cells
    if case["op"] == "step":
        return dict(bytes=2 * state, flops=3 * rhs + 3 * 4 * neq * cells)
    if case["op"] == "rhs":
        return dict(bytes=2 * state, flops=rhs)
    if case["op"] == "rhs_vjp":
        return dict(bytes=3 * state, flops=3 * rhs)
    if case["op"] == "step_vjp":
        return dict(bytes=3 * state, flops=2 * rhs + 9 * rhs)
    # the program keeps the checkpoints: forward run, replay of each stretch and the reverse sweep
    return dict(bytes=2 * state, flops=case["steps"] * (3 + 3 + 9) * rhs)


# ---------------------------------------------------------------------------
# the same discretization in plain torch, 64 bits
# ---------------------------------------------------------------------------
class _Exact:
    def __init__(self, c):
        p = _problem(c)
        self.nd, self.n, self.nf, self.bc, self.faces = p["ndim"], p["n"], p["num_fluids"], p["bc_lo"], p["faces"]
        self.dx, self.gam, self.pinf = p["dx"], p["gamma"], p["pi_inf"]
        self.weno, self.hll, self.low, self.kapila, self.eps = c["weno"], c["riemann"], c["low_mach"], c["model"], 1e-6
        self.G = [1 / (g - 1) for g in self.gam]
        self.Pi = [g * q / (g - 1) for g, q in zip(self.gam, self.pinf)]
        self.E = self.nf + self.nd
        self.tables = [self._table(d) for d in range(self.nd)] if self.faces else None

    def mix(self, a):
        if self.nf == 1:
            return self.G[0], self.Pi[0]
        return a[0] * self.G[0] + a[1] * self.G[1], a[0] * self.Pi[0] + a[1] * self.Pi[1]

    def rho(self, w):
        return w[0] if self.nf == 1 else w[0] + w[1]

    def cons(self, w):
        rho, v = self.rho(w), w[self.nf:self.E]
        Gam, Pi = self.mix(w[self.E + 1:])
        return torch.cat([w[:self.nf], rho * v, (Gam * w[self.E] + Pi + 0.5 * rho * (v * v).sum(0))[None], w[self.E + 1:]])

    def prim(self, q):
        rho = self.rho(q)
        v = q[self.nf:self.E] / rho
        Gam, Pi = self.mix(q[self.E + 1:])
        return torch.cat([q[:self.nf], v, ((q[self.E] - 0.5 * rho * (v * v).sum(0) - Pi) / Gam)[None], q[self.E + 1:]])

    def remap(self, d, lo, hi):
        """Source cells of positions lo .. hi - 1 along axis d, and the sign of the normal velocity there."""
        i, n = np.arange(lo, hi), self.n[d]
        if self.bc[d] == PERIODIC:
            src = i % n
        elif self.bc[d] == EXTRAP:
            src = np.clip(i, 0, n - 1)
        else:
            src = np.where(i < 0, -1 - i, np.where(i >= n, 2 * n - 1 - i, i))
        sign = np.where((self.bc[d] == WALL) & ((i < 0) | (i >= n)), -1.0, 1.0)
        return torch.from_numpy(src).cuda(), torch.from_numpy(sign).cuda()

    def padded(self, w, d, lo, hi):
        src, sign = self.remap(d, lo, hi)
        ax = 3 - d
        w = w.index_select(ax, src)
        if bool((sign < 0).any()):
            s = sign.reshape([-1 if k == ax - 1 else 1 for k in range(3)])
            m = self.nf + d
            w = torch.cat([w[:m], (w[m] * s)[None], w[m + 1:]])
        return w

    def widths(self, d, lo, hi):
        src, _ = self.remap(d, lo, hi)
        return np.diff(self.faces[d])[src.cpu().numpy()]

    def _table(self, d):
        """Per centre -1 .. n: candidate values at both faces and derivatives as weights of the five cells, and ideal weights."""
        n, h = self.n[d], self.widths(d, -3, self.n[d] + 3)
        cen = np.arange(n + 2) + 2
        hc = h[cen]
        e = np.empty((n + 2, 6))
        e[:, 2], e[:, 3] = -0.5, 0.5
        e[:, 1] = e[:, 2] - h[cen - 1] / hc
        e[:, 0] = e[:, 1] - h[cen - 2] / hc
        e[:, 4] = e[:, 3] + h[cen + 1] / hc
        e[:, 5] = e[:, 4] + h[cen + 2] / hc

        def inverse(r, k):
            a, b = e[:, r:r + k, None], e[:, r + 1:r + k + 1, None]
            j = np.arange(1, k + 1)
            return np.linalg.inv((b ** j - a ** j) / (j * (b - a)))

        m = np.zeros((n + 2, 3, 3, 5))  # centre, candidate, moment, cell
        for r in range(3):
            m[:, r, :, r:r + 3] = inverse(r, 3)
        five = inverse(0, 5)
        out = {"m": m}
        for side, xi in (("r", 0.5), ("l", -0.5)):
            val = m[:, :, 0] + xi * m[:, :, 1] + xi * xi * m[:, :, 2]
            v5 = (five * (xi ** np.arange(5))[None, :, None]).sum(1)
            d0 = v5[:, 0] / val[:, 0, 0]
            d2 = v5[:, 4] / val[:, 2, 4]
            out["v" + side], out["d" + side] = val, np.stack([d0, 1 - d0 - d2, d2], 1)
        return out

    def reconstruct(self, f, ax, d):
        """From cells padded by three: the left value of face c + 1/2 and the right value of face c - 1/2 at centres -1 .. n."""
        m = f.shape[ax] - 4
        s = [f.narrow(ax, k, m) for k in range(5)]
        if self.tables:
            T, res, ind = self.tables[d], [], []

            def apply(w):  # the centre's own value is taken out first: weights sum to one or to zero
                t = torch.from_numpy(np.ascontiguousarray(w)).cuda()
                shape = [-1 if k == ax else 1 for k in range(f.dim())]
                return sum(t[:, k].reshape(shape) * (s[k] - s[2]) for k in range(5) if k != 2)

            for r in range(3):
                ind.append(apply(T["m"][:, r, 1]) ** 2 + 13.0 / 3.0 * apply(T["m"][:, r, 2]) ** 2)
            for side in "rl":
                num, den = 0.0, 0.0
                for r in range(3):
                    dk = torch.from_numpy(np.ascontiguousarray(T["d" + side][:, r])).cuda()
                    a = dk.reshape([-1 if k == ax else 1 for k in range(f.dim())]) / (self.eps + ind[r]) ** 2
                    num, den = num + a * apply(T["v" + side][:, r]), den + a
                res.append(s[2] + num / den)
            return res

        def left(a, b, c, d, e):
            q = [(2 * a - 7 * b + 11 * c) / 6, (-b + 5 * c + 2 * d) / 6, (2 * c + 5 * d - e) / 6]
            be = [13 / 12 * (a - 2 * b + c) ** 2 + 0.25 * (a - 4 * b + 3 * c) ** 2,
                  13 / 12 * (b - 2 * c + d) ** 2 + 0.25 * (b - d) ** 2,
                  13 / 12 * (c - 2 * d + e) ** 2 + 0.25 * (3 * c - 4 * d + e) ** 2]
            lin = (0.1, 0.6, 0.3)
            if self.weno == 1:
                tau = (be[0] - be[2]).abs()
                al = [g * (1 + tau / (x + self.eps)) for g, x in zip(lin, be)]
            else:
                al = [g / (self.eps + x) ** 2 for g, x in zip(lin, be)]
            if self.weno == 3:
                t = al[0] + al[1] + al[2]
                al = [x / t for x in al]
                al = [x * (g + g * g - 3 * g * x + x * x) / (g * g + x * (1 - 2 * g)) for g, x in zip(lin, al)]
            return (al[0] * q[0] + al[1] * q[1] + al[2] * q[2]) / (al[0] + al[1] + al[2])

        return left(*s), left(*s[::-1])

    def side(self, W, d):
        rho, p, u = self.rho(W), W[self.E], W[self.nf + d]
        Gam, Pi = self.mix(W[self.E + 1:])
        v = W[self.nf:self.E]
        E = Gam * p + Pi + 0.5 * rho * (v * v).sum(0)
        return dict(W=W, rho=rho, p=p, u=u, E=E, c=torch.sqrt(((Gam + 1) * p + Pi) / (Gam * rho)))

    def flux(self, WL, WR, d):
        nf, E, N = self.nf, self.E, self.nf + d
        L, R = self.side(WL, d), self.side(WR, d)
        mach = torch.maximum(L["u"].abs() / L["c"], R["u"].abs() / R["c"]).clamp(max=1.0)
        if self.low == 1:
            mean, half = 0.5 * (L["u"] + R["u"]), mach * 0.5 * (L["u"] - R["u"])
            WL = torch.cat([WL[:N], (mean + half)[None], WL[N + 1:]])
            WR = torch.cat([WR[:N], (mean - half)[None], WR[N + 1:]])
            L, R = self.side(WL, d), self.side(WR, d)
        SL, SR = torch.minimum(L["u"] - L["c"], R["u"] - R["c"]), torch.maximum(L["u"] + L["c"], R["u"] + R["c"])

        def conserved(s):
            return torch.cat([s["W"][:nf], s["rho"] * s["W"][nf:E], s["E"][None]])

        def physical(s):
            f = conserved(s) * s["u"]
            return torch.cat([f[:N], (f[N] + s["p"])[None], f[N + 1:E], (f[E] + s["p"] * s["u"])[None]])

        if self.hll:
            a = torch.where(SL >= 0, 1.0, torch.where(SR <= 0, 0.0, SR))
            b = torch.where(SL >= 0, 0.0, torch.where(SR <= 0, 1.0, -SL))
            cc = torch.where((SL >= 0) | (SR <= 0), 0.0, SL * SR)
            r = torch.where((SL >= 0) | (SR <= 0), 1.0, 1 / (SR - SL))
            F = (a * physical(L) + b * physical(R) + cc * (conserved(R) - conserved(L))) * r
            al, ar = WL[E + 1:], WR[E + 1:]
            return torch.cat([F, (a * al * L["u"] + b * ar * R["u"] + cc * (ar - al)) * r]), (a * L["u"] + b * R["u"]) * r
        kL, kR = L["rho"] * (SL - L["u"]), R["rho"] * (SR - R["u"])
        star = (R["p"] - L["p"] + L["u"] * kL - R["u"] * kR) / (kL - kR)
        out = []
        for s, S, sup in ((L, SL, SL >= 0), (R, SR, SR <= 0)):
            chi = (S - s["u"]) / torch.where(sup, torch.ones_like(S), S - star)
            pu = s["p"] / torch.where(sup, torch.ones_like(S), S - s["u"])
            U = conserved(s)
            Us = torch.cat([U[:N], (s["rho"] * star)[None], U[N + 1:E], (s["E"] + (star - s["u"]) * (s["rho"] * star + pu))[None]])
            F = physical(s)
            Fs = F + S * (chi * Us - U)
            if self.low == 2:
                pd = (mach - 1) * kL * kR * (R["u"] - L["u"]) / (kR - kL)
                Fs = torch.cat([Fs[:N], (Fs[N] + pd)[None], Fs[N + 1:E], (Fs[E] + pd * star)[None]])
            out.append((torch.where(sup, F, Fs), torch.where(sup, s["u"], star), s["W"][E + 1:]))
        left = (SL >= 0) | (star >= 0)
        uf = torch.where(left, out[0][1], out[1][1])
        return torch.cat([torch.where(left, out[0][0], out[1][0]), torch.where(left, out[0][2], out[1][2]) * uf]), uf

    def axis(self, wp, w, d):
        ax = 3 - d
        lv, rv = self.reconstruct(wp, ax, d)
        m = lv.shape[ax] - 1
        F, uf = self.flux(lv.narrow(ax, 0, m), rv.narrow(ax, 1, m), d)
        h = 1.0 / self.dx[d]
        if self.faces:
            h = 1 / torch.from_numpy(self.widths(d, self._at, self._at + m - 1)).cuda()
            h = h.reshape([-1 if k == ax - 1 else 1 for k in range(3)])
        r = -torch.diff(F, dim=ax) * h
        if self.nf == 2:
            a, E = w[self.E + 1:], self.E
            if self.kapila:
                z = [g * (w[E] + pi) for g, pi in zip(self.gam, self.pinf)]
                K = (z[1] - z[0]) * a[0] * a[1] / (z[0] * a[1] + z[1] * a[0])
                a = torch.stack([a[0] + K, a[1] - K])
            r = torch.cat([r[:E + 1], r[E + 1:] + a * (torch.diff(uf, dim=ax - 1) * h)])
        return r

    def rhs(self, q):
        q, out = q.double(), []
        step = q.shape[1] if self.nd < 3 else max(1, 2 ** 22 // (q.shape[2] * q.shape[3]))
        whole = self.tables
        for k in range(0, q.shape[1], step):
            hi = min(k + step, q.shape[1])
            w = self.prim(q[:, k:hi])
            self._at, r = 0, 0.0
            for d in range(min(self.nd, 2)):
                r = r + self.axis(self.padded(w, d, -3, self.n[d] + 3), w, d)
            if self.nd == 3:
                if whole:
                    part = {x: v[k:hi + 2] for x, v in whole[2].items()}
                    self.tables = [whole[0], whole[1], part]
                self._at = k
                r = r + self.axis(self.padded_z(q, k - 3, hi + 3), w, 2)
                self.tables = whole
            out.append(r)
        return torch.cat(out, 1)

    def padded_z(self, q, lo, hi):
        return self.prim(self.padded(q, 2, lo, hi))

    def signal(self, q):
        top = torch.zeros((), dtype=torch.float64, device="cuda")
        step = q.shape[1] if self.nd < 3 else max(1, 2 ** 22 // (q.shape[2] * q.shape[3]))
        for k in range(0, q.shape[1], step):
            w = self.prim(q[:, k:k + step].double())
            s = 0.0
            for d in range(self.nd):
                h = 1.0 / self.dx[d]
                if self.faces:
                    lo, hi = (k, min(k + step, self.n[2])) if d == 2 else (0, self.n[d])
                    h = (1 / torch.from_numpy(self.widths(d, lo, hi)).cuda()).reshape([-1 if a == 2 - d else 1 for a in range(3)])
                t = self.side(w, d)
                s = s + (t["u"].abs() + t["c"]) * h
            top = torch.maximum(top, s.max())
        return top

    def step(self, q, dt):
        q = q.double()
        a = q + dt * self.rhs(q)
        a = 0.75 * q + 0.25 * (a + dt * self.rhs(a))
        return q / 3 + 2 / 3 * (a + dt * self.rhs(a))


def exact(case, seed):
    P = _Exact(case)
    q, bar = _inputs(case, seed)
    if case["op"] == "step":
        dt = CFL / P.signal(q)
        return P.step(q, dt), dt.reshape(1)
    if case["op"] == "rhs":
        return P.rhs(q)
    dt = _frozen_dt(case)
    q0 = q.detach().requires_grad_(True)
    if case["op"] == "rhs_vjp":
        return torch.autograd.grad(P.rhs(q0), q0, bar)[0]
    if case["op"] == "step_vjp":
        return torch.autograd.grad(P.step(q0, dt), q0, bar)[0]
    # sum over the steps of dt times the pressure of the last column: each step's own graph, walked back from the end
    states = [q]
    for _ in range(case["steps"]):
        states.append(P.step(states[-1], dt).detach())
    n, nd = _shape(case)
    scale = dt * math.prod(P.dx[1:nd])
    J = scale * sum(P.prim(s)[P.E, :, :, -1].sum() for s in states[1:])
    g = torch.zeros_like(q)
    for k in range(case["steps"], 0, -1):
        s = states[k].requires_grad_(True)
        g = g + torch.autograd.grad(scale * P.prim(s)[P.E, :, :, -1].sum(), s)[0]
        s = states[k - 1].detach().requires_grad_(True)
        g = torch.autograd.grad(P.step(s, dt), s, g)[0]
    return J, g
