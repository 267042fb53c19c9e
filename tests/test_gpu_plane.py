"""The one-pass 2D evaluation against the CPU oracle, and its two ways to a dt.

Sizes at the edges of its 30 x 14 output tiles and below them, every boundary
kind, both fluid counts and the compile-time options.  Bars: the parity bar 1e-12
per row over 6 fixed steps; and a step whose dt comes from the CFL number, whose
first stage reduces the signal maxima itself, against the same step at that dt:
FP32 bit for bit, FP64 to 1e-13 per row, dt the CFL number over max_signal.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import conservative_errors

pytestmark = pytest.mark.gpu
P, E, S = W.PERIODIC, W.EXTRAP, W.SLIPWALL

CASES = [
    ((3, 3), 2, (P, P), 0, 0, 0, 0, 0.0), ((30, 14), 2, (S, E), 0, 0, 0, 0, 0.0), ((31, 15), 2, (E, S), 1, 1, 0, 0, 0.0),
    ((29, 13), 1, (P, S), 0, 0, 1, 0, 0.0), ((61, 29), 2, (P, P), 3, 0, 2, 0, 0.0), ((5, 43), 2, (S, S), 2, 0, 0, 1, 0.0),
    ((92, 4), 1, (E, E), 0, 0, 0, 0, 0.3), ((45, 57), 2, (P, E), 0, 0, 1, 0, 0.3), ((60, 28), 2, (S, P), 0, 1, 0, 1, 0.0),
]


def _case(n, nf, bc, weno, riemann, low, model, stretch):
    c = W.random_case(2, n, nf=nf, seed=23, bc=bc, speed=40.0, pressure_jump=2.0, interface=False)
    c.weno_variant, c.riemann, c.low_mach, c.model = weno, riemann, low, model
    if stretch:
        c.faces = (W.stretched_faces(n[0], 1.0, stretch), W.stretched_faces(n[1], 1.0, stretch), None)
    return c


@pytest.mark.parametrize("args", CASES)
def test_one_pass_against_the_oracle(args):
    from paper_2503_07953_amd.solver import Solver
    print("[gpu-plane]", args, flush=True)
    c = _case(*args)
    O = oracle.Oracle(c)
    q = O.prim_to_cons(c.w)
    s = Solver.from_case(c)
    qd = s.to_device(q)
    dt = 0.4 / O.max_signal(q)
    O.run(q, 6, dt_fixed=dt)
    for _ in range(6):
        s.step(qd, dt_fixed=dt)
    s.check()
    err = conservative_errors(qd.cpu().numpy(), q, args[1], 2)
    assert err.max() <= 1e-12, err


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("args", CASES)
def test_cfl_step_against_its_own_dt(args, precision):
    from paper_2503_07953_amd.solver import Solver
    print("[gpu-plane cfl]", precision, args, flush=True)
    c = _case(*args)
    s = Solver.from_case(c, precision=precision)
    a = s.prim_to_cons(s.to_device(c.w))
    b = a.clone()
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    smax = s.max_signal(a)
    s.step(a, cfl=0.4, dt_out=dt)
    assert dt.item() == 0.4 / float(smax)
    s.step(b, dt_fixed=dt.item())
    s.check()
    if precision == "fp32":
        assert torch.equal(a, b)
    else:
        err = conservative_errors(b.cpu().numpy(), a.cpu().numpy(), args[1], 2)
        assert err.max() <= 1e-13, err
