"""The x pass of 3D grids against the CPU oracle where its waves run from one x
line into the next: lines shorter than a wave, just longer than one and of two
and more, every boundary kind, with the options that change its stencil work.
Bar: the parity bar 1e-12 per row over 3 fixed steps (grids below the marching
pass's sizes, above the 2048 waves up to which lines start on waves of their own).
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
    ((3, 64, 40), 2, P, 0, 0, 0.0), ((7, 50, 45), 1, S, 0, 0, 0.0), ((31, 60, 40), 2, E, 2, 0, 0.0),
    ((55, 46, 45), 2, S, 0, 1, 0.0), ((64, 40, 30), 2, E, 1, 0, 0.0), ((65, 33, 40), 1, P, 3, 0, 0.0),
    ((125, 30, 40), 2, P, 0, 0, 0.3), ((130, 30, 24), 2, S, 0, 2, 0.0),
]


def _case(n, nf, bcx, weno, low, stretch):
    c = W.random_case(3, n, nf=nf, seed=29, bc=(bcx, P, E), speed=40.0, pressure_jump=2.0, interface=False)
    c.weno_variant, c.low_mach = weno, low
    if stretch:
        c.faces = tuple(W.stretched_faces(m, 1.0, stretch) for m in n)
    return c


@pytest.mark.parametrize("args", CASES)
def test_lines_against_the_oracle(args):
    from paper_2503_07953_amd.solver import Solver
    print("[gpu-xlines]", args, flush=True)
    c = _case(*args)
    O = oracle.Oracle(c)
    q = O.prim_to_cons(c.w)
    s = Solver.from_case(c)
    qd = s.to_device(q)
    dt = 0.4 / O.max_signal(q)
    O.run(q, 3, dt_fixed=dt)
    for _ in range(3):
        s.step(qd, dt_fixed=dt)
    s.check()
    err = conservative_errors(qd.cpu().numpy(), q, args[1], 3)
    assert err.max() <= 1e-12, err
