"""The marching x-y pass of large 3D grids against the CPU FP64 oracle.

It is taken from 2^19 cells on in FP64 and from 2^23 on in the FP32 form.  The
sizes put the ends of its waves (58 outputs of 64 lanes, lines of nx + 6 lanes
one after the other) and of its chunks at awkward places: lines shorter than a
wave, exactly one, just over one, many; one-row and one-plane remainders.  Bar:
the parity bar of the separate passes, max|gpu - oracle| / max|oracle| <= 1e-12
per row; the FP32 form bit for bit against the separate passes on a small grid
whose periodic repetition is the large one.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import conservative_errors

pytestmark = pytest.mark.gpu
TOL = 1e-12
P, E, S = W.PERIODIC, W.EXTRAP, W.SLIPWALL


def _say(*a):
    print("[gpu-march]", *a, flush=True)


@pytest.mark.parametrize("n,nf,bc,weno,riemann,low,model", [
    ((52, 101, 101), 2, (E, S, P), 0, 0, 0, 0),    # a line is exactly one wave's outputs
    ((53, 100, 100), 2, (P, E, S), 1, 0, 0, 0),
    ((3, 420, 420), 2, (S, P, E), 0, 0, 0, 0),     # seven lines to a wave
    ((1040, 3, 170), 2, (S, E, P), 0, 1, 0, 0),    # three rows to a column
    ((330, 530, 3), 1, (P, S, E), 0, 0, 2, 0),
    ((58, 97, 95), 2, (E, P, S), 0, 0, 1, 0),
    ((116, 70, 65), 2, (E, E, E), 0, 0, 0, 1),
    ((90, 65, 90), 2, (S, S, S), 1, 1, 0, 0),
])
def test_march_rhs_and_step_match_oracle(n, nf, bc, weno, riemann, low, model):
    from paper_2503_07953_amd.solver import Solver
    _say(n, nf, bc, weno, riemann, low, model)
    assert n[0] * n[1] * n[2] >= 1 << 19
    c = W.random_case(3, n, nf=nf, seed=31, bc=bc, speed=300.0 if nf == 1 else 120.0, interface=model == 0)
    c.weno_variant, c.riemann, c.low_mach, c.model = weno, riemann, low, model
    O = oracle.Oracle(c)
    q = O.prim_to_cons(c.w)
    ref = O.rhs(q)
    S_ = Solver.from_case(c)
    qd = S_.to_device(q)
    err = conservative_errors(S_.rhs(qd).cpu().numpy(), ref, nf, 3)
    assert err.max() <= TOL, err
    dt = torch.zeros(1, dtype=torch.float64, device="cuda")
    S_.step(qd, cfl=0.5, dt_out=dt)
    S_.check()
    dts = O.run(q, 1, cfl=0.5)
    assert abs(dt.item() / dts[0] - 1) <= 1e-13
    err = conservative_errors(qd.cpu().numpy(), q, nf, 3)
    assert err.max() <= TOL, err


@pytest.mark.parametrize("n,reps", [((70, 61, 20), 100), ((131, 61, 20), 100)])
def test_march_fp32_equals_separate_passes_bitwise(n, reps):
    from paper_2503_07953_amd.solver import Solver
    _say("fp32", n, reps)
    assert n[0] * n[1] * n[2] < 1 << 23 <= n[0] * n[1] * n[2] * reps
    # a uniform mixture: finite over the steps (checked with the oracle on the small grid)
    c = W.random_case(3, n, nf=2, seed=32, bc=(S, E, P), speed=60.0, interface=False)
    small = Solver.from_case(c, precision="fp32")
    qs = small.prim_to_cons(small.to_device(c.w))
    kw = dict(c.problem_kwargs())
    kw["n"] = (n[0], n[1], n[2] * reps)
    big = Solver(**kw, precision="fp32")
    qb = qs.repeat(1, reps, 1, 1)

    def tiled(b, a):
        return torch.equal(b.view(a.shape[0], reps, *a.shape[1:]), a.unsqueeze(1).expand(-1, reps, -1, -1, -1))

    assert tiled(big.rhs(qb), small.rhs(qs))
    small.run(qs, 2, cfl=0.5)
    big.run(qb, 2, cfl=0.5)
    small.check()
    big.check()
    assert tiled(qb, qs)
