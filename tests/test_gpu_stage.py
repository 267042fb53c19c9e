"""The stage combination of every pass rounds as the written-out one: q1 =
fma(dt, r, q), q2 = fma(3/4, q, 1/4 fma(dt, r1, q1)), q3 = fma(1/3, q, 2/3 fma(dt,
r2, q2)) bit for bit, on the rows whose q_k the kernels keep (partial densities and
volume fractions), with r the RHS that `rhs` returns."""
from fractions import Fraction as Fr

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
P, E, S = W.PERIODIC, W.EXTRAP, W.SLIPWALL


def _fma(a, b, c):
    return np.array([float(Fr(float(x)) * Fr(float(y)) + Fr(float(z))) for x, y, z in np.broadcast(a, b, c)])


@pytest.mark.parametrize("nd,n,bc", [(1, (600,), (E,)), (2, (70, 45), (P, S)), (3, (40, 33, 20), (S, P, E)),
                                     (3, (120, 73, 61), (E, S, P))])  # x pass, 2D pass, axis passes, marching pass
def test_stages_round_as_written(nd, n, bc):
    from paper_2503_07953_amd.solver import Solver
    print("[gpu-stage]", n, flush=True)
    c = W.random_case(nd, n, nf=2, seed=8, bc=bc, speed=60.0, interface=False)
    sv = Solver.from_case(c)
    q = sv.prim_to_cons(sv.to_device(c.w))
    dt = 0.3 / sv.max_signal(q).item()
    q1, q2, q3 = torch.empty_like(q), torch.empty_like(q), q.clone()
    sv.step_save_stages(q3, dt, q1, q2)
    sv.check()
    cells = np.random.default_rng(1).integers(0, int(np.prod(n)), 300)
    rows = [0, 1, 3 + nd, 4 + nd]
    pick = lambda t: t.reshape(t.shape[0], -1)[rows][:, cells].cpu().numpy().ravel()
    r, r1, r2 = (pick(sv.rhs(t)) for t in (q, q1, q2))
    a, a1, a2, a3 = (pick(t) for t in (q, q1, q2, q3))
    assert np.array_equal(_fma(dt, r, a), a1)
    assert np.array_equal(_fma(0.75, a, 0.25 * _fma(dt, r1, a1)), a2)
    assert np.array_equal(_fma(1.0 / 3.0, a, (2.0 / 3.0) * _fma(dt, r2, a2)), a3)
