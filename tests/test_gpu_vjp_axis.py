"""The axis passes of the RHS adjoint where their waves end.

A wave holds 64 positions of a line, ghosts included, and gives 58 cells; lines
follow one another without a gap.  Two checks over line lengths around those
numbers: on periodic lines a shift of the inputs along any axis shifts the
result bit for bit (each cell's arithmetic is the same in every lane of every
wave), and with walls and extrapolation the result is that of torch autograd
of the FP64 reference, to the bar of the other adjoint tests (ten times the
reference's own spread under a one-ulp change of the state, at least 1e-11, at
most 1e-7).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import field_errors, noise_floor
from oracle import torch_ref as TR

pytestmark = pytest.mark.gpu
P, E, S = W.PERIODIC, W.EXTRAP, W.SLIPWALL


def _say(*a):
    print("[gpu-vjp-axis]", *a, flush=True)


def _solver(case):
    from paper_2503_07953_amd.solver import Solver
    return Solver.from_case(case, precision="fp64")


@pytest.mark.parametrize("n,shift", [
    ((48, 5), (1, 2)), ((49, 3), (29, 1)), ((7, 53), (3, 31)), ((54, 54), (5, 50)), ((3, 116), (1, 57)),
    ((131, 64), (60, 3)), ((6, 5, 50), (1, 2, 23)), ((59, 4, 3), (58, 1, 2)), ((5, 61, 7), (2, 3, 4)),
])
def test_periodic_shift_bitwise(n, shift):
    _say("shift", n, shift)
    nd = len(n)
    c = W.random_case(nd, n, nf=2, seed=91, bc=(P,) * nd, speed=50.0, interface=False)
    s = _solver(c)
    q = s.prim_to_cons(s.to_device(c.w))
    lam = torch.from_numpy(np.random.default_rng(5).normal(size=tuple(q.shape))).cuda()
    g = s.rhs_vjp(q, lam)
    dims = tuple(3 - d for d in range(nd))
    gs = s.rhs_vjp(torch.roll(q, shift, dims).contiguous(), torch.roll(lam, shift, dims).contiguous())
    s.check()
    assert torch.isfinite(g).all()
    assert torch.equal(gs, torch.roll(g, shift, dims))


@pytest.mark.parametrize("n,bc", [
    ((3, 4), (S, E)), ((5, 6), (E, S)), ((52, 7), (S, S)), ((53, 5), (E, E)), ((8, 58), (E, S)), ((59, 3), (S, E)),
    ((6, 116), (S, S)), ((111, 13), (E, S)), ((4, 9, 55), (S, E, S)), ((7, 3, 52), (E, S, E)), ((57,), (S,)), ((117,), (E,)),
])
def test_walls_and_extrapolation_match_reference(n, bc):
    _say("reference", n, bc)
    nd = len(n)
    c = W.random_case(nd, n, nf=2, seed=92, bc=bc, speed=50.0, interface=False)
    O = oracle.Oracle(c)
    q = O.prim_to_cons(c.w)
    lam = np.random.default_rng(6).normal(size=q.shape)
    prob = TR.Problem.from_case(c)

    def ref_fn(a):
        qt = torch.from_numpy(a.copy()).requires_grad_(True)
        return torch.autograd.grad(TR.rhs(prob, qt), qt, torch.from_numpy(lam))[0].numpy()

    ref, spread = noise_floor(ref_fn, q)
    s = _solver(c)
    got = s.rhs_vjp(s.to_device(q), s.to_device(lam)).cpu().numpy()
    s.check()
    err = field_errors(got, ref)
    _say("errors", err, "spread", spread)
    assert np.all(err <= np.minimum(np.maximum(10 * spread, 1e-11), 1e-7)), (err, spread)
