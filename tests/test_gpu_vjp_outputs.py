"""What the last pass of an RHS adjoint does with its result: adding to q_bar
(accumulate), and the reverse stage combination of a step, against the plain
result combined here.  Adding is two terms: bar 8 eps of them.  In a step the roundings of
the stages' cotangents pass through the later adjoints, sums of up to a few hundred
terms of either sign a cell: bar 1e-12 of the row's largest entry (a wrong coefficient
shows at 0.1).
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
P, E, S = W.PERIODIC, W.EXTRAP, W.SLIPWALL
CASES = [(1, (70,), 2, (S,)), (1, (64,), 1, (E,)), (2, (70, 45), 2, (E, S)), (2, (5, 130), 1, (P, E)),
         (3, (20, 17, 14), 2, (S, P, E)), (3, (3, 4, 67), 2, (E, S, P))]


def _setup(nd, n, nf, bc):
    from paper_2503_07953_amd.solver import Solver
    print("[gpu-vjp-outputs]", n, nf, bc, flush=True)
    c = W.random_case(nd, n, nf=nf, seed=90 + nd, bc=bc, speed=200.0 if nf == 1 else 60.0, interface=False)
    sv = Solver.from_case(c)
    q = sv.prim_to_cons(sv.to_device(c.w))
    g = torch.Generator(device="cuda").manual_seed(3)
    scale = q.flatten(1).abs().mean(1).clamp_min(1e-6)[:, None, None, None]
    rand = lambda: torch.randn(q.shape, generator=g, dtype=torch.float64, device="cuda") / scale
    return sv, q, rand


def _close(got, ref, terms, bar=8 * np.finfo(float).eps):
    err = ((got - ref).abs() / terms.clamp_min(1e-300)).max().item()
    print(f"[gpu-vjp-outputs] {err:.1e} of the terms", flush=True)
    assert err <= bar


@pytest.mark.parametrize("nd,n,nf,bc", CASES)
def test_accumulate_adds_the_plain_result(nd, n, nf, bc):
    sv, q, rand = _setup(nd, n, nf, bc)
    lam = rand()
    plain = sv.rhs_vjp(q, lam)
    before = plain.flip(1, 2, 3) + plain.abs().mean()
    out = before.clone()
    sv.rhs_vjp(q, lam, out=out, accumulate=True)
    sv.check()
    assert plain.abs().max() > 0
    _close(out, before + plain, before.abs() + plain.abs())


@pytest.mark.parametrize("nd,n,nf,bc", CASES)
def test_step_adjoint_is_three_rhs_adjoints_combined(nd, n, nf, bc):
    sv, q, rand = _setup(nd, n, nf, bc)
    dt = 0.2 / sv.max_signal(q).item()
    q1, q2 = torch.empty_like(q), torch.empty_like(q)
    sv.step_save_stages(q.clone(), dt, q1, q2)
    x = rand()
    got = sv.step_vjp_stages(q, q1, q2, dt, x)
    same = sv.step_vjp(q, dt, x)
    b2 = (2.0 / 3.0) * (x + dt * sv.rhs_vjp(q2, x))
    b1 = 0.25 * (b2 + dt * sv.rhs_vjp(q1, b2))
    v0 = sv.rhs_vjp(q, b1)
    sv.check()
    assert torch.equal(got, same)
    ref = x / 3 + 0.75 * b2 + (b1 + dt * v0)
    terms = ref.flatten(1).abs().amax(1)[:, None, None, None].expand_as(ref)
    _close(got, ref, terms, bar=1e-12)
