"""A face array that set_grid refuses leaves the context on the grid it had.

The refusal comes after the other axes' tables are known: none of them may be
installed alone, since the kernels read every axis' table once one is set."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd,n,axis", [(3, (20, 17, 14), 2), (3, (20, 17, 14), 1), (2, (33, 40), 1), (1, (70,), 0)])
@pytest.mark.parametrize("precision", ("fp64", "fp32"))
def test_a_refused_axis_changes_nothing(nd, n, axis, precision):
    from paper_2503_07953_amd import _lib as L
    from paper_2503_07953_amd.solver import Solver
    print("[gpu-set-grid]", n, axis, precision, flush=True)
    c = W.random_case(nd, n, nf=2, seed=17, bc=(W.EXTRAP,) * nd, speed=60.0, interface=False)
    S = Solver.from_case(c, precision=precision)
    q = S.prim_to_cons(S.to_device(c.w))
    uniform = S.rhs(q).clone()
    # increasing and finite, but one cell 1e200 times smaller than its neighbours
    bad = np.arange(n[axis] + 1) * c.dx[axis]
    bad[1] = 1e-200
    with pytest.raises(L.MfcError, match="singular"):
        S.set_grid(axis, bad)
    assert torch.equal(S.rhs(q), uniform)
    good = np.arange(n[0] + 1) / n[0]
    S.set_grid(0, (good + 0.3 * np.sin(2 * np.pi * good) / (2 * np.pi)) * n[0] * c.dx[0])
    stretched = S.rhs(q).clone()
    assert not torch.equal(stretched, uniform)
    with pytest.raises(L.MfcError, match="singular"):
        S.set_grid(axis, bad)
    assert torch.equal(S.rhs(q), stretched)
    S.check()
