"""Evaluation and differentiation with two teams of lanes per monomial at the
edges of the teams' sizes, against the oracle."""
import numpy as np
import pytest

import mdinputs
import oracle
from gpu_helpers import TOL, dev, host, matrix_series_err, scaled_err

pytestmark = pytest.mark.gpu

N = 4


@pytest.mark.parametrize("L,D", [(L, D) for L in (1, 2, 4) for D in (1, 2, 3, 4, 5, 8, 9, 10, 16, 17, 32, 33, 34, 64, 65, 127, 128)] +
                         [(8, 1), (8, 2), (8, 5), (8, 9), (8, 16)])
def test_eval_diff(L, D):
    import torch

    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(L, N, D - 1, mons=4, kmin=1, kmax=4, exps=(1, 2, 3), seed=D)
    cst = mdinputs.random_constant(s, 2)
    x = mdinputs.random_series(np.random.default_rng(D), L, N, D, 0.5, 1.5)
    plan = mdn.Plan.from_system(s)
    ws = mdn.workspace(plan.workspace_bytes())
    b = torch.empty((L, N, D), dtype=torch.float64, device="cuda")
    A = torch.empty((L, N, N, D), dtype=torch.float64, device="cuda")
    mdn.eval_diff(plan, dev(s.cff), dev(cst), dev(x), b, A, ws)
    torch.cuda.synchronize()
    ob, oA, scale = oracle.eval_diff(s, s.cff, cst, x)
    assert scaled_err(host(b), ob, scale) <= TOL[L]
    assert matrix_series_err(host(A), oA) <= TOL[L]


@pytest.mark.parametrize("L,D", [(L, D) for L in (2, 4) for D in (1, 2, 3, 5, 8, 9, 16, 17, 32, 33, 65, 128)])
def test_complex_eval_diff(L, D):
    import paper_2301_12659_amd as mdn

    from test_gpu_complex import cerr

    s = mdinputs.tiny(L, N, D - 1, mons=4, kmin=1, kmax=4, exps=(1, 2), seed=D)
    cff, cst, x = mdinputs.complex_random(s, 60 + D)
    b, A = mdn.ComplexNewton(s, cff, cst, x).eval_diff()
    ref = oracle.complex_step(s, cff, cst, x, step=False)
    assert cerr(host(b), ref["b"]) <= TOL[L]
    assert cerr(host(A), np.moveaxis(ref["A"], 2, -1)) <= TOL[L]


@pytest.mark.parametrize("D", [1, 2, 5, 9, 17, 33, 65])
@pytest.mark.parametrize("exps", [(1,), (1, 2, 3)])
def test_values_only(D, exps):
    """Steps whose residual alone has four limbs (the values without the derivatives)."""
    import torch

    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(4, 5, D - 1, mons=3, kmin=1, kmax=5, exps=exps, seed=3)
    cst = oracle.manufacture(s)
    drv = mdn.Newton(s, cst)
    for _ in range(12):
        drv.step(prec_solve=2)
    torch.cuda.synchronize()
    assert drv.status_code() == 0
    err = oracle.absdiff(host(drv.x), s.xstar).max(axis=-1) / np.abs(s.xstar[0]).max(axis=-1)
    assert float(err.max()) <= TOL[4]
