"""Evaluation and differentiation on digits (octo doubles, orders from 17): at
the edges of the kernel's sizes and on series whose coefficients' sizes differ
widely, against the oracle."""
import numpy as np
import pytest

import mdinputs
import oracle
from gpu_helpers import TOL, dev, host, matrix_series_err, scaled_err

pytestmark = pytest.mark.gpu

L, N = 8, 4


def points(D):
    x = mdinputs.random_series(np.random.default_rng(D), L, N, D, 0.5, 1.5)
    k = np.arange(D)
    scale = lambda e: np.ldexp(x, np.asarray(e).astype(np.int32))
    yield "even", x
    # every variable a slope of its own: terms of a product hundreds of bits apart
    yield "steep", scale(np.array([-3, 1, 2, -2])[:, None] * k)
    # exp-like decay
    yield "factorial", scale(-np.round(np.cumsum(np.log2(np.maximum(k, 1))))[None])
    yield "wild", scale(np.random.default_rng(D + 1).integers(-25, 26, size=(N, D)))
    yield "zeros", x * (np.random.default_rng(D + 2).random((N, D)) < 0.5)
    start = x.copy()
    start[:, :, 1:] = 0.0
    yield "start", start


@pytest.mark.parametrize("D", [17, 31, 32, 33, 64, 65, 128])
def test_eval_diff(D):
    import torch

    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(L, N, D - 1, mons=3, kmin=1, kmax=4, exps=(1, 2, 3), seed=D)
    cst = mdinputs.random_constant(s, 2)
    plan = mdn.Plan.from_system(s)
    ws = mdn.workspace(plan.workspace_bytes())
    b = torch.empty((L, N, D), dtype=torch.float64, device="cuda")
    A = torch.empty((L, N, N, D), dtype=torch.float64, device="cuda")
    for name, x in points(D):
        x = np.ascontiguousarray(x)
        mdn.eval_diff(plan, dev(s.cff), dev(cst), dev(x), b, A, ws)
        torch.cuda.synchronize()
        ob, oA, scale = oracle.eval_diff(s, s.cff, cst, x)
        assert scaled_err(host(b), ob, scale) <= TOL[L], name
        assert matrix_series_err(host(A), oA) <= TOL[L], name


def test_values_only():
    """A step whose residual alone has eight limbs (team A without team B)."""
    import torch

    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(L, 5, 19, mons=3, kmin=1, kmax=5, exps=(1, 2), seed=3)
    cst = oracle.manufacture(s)
    drv = mdn.Newton(s, cst)
    for _ in range(12):
        drv.step(prec_solve=4)
    torch.cuda.synchronize()
    assert drv.status_code() == 0
    err = oracle.absdiff(host(drv.x), s.xstar).max(axis=-1) / np.abs(s.xstar[0]).max(axis=-1)
    assert float(err.max()) <= TOL[L]


def test_nonfinite_is_reported():
    import torch

    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(L, 4, 20, mons=3, kmin=2, kmax=3, exps=(1,), seed=4)
    x = s.start()
    x[0, 1, 5] = np.nan
    drv = mdn.Newton(s, mdinputs.random_constant(s, 2), x)
    drv.step()
    torch.cuda.synchronize()
    assert drv.status_code() == mdn.MD_ENONFINITE
