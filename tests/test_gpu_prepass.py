"""Coefficient 0 of the derivatives by scans over the lanes (supports past the
registers of one thread, octo doubles): a step against the oracle at the edges
of the lanes' shares."""
import pytest
import torch

import mdinputs
import oracle
from gpu_helpers import TOL, host, step_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n,kmin,kmax", [(8, 5, 1, 1), (8, 6, 1, 4), (8, 20, 15, 18), (2, 12, 1, 9), (4, 36, 31, 34),
                                           (4, 70, 62, 66), (2, 140, 126, 131)])
@pytest.mark.parametrize("exps", [(1,), (1, 2, 3)])
def test_step(L, n, kmin, kmax, exps):
    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(L, n, 1, mons=2, kmin=kmin, kmax=kmax, exps=exps, seed=n)
    cst = oracle.manufacture(s)
    drv = mdn.Newton(s, cst)
    drv.step()
    torch.cuda.synchronize()
    assert drv.status_code() == 0
    ref = oracle.newton_step(s, s.cff, cst, s.start())["x"]
    assert step_err(host(drv.x), ref, s.start()) <= TOL[L]


@pytest.mark.parametrize("L,n", [(2, 1), (2, 3), (2, 8), (2, 9), (2, 16), (2, 17), (4, 1), (4, 5), (4, 8), (4, 9)])
def test_steps_of_small_systems(L, n):
    """M of a small system in one launch: single steps and pipelined ones."""
    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(L, n, 6, mons=3, kmin=1, kmax=min(n, 4), exps=(1, 2, 3), seed=40 + n)
    cst = oracle.manufacture(s)
    one, many = mdn.Newton(s, cst), mdn.Newton(s, cst)
    one.step()
    torch.cuda.synchronize()
    assert one.status_code() == 0
    ref = oracle.newton_step(s, s.cff, cst, s.start())["x"]
    assert step_err(host(one.x), ref, s.start()) <= TOL[L]
    for _ in range(2):
        one.step()
    many.steps(3)
    torch.cuda.synchronize()
    assert many.status_code() == 0
    assert step_err(host(many.x), host(one.x), s.start()) <= TOL[L]


@pytest.mark.parametrize("L,n", [(2, 16), (4, 8)])
def test_small_systems_that_need_the_factorization(L, n):
    from test_gpu_inverse import error, linear_system, step

    s, cst = linear_system(L, n, 5, spread=13.0)
    got, status, x0 = step(s, cst)
    assert status == 0
    assert error(s, cst, got, x0) <= TOL[L] * 1e13
