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
