"""Paths of other orders in one batch: a path's step does not depend on the
paths beside it."""
import numpy as np
import pytest

import mdinputs
import oracle
from gpu_helpers import TOL, dev, host, step_err

pytestmark = pytest.mark.gpu


def step(paths, csts, points, prec_solve):
    import torch

    import paper_2301_12659_amd as mdn

    b = mdn.Batch(paths)
    status = torch.zeros(len(paths), dtype=torch.int32, device="cuda")
    norms = torch.zeros(2 * len(paths), dtype=torch.float64, device="cuda")
    x = dev(b.pack_series(points))
    b.step(dev(b.pack_cff([s.cff for s in paths])), dev(b.pack_series(csts)), x, status, norms,
           mdn.workspace(b.workspace_bytes()), prec_solve=prec_solve)
    torch.cuda.synchronize()
    assert host(status).tolist() == [0] * len(paths)
    return b.unpack_series(host(x))


@pytest.mark.parametrize("L,prec_solve", [(2, None), (4, None), (4, 2)])
@pytest.mark.parametrize("top", [65, 90, 115, 120])
def test_tiles_of_mixed_orders(L, prec_solve, top):
    """62, 63 and 64 coefficients, whose tiles of the Jacobian are the largest,
    beside more coefficients in smaller tiles: bit for bit as alone, and the
    oracle's step."""
    paths = [mdinputs.tiny(L, 4, D - 1, mons=3, kmin=1, kmax=4, seed=D) for D in (62, 63, 64, top)]
    csts = [oracle.manufacture(s) for s in paths]
    points = []
    for s in paths:  # a point whose Jacobian series has all its coefficients
        x = s.xstar.copy()
        x[0] *= 1.25
        points.append(x)
    got = step(paths, csts, points, prec_solve)
    for s, c, x, y in zip(paths, csts, points, got):
        assert np.array_equal(y, step([s], [c], [x], prec_solve)[0]), s.D
        if prec_solve is None:
            ref = oracle.newton_step(s, s.cff, c, x)["x"]
            assert step_err(y, ref, x) <= TOL[L], s.D


@pytest.mark.parametrize("L,prec_solve", [(4, None), (4, 2)])
def test_more_large_paths_than_the_workspace_holds(L, prec_solve):
    """(more than two paths a compute unit, 256 MB in all)"""
    s = mdinputs.tiny(L, 20, 23, mons=3, kmin=1, kmax=3, seed=12)
    cst = oracle.manufacture(s)
    P = 540
    one = step([s], [cst], [s.start()], prec_solve)[0]
    for x in step([s] * P, [cst] * P, [s.start()] * P, prec_solve):
        assert step_err(x, one, s.start()) <= TOL[prec_solve or L]


@pytest.mark.parametrize("L,prec_solve", [(2, None), (4, None), (4, 2)])
@pytest.mark.parametrize("n,D", [(1, 1), (2, 16), (2, 17), (3, 10), (3, 11), (16, 8), (16, 9), (17, 8), (15, 5)])
def test_stages_in_one_block_and_in_several(L, prec_solve, n, D):
    s = mdinputs.tiny(L, n, D - 1, mons=3, kmin=1, kmax=min(n, 3), seed=D)
    cst = oracle.manufacture(s)
    x0 = s.start()
    x0[0] *= 1.0 + 2.0**-20
    ref = oracle.newton_step(s, s.cff, cst, x0)["x"]
    for P in (1, 300):  # a row's sums in several parts and in one
        got = step([s] * P, [cst] * P, [x0] * P, prec_solve)
        # (a solve in double doubles: its own error times the size of the update)
        tol = TOL[L] if prec_solve is None else TOL[2]
        for x in got[:: max(1, P // 3)]:
            assert step_err(x, ref, x0) <= tol
