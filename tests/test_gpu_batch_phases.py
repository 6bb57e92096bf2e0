"""The batched step's launches over all paths: sizes at the edges of their
tiles in one batch, matrices that the refinement leaves to the factorization,
and more paths than the workspace holds at once."""
import numpy as np
import pytest

import mdinputs
import oracle
from gpu_helpers import TOL, dev, host, step_err
from test_gpu_inverse import linear_system

pytestmark = pytest.mark.gpu


def step(paths, csts, prec_solve=None):
    import torch

    import paper_2301_12659_amd as mdn

    b = mdn.Batch(paths)
    status = torch.zeros(len(paths), dtype=torch.int32, device="cuda")
    norms = torch.zeros(2 * len(paths), dtype=torch.float64, device="cuda")
    x = dev(b.pack_series([s.start() for s in paths]))
    b.step(dev(b.pack_cff([s.cff for s in paths])), dev(b.pack_series(csts)), x, status, norms,
           mdn.workspace(b.workspace_bytes()), prec_solve=prec_solve)
    torch.cuda.synchronize()
    return b.unpack_series(host(x)), host(status).tolist()


@pytest.mark.parametrize("L", [2, 4])
def test_sizes_in_one_batch(L):
    sizes = [(1, 2), (2, 8), (3, 9), (5, 16), (8, 17), (9, 32), (32, 5), (33, 4), (4, 33), (64, 3), (65, 6), (3, 65),
             (128, 2), (5, 128)]
    paths = [mdinputs.tiny(L, n, D - 1, mons=3, kmin=1, kmax=min(n, 4), seed=7 * n + D) for n, D in sizes]
    csts = [oracle.manufacture(s) for s in paths]
    got, status = step(paths, csts)
    assert status == [0] * len(paths)
    for s, c, x in zip(paths, csts, got):
        ref = oracle.newton_step(s, s.cff, c, s.start())["x"]
        assert step_err(x, ref, s.start()) <= TOL[L], (s.n, s.D)


@pytest.mark.parametrize("L", [2, 4])
def test_paths_that_need_the_factorization(L):
    import paper_2301_12659_amd as mdn

    made = [linear_system(L, 9, 3), linear_system(L, 12, 5, spread=13.0), linear_system(L, 9, 7)]
    A = made[2][0].cff.reshape(L, 9, 9)
    A[:, 8, :] = A[:, 0, :]
    got, status = step([s for s, _ in made], [c for _, c in made])
    assert status == [0, 0, mdn.MD_ESINGULAR]
    for (s, c), x, tol in zip(made[:2], got, (TOL[L], TOL[L] * 1e13)):
        ref = oracle.newton_step(s, s.cff, c, s.start())["x"]
        assert float(oracle.absdiff(x, ref).max() / max(np.abs(s.start()[0]).max(), np.abs(ref[0]).max())) <= tol


@pytest.mark.parametrize("L,prec_solve", [(2, None), (4, 2)])
def test_more_paths_than_the_workspace_holds(L, prec_solve):
    s = mdinputs.tiny(L, 3, 6, mons=3, kmin=1, kmax=3, seed=11)
    cst = oracle.manufacture(s)
    one, _ = step([s], [cst], prec_solve)
    got, status = step([s] * 1100, [cst] * 1100, prec_solve)
    assert status == [0] * 1100
    for x in got:
        assert step_err(x, one[0], s.start()) <= TOL[prec_solve or L]
