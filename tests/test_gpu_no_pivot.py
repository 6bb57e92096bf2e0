"""A_0 without a pivot in a later panel of the elimination (a column of zeros):
reported singular by every caller of the inverse in doubles, those that go on
in the same launch among them."""
import numpy as np
import pytest

import mdinputs
from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


def system(L, n, column):
    """A system whose polynomials do not depend on one variable."""
    s = mdinputs.tiny(L, n, 3, mons=3, kmin=1, kmax=3, exps=(1, 2), seed=n)
    for j in range(s.m):
        if column in s.var[s.mon_ptr[j]:s.mon_ptr[j + 1]]:
            s.cff[:, j] = 0.0
    return s, mdinputs.random_constant(s, 1)


# (double double up to 16 variables and quad double up to 8: M in one launch)
@pytest.mark.parametrize("L,n,column", [(2, 9, 8), (2, 12, 8), (2, 12, 11), (2, 16, 8), (2, 16, 13), (4, 8, 5),
                                        (4, 9, 8), (2, 17, 16), (2, 33, 32), (4, 64, 40), (2, 70, 69), (4, 128, 127),
                                        (8, 20, 11)])
def test_single_and_pipelined_steps(L, n, column):
    import torch

    import paper_2301_12659_amd as mdn

    s, cst = system(L, n, column)
    one, many = mdn.Newton(s, cst), mdn.Newton(s, cst)
    one.step()
    many.steps(3)
    torch.cuda.synchronize()
    assert one.status_code() == mdn.MD_ESINGULAR
    assert many.status_code() == mdn.MD_ESINGULAR


@pytest.mark.parametrize("L", [2, 4])
def test_batch(L):
    import torch

    import paper_2301_12659_amd as mdn

    made = [system(L, n, c) for n, c in ((9, 8), (16, 12), (17, 16), (40, 33), (70, 64), (128, 127))]
    regular = mdinputs.tiny(L, 9, 3, mons=3, kmin=1, kmax=3, seed=9)
    made.append((regular, mdinputs.random_constant(regular, 1)))
    paths = [s for s, _ in made]
    b = mdn.Batch(paths)
    status = torch.zeros(len(paths), dtype=torch.int32, device="cuda")
    norms = torch.zeros(2 * len(paths), dtype=torch.float64, device="cuda")
    x = dev(b.pack_series([s.start() for s in paths]))
    b.step(dev(b.pack_cff([s.cff for s in paths])), dev(b.pack_series([c for _, c in made])), x, status, norms,
           mdn.workspace(b.workspace_bytes()))
    torch.cuda.synchronize()
    assert host(status).tolist() == [mdn.MD_ESINGULAR] * (len(paths) - 1) + [0]
