"""The refinement of a row ends where its residuals reach their rounding errors,
whatever the number of limbs: well conditioned matrices, rows and columns times
powers of two that leave them below the bound of the refinement, give the
solution of the matrix without them.  (The factorization's errors grow with the
scales, so that a row which does not end shows.)"""
import numpy as np
import pytest

import oracle
from gpu_helpers import host
from test_gpu_inverse import linear_system
from test_gpu_inverse_bound import bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n", [(2, 5), (2, 16), (2, 40), (2, 100), (4, 8), (4, 30), (4, 100), (8, 20), (8, 66),
                                 (8, 100), (8, 130)])
@pytest.mark.parametrize("seed", range(4))
def test_scales_below_the_bound(L, n, seed):
    import torch

    import paper_2301_12659_amd as mdn

    s, cst = linear_system(L, n, 8)
    rng = np.random.default_rng(100 * n + seed)
    r = np.ldexp(1.0, rng.integers(0, 13, n))
    c = np.ldexp(1.0, rng.integers(0, 13, n))
    x0 = s.start()
    plain = mdn.Newton(s, cst, x0)
    plain.step()
    A = s.cff.reshape(L, n, n)
    A *= r[None, :, None] * c[None, None, :]
    scaled = mdn.Newton(s, cst * r[None, :, None], x0 / c[None, :, None])
    scaled.step()
    torch.cuda.synchronize()
    assert plain.status_code() == scaled.status_code() == 0
    x, y = host(plain.x), host(scaled.x) * c[None, :, None]
    # x0 + dx with dx = M b; b and M within the bound of their sizes
    size = np.abs(x0[0]).max() + np.abs(x[0]).max()
    assert float(oracle.absdiff(y, x).max()) <= bound(L, n, 0.0) * size
