"""Matrices A_0 about the conditioning from which the factorization replaces the
refinement (rows of one matrix may take either way to stop): the step's error
stays with the conditioning, alone and in a batch."""
import pytest

from gpu_helpers import dev, host
from test_gpu_inverse import error, linear_system, step

pytestmark = pytest.mark.gpu


def bound(L, n, spread):
    """The working precision times the conditioning and the n terms of a sum, a
    few units of the last place each (16)."""
    return 16.0 * n * 10.0**spread * 2.0 ** (-53 * L)


@pytest.mark.parametrize("L,n", [(2, 7), (2, 16), (2, 40), (4, 8), (4, 64), (4, 100), (8, 33)])
@pytest.mark.parametrize("spread", [8.0, 10.5, 11.5, 12.0, 12.5])
def test_step(L, n, spread):
    s, cst = linear_system(L, n, 6, spread=spread)
    got, status, x0 = step(s, cst)
    assert status == 0
    assert error(s, cst, got, x0) <= bound(L, n, spread)


@pytest.mark.parametrize("L", [2, 4])
def test_batch(L):
    import torch

    import paper_2301_12659_amd as mdn

    spreads = [0.0, 8.0, 10.5, 11.5, 12.0, 12.5] * 2
    made = [linear_system(L, n, 6, spread=e) for e, n in zip(spreads, [12] * 6 + [70] * 6)]
    paths = [s for s, _ in made]
    b = mdn.Batch(paths)
    status = torch.zeros(len(paths), dtype=torch.int32, device="cuda")
    norms = torch.zeros(2 * len(paths), dtype=torch.float64, device="cuda")
    x = dev(b.pack_series([s.start() for s in paths]))
    b.step(dev(b.pack_cff([s.cff for s in paths])), dev(b.pack_series([c for _, c in made])), x, status, norms,
           mdn.workspace(b.workspace_bytes()))
    torch.cuda.synchronize()
    assert host(status).tolist() == [0] * len(paths)
    for (s, c), y, e in zip(made, b.unpack_series(host(x)), spreads):
        assert error(s, c, y, s.start()) <= bound(L, s.n, e), (s.n, e)


# (sizes whose M is refined: a factorization's errors grow with the scales)
@pytest.mark.parametrize("L,n", [(2, 5), (2, 16), (2, 40), (2, 100), (4, 8), (4, 30), (4, 100), (8, 20), (8, 130)])
@pytest.mark.parametrize("rows,columns", [(50, 0), (0, 50), (-45, 38), (20, 20)])
def test_scales_of_rows_and_columns(L, n, rows, columns):
    """Powers of two in the rows and columns of a well conditioned matrix: the
    solution is that of the matrix without them, times the columns' scales."""
    import numpy as np
    import torch

    import oracle
    import paper_2301_12659_amd as mdn

    s, cst = linear_system(L, n, 8)
    rng = np.random.default_rng(n)
    r = np.ldexp(1.0, rng.integers(0, abs(rows) + 1, n) * np.sign(rows))
    c = np.ldexp(1.0, rng.integers(0, abs(columns) + 1, n) * np.sign(columns))
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
