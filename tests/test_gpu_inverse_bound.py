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
