"""md_newton_steps beyond one column a lane, and where A_0 goes to the
factorization: the iterates of as many calls of md_newton_step, bit for bit; the
staged solve's workgroups for two coefficients each (many coefficients)."""
import numpy as np
import pytest

import mdinputs
import oracle
from gpu_helpers import TOL, dev, host, step_err
from test_gpu_inverse import linear_system

pytestmark = pytest.mark.gpu


def compare(s, cst, count):
    import torch

    import paper_2301_12659_amd as mdn

    one, many = mdn.Newton(s, cst), mdn.Newton(s, cst)
    for _ in range(count):
        one.step()
    many.steps(count)
    torch.cuda.synchronize()
    assert one.status_code() == many.status_code() == 0
    assert np.array_equal(host(many.x), host(one.x))
    assert np.array_equal(host(many.norms), host(one.norms))
    return host(one.x)


@pytest.mark.parametrize("L,n", [(2, 1), (2, 8), (2, 16), (2, 17), (2, 65), (2, 128), (2, 129), (2, 150), (2, 192), (2, 193),
                                 (4, 8), (4, 9), (4, 65), (4, 128), (4, 129), (4, 192)])
@pytest.mark.parametrize("count", [2, 5])
def test_bit_identical(L, n, count):
    s = mdinputs.tiny(L, n, 5, mons=3, kmin=1, kmax=min(n, 4), seed=n)
    cst = oracle.manufacture(s)
    got = compare(s, cst, count)
    if count == 5:  # converged (six coefficients take three steps)
        assert step_err(got, s.xstar, s.start()) <= TOL[L]


@pytest.mark.parametrize("L,n", [(2, 6), (2, 16), (2, 40), (2, 70), (4, 8), (4, 33), (4, 100)])
@pytest.mark.parametrize("spread", [11.5, 13.0])
def test_bit_identical_where_factorized(L, n, spread):
    s, _ = linear_system(L, n, 5, spread=spread)
    s.d = 3
    s.xstar = mdinputs.random_md(np.random.default_rng(n), L, (n, 4), 0.5, 1.5)
    compare(s, mdinputs.random_constant(s, 1), 3)


@pytest.mark.parametrize("L,n,D", [(2, 128, 71), (2, 128, 72), (2, 128, 128), (2, 192, 46), (2, 192, 47), (2, 192, 88),
                                   (2, 192, 89), (4, 65, 128), (4, 128, 73), (4, 128, 128)])
def test_solve_with_many_coefficients(L, n, D):
    """The residual of the solution of the block Toeplitz system."""
    import torch

    import paper_2301_12659_amd as mdn

    rng = np.random.default_rng([L, n, D])
    A = mdinputs.random_md(rng, L, (n, n, D), -1.0, 1.0)
    i = np.arange(n)
    A[0, i, i, 0] += 2.0 * n
    A *= np.ldexp(1.0, -2 * np.arange(D))  # damped: the solution's coefficients stay in range
    b = mdinputs.random_md(rng, L, (n, D), -1.0, 1.0) * np.ldexp(1.0, -2 * np.arange(D))
    tA, tb = dev(A), dev(b)
    a0 = tA[..., 0].clone(memory_format=torch.contiguous_format)
    tau = torch.zeros((L, n), dtype=torch.float64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    mdn.qr(L, n, a0, tau, status)
    dx = tb.clone()
    mdn.series_solve(L, n, D - 1, a0, tau, tA, dx, mdn.workspace(mdn.solve_workspace_bytes(L, n, D - 1)), status)
    r = torch.empty_like(tb)
    mdn.linear_residual(L, n, D - 1, tA, tb, dx, r)
    torch.cuda.synchronize()
    assert int(status) == 0
    x, size = np.abs(host(dx)[0]), np.abs(b[0])
    for k in range(D):
        for j in range(k + 1):
            size[:, k] += np.abs(A[0, :, :, j]) @ x[:, k - j]
    assert float((np.abs(host(r)[0]) / size).max()) <= TOL[L]


@pytest.mark.parametrize("L,mons", [(2, 1007), (2, 1009), (4, 1009)])  # 65 (mons + 1) monomials: about 64 x 1024
def test_bit_identical_with_many_monomials(L, mons):
    s = mdinputs.make_system("many", L, 65, 1, mons, 1, 3, (1,), 3, None, boost=True, damping=0.25, boost_gamma=2.0,
                             vectorized=True)
    compare(s, mdinputs.random_constant(s, 1), 3)
