"""QR, M = R^{-1} Q^T and the staged solve of A(t) dx(t) = b(t) at the edges of
their kernels' sizes: the residual of the solution."""
import numpy as np
import pytest

import mdinputs
import oracle
from gpu_helpers import TOL, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n", [(L, n) for L in (2, 4) for n in (1, 2, 8, 9, 16, 17, 63, 64, 65, 77, 127, 128, 129, 191, 192, 193)] +
                         [(1, 7), (1, 16), (8, 5), (8, 64), (8, 65), (8, 129)])
@pytest.mark.parametrize("D", [1, 2, 11, 27])
def test_residual_of_the_solution(L, n, D):
    import torch

    import paper_2301_12659_amd as mdn

    rng = np.random.default_rng([L, n, D])
    A = mdinputs.random_md(rng, L, (n, n, D), -1.0, 1.0)
    i = np.arange(n)
    A[0, i, i, 0] += 2.0 * n  # the sums of a row's other terms stay below it
    A[:, :, :, 1:] *= 0.25
    b = mdinputs.random_md(rng, L, (n, D), -1.0, 1.0)
    tA, tb = dev(np.ascontiguousarray(A)), dev(np.ascontiguousarray(b))
    a0 = tA[..., 0].clone(memory_format=torch.contiguous_format)  # (factorized in place)
    tau = torch.zeros((L, n), dtype=torch.float64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    mdn.qr(L, n, a0, tau, status)
    dx = tb.clone()
    ws = mdn.workspace(mdn.solve_workspace_bytes(L, n, D - 1))
    mdn.series_solve(L, n, D - 1, a0, tau, tA, dx, ws, status)
    r = torch.empty_like(tb)
    mdn.linear_residual(L, n, D - 1, tA, tb, dx, r)
    torch.cuda.synchronize()
    assert int(status) == 0
    x = np.abs(host(dx)[0])
    size = np.abs(b[0])
    for k in range(D):
        for j in range(k + 1):
            size[:, k] += np.abs(A[0, :, :, j]) @ x[:, k - j]
    assert float((np.abs(host(r)[0]) / size).max()) <= TOL[L]


@pytest.mark.parametrize("L,n", [(1, 6), (2, 1), (2, 33), (4, 16), (4, 65), (8, 9)])
@pytest.mark.parametrize("cond", [1, 2.0**44])
def test_adjoint_from_the_matrix(L, n, cond):
    """The adjoint solve from A_0 (by refinement, or factorized where A_0 is ill
    conditioned) against the one from its factors."""
    import torch

    import paper_2301_12659_amd as mdn

    D = 6
    rng = np.random.default_rng([L, n])
    A = mdinputs.random_md(rng, L, (n, n, D), -1.0, 1.0)
    i = np.arange(n)
    A[0, i, i, 0] += 2.0 * n
    if n > 1:
        A[:, 0, :, 0] /= cond  # a row of A_0 far below the others
    tA = dev(np.ascontiguousarray(A))
    g = mdinputs.random_md(rng, L, (n, D), -1.0, 1.0)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    tau = torch.zeros((L, n), dtype=torch.float64, device="cuda")
    a0 = tA[..., 0].clone(memory_format=torch.contiguous_format)
    one, two = dev(g), dev(g)
    mdn._adjoint_solve_a0(L, n, D - 1, a0, tau, tA, one, status)
    a0 = tA[..., 0].clone(memory_format=torch.contiguous_format)
    mdn.qr(L, n, a0, tau, status)
    mdn.adjoint_solve(L, n, D - 1, a0, tau, tA, two, mdn.workspace(mdn.adjoint_workspace_bytes(L, n, D - 1)), status)
    torch.cuda.synchronize()
    assert int(status) == 0
    x, y = host(one), host(two)
    # every stage may carry the conditioning of A_0 once more
    bound = TOL[L] * (float(cond) if n > 1 else 1.0) ** 2
    assert float((oracle.absdiff(x, y) / np.maximum(np.abs(y[0]).max(axis=0), 1e-300)).max()) <= bound
