"""M = A_0^{-1} of the Newton step: the refinement from an inverse in doubles
and the factorization it falls back to, through one step on a dense linear
system A_0 x + c = 0 at degree 0 (the step from any point is the solution), at
the edges of the kernels' tiles, with matrices that need row exchanges, with
an ill conditioned one (factorized) and with a singular one."""
import numpy as np
import pytest

import mdinputs
import oracle
from gpu_helpers import TOL

pytestmark = pytest.mark.gpu


def linear_system(L, n, seed, spread=0.0):
    """p_i = sum_j A_ij x_j + c_i with the large entries of A on a cyclic shift
    of the diagonal (every pivot needs a row exchange); `spread`: decades
    between the largest and the smallest scale of the variables' solution
    directions (an ill conditioned A that row and column scaling do not mend)."""
    rng = np.random.default_rng([seed, n])
    A = mdinputs.random_md(rng, L, (n, n), -1.0, 1.0)
    if spread:
        u, _, vt = np.linalg.svd(A[0])
        A[0] = u @ np.diag(10.0 ** np.linspace(0.0, -spread, n)) @ vt
        for l in range(1, L):
            A[l] = rng.uniform(-1.0, 1.0, (n, n)) * 0.5 * np.spacing(np.abs(A[l - 1]))
    else:
        i = np.arange(n)
        A[:, i, (i + 1) % n] = 0.0
        A[0, i, (i + 1) % n] = 2.0 * n
    var = np.tile(np.arange(n, dtype=np.int32), n)
    s = mdinputs.System(f"linear_L{L}_n{n}", L, n, 0, (np.arange(n + 1) * n).astype(np.int32),
                        np.arange(n * n + 1, dtype=np.int32), var, np.ones(n * n, np.int32),
                        np.ascontiguousarray(A.reshape(L, n * n)), mdinputs.random_md(rng, L, (n, 1), 0.5, 1.5), seed)
    return s, mdinputs.random_md(rng, L, (n, 1), -1.0, 1.0)


def step(s, cst):
    import torch

    import paper_2301_12659_amd as mdn

    x0 = s.start()
    drv = mdn.Newton(s, cst, x0)
    drv.step()
    torch.cuda.synchronize()
    return drv.x.cpu().numpy(), drv.status_code(), x0


def error(s, cst, got, x0):
    ref = oracle.newton_step(s, s.cff, cst, x0)["x"]
    return float(oracle.absdiff(got, ref).max() / max(np.abs(x0[0]).max(), np.abs(ref[0]).max()))


@pytest.mark.parametrize("L", [2, 4, 8])
@pytest.mark.parametrize("n", [1, 2, 8, 9, 31, 33, 64, 65, 127, 129, 192, 193])
def test_step_on_a_linear_system(L, n):
    if L == 8 and n > 129:
        n = 150 if n == 192 else 193
    s, cst = linear_system(L, n, 3)
    got, status, x0 = step(s, cst)
    assert status == 0
    assert error(s, cst, got, x0) <= TOL[L]


@pytest.mark.parametrize("L,n", [(2, 20), (4, 40), (8, 12)])
def test_ill_conditioned(L, n):
    # cond about 1e13: no refinement from an inverse in doubles
    s, cst = linear_system(L, n, 5, spread=13.0)
    got, status, x0 = step(s, cst)
    assert status == 0
    assert error(s, cst, got, x0) <= TOL[L] * 1e13


@pytest.mark.parametrize("L,n", [(2, 9), (4, 64), (4, 70), (8, 5)])
def test_singular(L, n):
    import paper_2301_12659_amd as mdn

    s, cst = linear_system(L, n, 7)
    A = s.cff.reshape(L, n, n)
    A[:, n - 1, :] = A[:, 0, :]
    _, status, _ = step(s, cst)
    assert status == mdn.MD_ESINGULAR


@pytest.mark.parametrize("L", [2, 4])
def test_scales_that_the_factorization_refuses(L):
    """A diagonal entry below n 2^(-53 L) of the largest is reported singular,
    whatever the conditioning of the scaled matrix."""
    import paper_2301_12659_amd as mdn

    n = 6
    s, cst = linear_system(L, n, 9)
    A = s.cff.reshape(L, n, n)
    A[:] = 0.0
    A[0] = np.diag([1.0] * (n - 1) + [2.0 ** (-53 * L - 4)])
    _, status, _ = step(s, cst)
    assert status == mdn.MD_ESINGULAR
