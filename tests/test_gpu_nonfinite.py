"""Values that are not finite in the evaluation: every coefficient that one of
them enters, if only times a zero, is a not-a-number, at every precision."""
import numpy as np
import pytest

import mdinputs
from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu

N = 4


def product(a, b):
    return np.array([np.sum(a[:s + 1] * b[s::-1]) for s in range(len(a))])


def reference(s, x):
    """Values and derivatives in doubles, every term of every product formed:
    b [n][D] without the constant, A [n][n][D]."""
    D = x.shape[1]
    b, A = np.zeros((N, D)), np.zeros((N, N, D))
    for i in range(N):
        for j in range(s.poly_ptr[i], s.poly_ptr[i + 1]):
            q = range(s.mon_ptr[j], s.mon_ptr[j + 1])
            var, exp, c = [s.var[t] for t in q], [s.exp[t] for t in q], s.cff[0, j]
            common = None
            for v, e in zip(var, exp):
                for _ in range(e - 1):
                    common = x[v] if common is None else product(common, x[v])
            f = None if common is None else c * common  # (None: the scalar c)
            back = [None] * (len(var) + 1)  # back[t]: the product of the last t variables
            for t in range(1, len(var)):
                back[t] = x[var[-t]] if t == 1 else product(back[t - 1], x[var[-t]])
            for t, (v, e) in enumerate(zip(var, exp)):
                rest = back[len(var) - 1 - t]
                one = c * np.eye(1, D)[0] if f is None else f
                if rest is not None:
                    one = c * rest if f is None else product(f, rest)
                A[i, v] += e * one
                f = c * x[v] if f is None else product(f, x[v])
            b[i] += f
    return b, A


@pytest.mark.parametrize("L,D", [(2, 12), (4, 33), (8, 12), (8, 17), (8, 40), (8, 128)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_eval_diff(L, D, value):
    import torch

    import paper_2301_12659_amd as mdn

    s = mdinputs.tiny(L, N, D - 1, mons=4, kmin=1, kmax=4, exps=(1, 2, 3), seed=D)
    x = mdinputs.random_point(s, 3)
    x[:, 2, 1:] = 0.0
    x[:, 3] = 0.0
    x[:, 1, 5] = 0.0
    x[0, 1, 5] = value
    plan = mdn.Plan.from_system(s)
    b = torch.empty((L, N, D), dtype=torch.float64, device="cuda")
    A = torch.empty((L, N, N, D), dtype=torch.float64, device="cuda")
    mdn.eval_diff(plan, dev(s.cff), dev(mdinputs.random_constant(s, 2)), dev(x), b, A, mdn.workspace(plan.workspace_bytes()))
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        rb, rA = reference(s, x[0])
    assert not np.isfinite(rb).all() and not np.isfinite(rA).all()
    assert np.array_equal(np.isfinite(host(b)[0]), np.isfinite(rb))
    assert np.array_equal(np.isfinite(host(A)[0]), np.isfinite(rA))
