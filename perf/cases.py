"""The work that a user of this package has it do, as cases that can be timed.

A case names a path through the public entry points and its sizes:

  newton    Newton steps at a series from x*(0) (``newton_step`` for one step,
            ``newton_steps`` for several)
  mixed     steps whose residual has L limbs and whose solve has Ls < L
  stagger   Newton's method with the staggered order schedule, to convergence
  complex   one Newton step on complex data
  batch     one step of many independent systems of uneven size
  train     forward and backward of a differentiable solve (gradient with
            respect to the monomial coefficients)
  eval      evaluation and differentiation alone
  column    a step on the one-column triangular system (row i is
            x_0 x_1 ... x_i) with its exponential solution
  refine    iterative refinement of a trial solution of the block Toeplitz
            system: its residual, the QR of A_0, the solve for the correction

Systems are those of the tests and the benchmark: random sparse supports with
a dominant linear term per row, damped solutions, starts at x*(0).  The
supports belong to the case (one system structure), the numbers to the seed.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2301_12659_amd as mdn


def listed():
    return [
        # the small double-double system: latency of a whole short solve
        _case("newton_small_dd", "newton", L=2, n=8, D=16, mons=8, kmin=3, kmax=3, emax=1, count=4),
        # the system of the headline measurement, pipelined steps to convergence
        _case("newton_medium_qd", "newton", L=4, n=64, D=64, mons=32, kmin=2, kmax=6, emax=2, count=6),
        # a single step at odd sizes: nothing is a multiple of a tile
        _case("newton_ragged_qd", "newton", L=4, n=77, D=51, mons=19, kmin=1, kmax=5, emax=3, count=1),
        # the largest configuration: octo doubles, the longest series
        _case("newton_large_od", "newton", L=8, n=128, D=128, mons=64, kmin=4, kmax=8, emax=3, count=1),
        # quad-double residual, double-double solve
        _case("mixed_medium_qd_dd", "mixed", L=4, Ls=2, n=64, D=64, mons=32, kmin=2, kmax=6, emax=2, count=7),
        # time to solution with the staggered orders (many short steps, the host looks at each)
        _case("stagger_medium_qd", "stagger", L=4, n=64, D=64, mons=32, kmin=2, kmax=6, emax=2),
        # complex data on the medium tables
        _case("complex_medium_qd", "complex", L=4, n=64, D=64, mons=32, kmin=2, kmax=6, emax=2),
        # many paths of uneven size, one step of each
        _case("batch_qd", "batch", L=4, Ls=4, paths=1024, nlo=16, nhi=96, mlo=8, mhi=32, kmin=2, kmax=5),
        # a training step: solve, loss on the last coefficients, adjoint, gradient
        _case("train_qd", "train", L=4, n=32, D=32, mons=32, kmin=3, kmax=5, emax=2, count=6),
        # evaluation and differentiation alone, octo doubles, ragged order
        _case("eval_ragged_od", "eval", L=8, n=30, D=41, mons=12, kmin=2, kmax=6, emax=3),
        # the triangular test system with its long monomials
        _case("column_od", "column", L=8, n=160, D=64),
        # residual, factorization and solve at a dimension past one tile
        _case("refine_dd", "refine", L=2, n=150, D=37),
    ]


def _case(name, kind, **sizes):
    return {"name": name, "kind": kind, **sizes}


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One case of the same paths, its sizes spread over the ranges in use."""
    kind = rng.choice(["newton", "newton", "newton", "mixed", "stagger", "complex", "batch", "train", "eval", "eval",
                       "column", "refine"])
    c = {"kind": kind}
    L = rng.choice([2, 4, 4, 8])
    if kind in ("newton", "mixed", "stagger", "complex", "train", "eval"):
        if kind == "train":
            L = rng.choice([2, 4])
        if kind == "mixed":
            L = rng.choice([4, 8])
        if kind == "newton" and rng.random() < 0.1:
            L = 1
        big = 96 if L == 8 else 128
        if kind in ("complex", "train", "stagger"):
            big //= 2
        n = _logint(rng, 4, big)
        D = _logint(rng, 2 if kind in ("newton", "eval") else 8, 24 if L == 1 else 96 if L == 8 else 128)
        kmin = rng.randint(1, 3)
        c.update(L=L, n=n, D=D, mons=_logint(rng, 3, 32), kmin=kmin, kmax=min(n, kmin + rng.randint(0, 4)),
                 emax=rng.randint(1, 2 if kind in ("complex", "stagger") else 3))
        c["kmin"] = min(c["kmin"], c["kmax"])
        if kind in ("newton", "mixed", "train"):
            c["count"] = rng.randint(1, 6)
        if kind == "mixed":
            c["Ls"] = rng.choice([2, 4]) if L == 8 else 2
    elif kind == "batch":
        L = rng.choice([2, 4])
        nlo = rng.randint(3, 32)
        c.update(L=L, Ls=2 if rng.random() < 0.4 else L, paths=_logint(rng, 40, 1000), nlo=nlo,
                 nhi=nlo + rng.randint(4, 60), mlo=rng.randint(3, 8), mhi=rng.randint(9, 32), kmin=2, kmax=5)
        c["kmin"] = min(c["kmin"], c["nlo"])
        c["kmax"] = min(c["kmax"], c["nlo"])
    elif kind == "column":
        c.update(L=L, n=_logint(rng, 16, 128 if L == 8 else 192), D=_logint(rng, 8, 64))
    else:
        c.update(L=L, n=_logint(rng, 5, 100 if L == 8 else 200), D=_logint(rng, 3, 64))
    return c


# ------------------------------------------------------------------ numbers


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _limbs(rng, lead, L):
    """Multiple doubles with the given leading limbs and random limbs below
    them, each within half a unit in the last place of the one above."""
    out = np.zeros((L,) + lead.shape)
    out[0] = lead
    for l in range(1, L):
        out[l] = rng.uniform(-0.5, 0.5, size=lead.shape) * np.where(out[l - 1] != 0.0, np.spacing(np.abs(out[l - 1])), 0.0)
    return out


def _damping(c):
    """Coefficient k of a solution is drawn in damping^k [0.5, 1.5]: powers of
    two, smaller for monomials of high degree."""
    return 0.125 if c.get("kmax", 2) * c.get("emax", 1) > 12 or c["L"] == 2 else 0.25


def _path_sizes(c):
    """[(n, D, monomials per polynomial)] of the case's systems."""
    if c["kind"] != "batch":
        return [(c["n"], c["D"], c["mons"])]
    rng = np.random.default_rng([c["paths"], c["nlo"], c["nhi"], c["mlo"], c["mhi"], 7])
    n = rng.integers(c["nlo"], c["nhi"] + 1, size=c["paths"])
    D = rng.choice([16, 32, 64], size=c["paths"])
    m = rng.integers(c["mlo"], c["mhi"] + 1, size=c["paths"])
    return [(int(a), int(b), int(q)) for a, b, q in zip(n, D, m)]


def _supports(c):
    """Supports of every monomial of every system, one row per monomial: the
    random ones of a polynomial, then its linear term.  Variables are sorted;
    a row's unused places hold -1 (exponent 0)."""
    sizes = _path_sizes(c)
    rng = np.random.default_rng([c["L"], sizes[0][0], sizes[0][1], sizes[0][2], len(sizes), c["kmin"], c["kmax"], 11])
    ns = np.array([s[0] for s in sizes])
    ms = np.array([s[2] for s in sizes])
    per = np.repeat(ms + 1, ns)  # monomials of every polynomial
    path = np.repeat(np.repeat(np.arange(len(sizes)), ns), per)
    row = np.repeat(np.concatenate([np.arange(n) for n in ns]), per)
    linear = np.zeros(len(path), bool)
    linear[np.cumsum(per) - 1] = True
    nn = ns[path]
    K = c["kmax"]
    k = np.minimum(rng.integers(c["kmin"], K + 1, size=len(path)), nn)
    var = np.full((len(path), K), -1, np.int64)
    todo = np.arange(len(path))
    place = np.arange(K)[None, :]
    while len(todo):
        v = np.floor(rng.random((len(todo), K)) * nn[todo, None]).astype(np.int64)
        v = np.sort(np.where(place < k[todo, None], v, 1 << 30), axis=1)
        var[todo] = v
        todo = todo[np.any((v[:, 1:] == v[:, :-1]) & (v[:, 1:] < (1 << 30)), axis=1)]
    var[var == 1 << 30] = -1
    k[linear] = 1
    var[linear] = -1
    var[linear, 0] = row[linear]
    ex = np.where(var >= 0, rng.integers(1, c.get("emax", 1) + 1, size=var.shape), 0)
    ex[linear, 0] = 1
    return SimpleNamespace(sizes=sizes, ns=ns, path=path, row=row, k=k, var=var, exp=ex, linear=linear)


def _columns(c):
    n = c["n"]
    place = np.arange(n)[None, :]
    row = np.arange(n)
    var = np.where(place <= row[:, None], place, -1)
    return SimpleNamespace(sizes=[(n, c["D"], 1)], ns=np.array([n]), path=np.zeros(n, np.int64), row=row, k=row + 1,
                           var=var, exp=(var >= 0).astype(np.int64), linear=np.zeros(n, bool))


def _mul(a, b):
    """Truncated products of the rows of a and b (series)."""
    D = a.shape[-1]
    out = a[..., :1] * b
    for i in range(1, D):
        out[..., i:] += a[..., i:i + 1] * b[..., :D - i]
    return out


def _powers(sup, X, rows, var0):
    """Factor x_v^e of every place of the monomials `rows`, [places][rows][D],
    ones where a place is unused; X [variables][D], var0 the first variable of
    a row's system in X."""
    D = X.shape[1]
    one = torch.zeros((1, D), dtype=X.dtype, device=X.device)
    one[0, 0] = 1.0
    Xe = torch.cat([X, one])
    var = torch.as_tensor(np.where(sup.var[rows] >= 0, sup.var[rows] + var0[:, None], X.shape[0]), device=X.device)
    ex = sup.exp[rows]
    out = []
    for a in range(var.shape[1]):
        f = Xe[var[:, a]]
        for e in range(1, int(ex[:, a].max(initial=0))):
            sel = torch.as_tensor(np.nonzero(ex[:, a] > e)[0], device=X.device)
            f[sel] = _mul(f[sel], Xe[var[sel, a]])
        out.append(f)
    return out


def _prod(factors):
    f = factors[0]
    for g in factors[1:]:
        f = _mul(f, g)
    return f


def _numbers(c, seed):
    """Everything of a case that is numbers, as numpy arrays, from the seed
    alone: cff [.., L, m], xstar, cst and x0 [.., L, n, D] (flat over the
    systems for a batch, a leading plane axis of 2 for complex data)."""
    rng = np.random.default_rng([seed, 20231])
    L = c["L"]
    dev = _device()
    if c["kind"] == "column":
        sup = _columns(c)
        n, D = c["n"], c["D"]
        alpha = np.where(rng.random(n) < 0.5, -1.0, 1.0) * np.round((1.0 - 0.25 * rng.random(n)) * 2 ** 20) / 2 ** 20
        S = np.cumsum(alpha)
        xs, b = np.ones((n, D)), np.ones((n, D))
        for q in range(1, D):
            xs[:, q] = xs[:, q - 1] * alpha / q
            b[:, q] = b[:, q - 1] * S / q
        cff = np.zeros((L, n))
        cff[0] = 1.0
        cst = _limbs(rng, -b, L)
        cst[1:, :, 0] = 0.0
        x0 = np.zeros((L, n, D))
        x0[0, :, 0] = 1.0
        return SimpleNamespace(sup=sup, cff=cff, cst=cst, x0=x0)
    sup = _supports(c)
    planes = 2 if c["kind"] == "complex" else 1
    nvar = int(sup.ns.sum())
    voff = np.concatenate([[0], np.cumsum(sup.ns)])[:-1]
    m = len(sup.row)
    damp = _damping(c)
    Ds = np.array([s[1] for s in sup.sizes])
    lead_c = rng.uniform(-1.0, 1.0, size=(planes, m))
    x_at0 = rng.uniform(0.5, 1.5, size=(planes, nvar))
    # the linear term dominates its row: twice the sum of the sizes of the
    # other derivatives at x*(0), rounded up to a power of two
    place = sup.var >= 0
    g = sup.path
    gv = np.where(place, sup.var + voff[g][:, None], 0)
    mag = np.where(place, np.sqrt((x_at0 ** 2).sum(axis=0))[gv] ** sup.exp, 1.0).prod(axis=1)
    size = np.abs(lead_c[0] + 1j * lead_c[-1] if planes == 2 else lead_c[0]) * mag * (sup.exp.sum(axis=1) / 0.5)
    polys = voff[g] + sup.row
    rowsum = np.bincount(polys[~sup.linear], weights=size[~sup.linear], minlength=nvar) + 1.0
    lead_c[0, sup.linear] = np.exp2(np.ceil(np.log2(2.0 * rowsum)))[polys[sup.linear]]
    lead_c[1:, sup.linear] = 0.0
    cff = np.stack([_limbs(rng, lead_c[p], L) for p in range(planes)])
    cff[:, 1:, sup.linear] = 0.0
    # the solution and the constant series that makes it one, system by order
    parts = {}
    for D in sorted(set(Ds.tolist())):
        which = np.nonzero(Ds == D)[0]
        vsel = np.concatenate([np.arange(voff[p], voff[p] + sup.ns[p]) for p in which])
        lead = rng.uniform(0.5, 1.5, size=(planes, len(vsel), D)) * damp ** np.arange(D)
        lead[:, :, 0] = x_at0[:, vsel]
        new = np.zeros(nvar, np.int64)
        new[vsel] = np.arange(len(vsel))
        rows = np.nonzero(Ds[g] == D)[0]
        z = torch.as_tensor(lead[0] + 1j * lead[1] if planes == 2 else lead[0], device=dev)
        w = torch.as_tensor(cff[0, 0, rows] + 1j * cff[1, 0, rows] if planes == 2 else cff[0, 0, rows], device=dev)
        val = _prod(_powers(sup, z, rows, new[voff[g[rows]]])) * w[:, None]
        # (the monomials of a polynomial are consecutive rows: sums in a fixed order)
        lengths = torch.as_tensor(np.bincount(new[polys[rows]], minlength=len(vsel)), device=dev)
        val = torch.view_as_real(val).reshape(len(rows), -1) if planes == 2 else val
        p = torch.segment_reduce(val.contiguous(), "sum", lengths=lengths, axis=0, unsafe=True)
        p = -p.cpu().numpy()
        p = p[:, 0::2] + 1j * p[:, 1::2] if planes == 2 else p
        lp = np.stack([p.real, p.imag]) if planes == 2 else p[None]
        xs = np.stack([_limbs(rng, lead[q], L) for q in range(planes)])
        cs = np.stack([_limbs(rng, lp[q], L) for q in range(planes)])
        parts[D] = (which, new, xs, cs)
    if c["kind"] == "batch":
        X = int((sup.ns * Ds).sum())
        xoff = np.concatenate([[0], np.cumsum(sup.ns * Ds)])[:-1]
        cst, x0 = np.zeros((L, X)), np.zeros((L, X))
        for D, (which, new, xs, cs) in parts.items():
            start = xs[0].copy()
            start[:, :, 1:] = 0.0
            for p in which:
                a, b = new[voff[p]], new[voff[p]] + sup.ns[p]
                sl = slice(xoff[p], xoff[p] + sup.ns[p] * D)
                cst[:, sl] = cs[0][:, a:b].reshape(L, -1)
                x0[:, sl] = start[:, a:b].reshape(L, -1)
        return SimpleNamespace(sup=sup, cff=cff[0], cst=cst, x0=x0)
    _, _, xs, cs = parts[c["D"]]
    x0 = xs.copy()
    x0[..., 1:] = 0.0
    if planes == 1:
        cff, cs, x0, xs = cff[0], cs[0], x0[0], xs[0]
    return SimpleNamespace(sup=sup, cff=cff, cst=cs, x0=x0, xstar=xs)


def _refine_numbers(c, seed):
    """A damped Jacobian series with a dominant diagonal at coefficient 0, a
    right-hand side and a trial solution: A [L, n, n, D], b and trial [L, n, D]."""
    g = torch.Generator().manual_seed(int(seed) * 7919 + 5)
    L, n, D = c["L"], c["n"], c["D"]
    damp = torch.pow(torch.tensor(0.25, dtype=torch.float64), torch.arange(D, dtype=torch.float64))

    def limbs(lead):
        out = [lead]
        for _ in range(1, L):
            ulp = torch.nextafter(out[-1].abs(), torch.tensor(math.inf, dtype=torch.float64)) - out[-1].abs()
            out.append((torch.rand(lead.shape, generator=g, dtype=torch.float64) - 0.5) * ulp)
        return torch.stack(out)

    u = lambda *s: 2.0 * torch.rand(s, generator=g, dtype=torch.float64) - 1.0  # noqa: E731
    A0 = u(n, n, D) * damp
    A0[torch.arange(n), torch.arange(n), 0] += 2.0 ** math.ceil(math.log2(n))
    return limbs(A0), limbs(u(n, D) * damp), limbs(u(n, D) * damp / n)


def _eval_point(xstar):
    """A series off the solution: its coefficients from 1 on halved."""
    x = xstar.copy()
    x[..., 1:] *= 0.5
    return x


# ------------------------------------------------------------------ states


def _plan_tables(sup, p=0):
    """(poly_ptr, mon_ptr, var, exp) of system p."""
    rows = np.nonzero(sup.path == p)[0] if len(sup.sizes) > 1 else np.arange(len(sup.row))
    v, e = sup.var[rows], sup.exp[rows]
    on = v >= 0
    mon = np.concatenate([[0], np.cumsum(on.sum(axis=1))])
    poly = np.concatenate([[0], np.cumsum(np.bincount(sup.row[rows], minlength=sup.ns[p]))])
    return poly.astype(np.int32), mon.astype(np.int32), v[on].astype(np.int32), e[on].astype(np.int32)


def prepare(case, seed):
    c = case
    kind, L = c["kind"], c["L"]
    dev = torch.device("cuda")
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)  # noqa: E731
    s = SimpleNamespace(c=c, status=torch.zeros(1, dtype=torch.int32, device=dev))
    if kind == "refine":
        s.A, s.b, s.trial = (a.to(dev) for a in _refine_numbers(c, seed))
        n, D = c["n"], c["D"]
        s.tau = torch.zeros((L, n), dtype=torch.float64, device=dev)
        s.r = torch.empty((L, n, D), dtype=torch.float64, device=dev)
        s.qr_ws = mdn.workspace(mdn.qr_workspace_bytes(L, n))
        s.ws = mdn.workspace(mdn.solve_workspace_bytes(L, n, D - 1))
        return s
    num = _numbers(c, seed)
    if kind == "batch":
        sizes = num.sup.sizes
        cuts = np.concatenate([[0], np.cumsum([n * (m + 1) for n, _, m in sizes])])
        systems = []
        for p, (n, D, _) in enumerate(sizes):
            sl = slice(cuts[p], cuts[p + 1])
            one = SimpleNamespace(sizes=[sizes[p]], ns=num.sup.ns[p:p + 1], row=num.sup.row[sl], var=num.sup.var[sl],
                                  exp=num.sup.exp[sl])
            pp, mp, v, e = _plan_tables(one)
            systems.append(SimpleNamespace(L=L, n=n, d=D - 1, poly_ptr=pp, mon_ptr=mp, var=v, exp=e))
        s.batch = mdn.Batch(systems, L)
        s.cff, s.cst, s.x0 = t(num.cff), t(num.cst), t(num.x0)
        s.x = s.x0.clone()
        s.status = torch.zeros(len(sizes), dtype=torch.int32, device=dev)
        s.norms = torch.zeros(2 * len(sizes), dtype=torch.float64, device=dev)
        s.ws = mdn.workspace(s.batch.workspace_bytes())
        return s
    n, D = c["n"], c["D"]
    s.plan = mdn.Plan(L, n, D - 1, *_plan_tables(num.sup))
    s.cff, s.cst, s.x0 = t(num.cff), t(num.cst), t(num.x0)
    if kind == "train":
        s.cff.requires_grad_(True)
        return s
    s.x = s.x0.clone()
    s.norms = torch.zeros((2, D), dtype=torch.float64, device=dev)
    s.ws = mdn.workspace(mdn.complex_workspace_bytes(s.plan) if kind == "complex" else s.plan.workspace_bytes())
    if kind == "eval":
        s.x = t(_eval_point(num.xstar))
        s.b = torch.empty((L, n, D), dtype=torch.float64, device=dev)
        s.A = torch.empty((L, n, n, D), dtype=torch.float64, device=dev)
    if kind == "stagger":
        # the start is known to half the working precision: x_0 from a few
        # steps at order 1, its trailing limbs dropped
        p0 = mdn.Plan(L, n, 0, *_plan_tables(num.sup))
        z = s.x0[:, :, :1].contiguous()
        mdn.newton_steps(p0, 4, s.cff, s.cst[:, :, :1].contiguous(), z, s.status, torch.zeros((2, 1), dtype=torch.float64, device=dev),
                         mdn.workspace(p0.workspace_bytes()))
        s.x0[:, :, :1] = z
        s.x0[(L + 1) // 2:] = 0.0
        s.tol = mdn.default_stagger_tol(L, c["kmax"])
    return s


# ------------------------------------------------------------------ passes


def run(state):
    s, c = state, state.c
    kind, L = c["kind"], c["L"]
    if kind == "eval":
        mdn.eval_diff(s.plan, s.cff, s.cst, s.x, s.b, s.A, s.ws)
        return {"b": s.b, "A": s.A}
    if kind == "refine":
        n, d = c["n"], c["D"] - 1
        mdn.linear_residual(L, n, d, s.A, s.b, s.trial, s.r)
        a0 = s.A[..., 0].contiguous()
        mdn.qr(L, n, a0, s.tau, s.status, s.qr_ws)
        dx = s.r.clone()
        mdn.series_solve(L, n, d, a0, s.tau, s.A, dx, s.ws, s.status)
        return {"r": s.r, "qr": a0, "tau": s.tau, "dx": dx, "status": s.status}
    if kind == "train":
        s.cff.grad = None
        x = mdn.newton_solve(s.cff, s.plan, s.cst, s.x0, c["count"])
        loss = mdn.top_coefficient_loss(x, _ktop(c))
        mdn.md_backward(loss)
        return {"x": x, "loss": loss, "grad": s.cff.grad}
    s.x.copy_(s.x0)
    if kind == "batch":
        s.batch.step(s.cff, s.cst, s.x, s.status, s.norms, s.ws, prec_solve=c["Ls"])
    elif kind == "complex":
        mdn.newton_step_complex(s.plan, s.cff, s.cst, s.x, s.status, s.norms, s.ws)
    elif kind == "mixed":
        for _ in range(c["count"]):
            mdn.newton_step_mixed(s.plan, c["Ls"], s.cff, s.cst, s.x, s.status, s.norms, s.ws)
    elif kind == "stagger":
        rep, _ = mdn.newton_staggered(s.plan, L, False, 40, s.tol, s.cff, s.cst, s.x, s.status, s.norms, s.ws)
        return {"x": s.x, "converged": int(rep.converged)}
    elif c.get("count", 1) == 1:
        mdn.newton_step(s.plan, s.cff, s.cst, s.x, s.status, s.norms, s.ws)
    else:
        mdn.newton_steps(s.plan, c["count"], s.cff, s.cst, s.x, s.status, s.norms, s.ws)
    return {"x": s.x, "status": s.status}


def _ktop(c):
    """First coefficient of the loss."""
    return max(0, c["D"] - 8)


# ------------------------------------------------------------------ what a pass cannot do without


def _products(sup, emax):
    """Series products of the evaluation and differentiation of every system:
    the prefix, suffix and cross products of the reverse mode (3k - 5 for k
    variables of exponent one), the common factors and the powers."""
    k = sup.k
    big = ((sup.exp >= 2) & (sup.var >= 0)).sum(axis=1)
    per = np.where(k >= 2, 3 * k - 3 - 2 * (big == 0), np.where(big > 0, 1, 0)) + np.maximum(big - 1, 0)
    if len(sup.sizes) == 1:
        return [int(np.maximum(per, 0).sum()) + sup.sizes[0][0] * max(emax - 2, 0)]
    return np.bincount(sup.path, weights=np.maximum(per, 0), minlength=len(sup.sizes)).tolist()


def _mul_flops(L):
    """Flops of a multiply-add of L-limb numbers that no scheme avoids: the
    L (L + 1) / 2 products of limbs that count and the rounding errors of
    the L (L - 1) / 2 leading ones, a fused multiply-add each."""
    return 2 * L * L


def work(case):
    c = case
    L, Ls = c["L"], c.get("Ls", c["L"])
    kind = c["kind"]
    if kind == "refine":
        n, D = c["n"], c["D"]
        ops = n * n * D * (D + 1) / 2 * 2 + 2 * n ** 3 / 3 + 2 * n * n * D
        return {"bytes": 8.0 * L * (n * n * D + 4 * n * D + 2 * n * n), "flops": ops * _mul_flops(L)}
    sup = _columns(c) if kind == "column" else _supports(c)
    flops = nbytes = 0.0
    prods = _products(sup, c.get("emax", 1))
    scale = 4.0 if kind == "complex" else 1.0
    planes = 2 if kind == "complex" else 1
    count = c.get("count", 6 if kind == "stagger" else 1)
    for (n, D, mons), pr in zip(sup.sizes, prods):
        ev = pr * D * (D + 1) / 2
        N = n * planes
        solve = 2 * n ** 3 / 3 * scale + n * n * D * scale + n * n * D * (D - 1) / 2 * scale
        m = n * (mons + 1) if kind != "column" else n
        nbytes += 8.0 * L * planes * (3 * n * D + m)
        if kind == "eval":
            flops += ev * _mul_flops(L)
            nbytes += 8.0 * L * n * n * D
        elif kind == "train":
            flops += (count + 1) * (ev + solve) * _mul_flops(L)
        else:
            flops += count * scale * ev * _mul_flops(Ls if Ls < L else L) + count * solve * _mul_flops(Ls)
            if Ls < L:  # the values once more at the residual's precision
                flops += count * ev / 3 * _mul_flops(L)
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits


def _eval64(sup, cff, cst, x):
    """b = -p(x) and A = p'(x) of one system, series as rows of doubles."""
    n, D = x.shape
    rows = np.arange(len(sup.row))
    var0 = np.zeros(len(rows), np.int64)
    F = _powers(sup, x, rows, var0)
    K = len(F)
    low = SimpleNamespace(var=np.where(sup.exp >= 2, sup.var, -1), exp=np.maximum(sup.exp - 1, 0))
    G = _powers(low, x, rows, var0)  # x^(e - 1)
    suf = [None] * (K + 1)
    for a in range(K - 1, 0, -1):
        suf[a] = F[a] if suf[a + 1] is None else _mul(F[a], suf[a + 1])
    A = torch.zeros((n * n, D), dtype=x.dtype, device=x.device)
    pre = torch.zeros_like(F[0])
    pre[:, 0] = cff
    for a in range(K):
        on = np.nonzero(sup.var[:, a] >= 0)[0]
        sel = torch.as_tensor(on, device=x.device)
        d = _mul(pre[sel], G[a][sel]) if sup.exp.max() > 1 else pre[sel]
        if suf[a + 1] is not None:
            d = _mul(d, suf[a + 1][sel])
        ex = torch.as_tensor(sup.exp[on, a], device=x.device)
        at = torch.as_tensor(sup.row[on] * n + sup.var[on, a], device=x.device)
        A.index_add_(0, at, d * ex[:, None])
        pre = _mul(pre, F[a])
    p = cst.clone()
    p.index_add_(0, torch.as_tensor(sup.row, device=x.device), pre)
    return -p, A.reshape(n, n, D)


def _toeplitz64(A, b):
    """dx of the block Toeplitz system (A [n, n, D], b [n, D]), on the CPU."""
    A, b = A.cpu(), b.cpu()
    n, D = b.shape
    Ak = A.permute(2, 0, 1).contiguous()
    lu, piv = torch.linalg.lu_factor(Ak[0])
    dx = torch.zeros((D, n, 1), dtype=b.dtype)
    for k in range(D):
        r = b[:, k:k + 1]
        if k:
            r = r - torch.bmm(Ak[1:k + 1], dx[:k].flip(0)).sum(dim=0)
        dx[k] = torch.linalg.lu_solve(lu, piv, r)
    return dx[..., 0].t().contiguous()


def _wide(v, L):
    out = torch.zeros((L,) + tuple(v.shape), dtype=torch.float64)
    out[0] = v.cpu()
    return out


def exact(case, seed):
    c = case
    kind, L = c["kind"], c["L"]
    if kind == "batch":
        return None
    if kind == "refine":
        A, b, trial = (a[0] for a in _refine_numbers(c, seed))
        n, D = b.shape
        Ak = A.permute(2, 0, 1).contiguous()
        r = b.clone()
        for k in range(D):
            r[:, k] -= torch.bmm(Ak[:k + 1], trial.t()[:k + 1].flip(0)[..., None]).sum(dim=0)[:, 0]
        q, tau = torch.geqrf(A[..., 0])
        q[-1, -1] = -q[-1, -1]  # the last column too gets its reflector (tau = 2)
        tau[-1] = 2.0
        return {"r": _wide(r, L), "qr": _wide(q, L), "tau": _wide(tau, L), "dx": _wide(_toeplitz64(A, r), L),
                "status": None}
    num = _numbers(c, seed)
    dev = _device()
    lead = (lambda a: torch.as_tensor(a[0, 0] + 1j * a[1, 0] if kind == "complex" else a[0], device=dev))
    cff, cst, x = lead(num.cff), lead(num.cst), lead(num.x0)
    if kind == "eval":
        b, A = _eval64(num.sup, cff, cst, lead(_eval_point(num.xstar)))
        return {"b": _wide(b, L), "A": _wide(A, L)}
    count = 10 if kind == "stagger" else c.get("count", 1)
    for _ in range(count):
        b, A = _eval64(num.sup, cff, cst, x)
        x = x + _toeplitz64(A, b).to(dev)
    if kind == "complex":
        return {"x": torch.stack([_wide(x.real, L), _wide(x.imag, L)]), "status": None}
    if kind == "stagger":
        return {"x": _wide(x, L), "converged": None}
    if kind != "train":
        return {"x": _wide(x, L), "status": None}
    # the adjoint: T^T lambda = dloss/dx, the same system with transposed
    # blocks and the coefficients in reverse, then the gradient by rows
    kt = _ktop(c)
    g = torch.zeros_like(x)
    g[:, kt:] = 2.0 * x[:, kt:]
    _, A = _eval64(num.sup, cff, cst, x)
    lam = _toeplitz64(A.permute(1, 0, 2), g.flip(1)).flip(1).to(dev)
    rows = np.arange(len(num.sup.row))
    val = _prod(_powers(num.sup, x, rows, np.zeros(len(rows), np.int64)))
    grad = -(lam[torch.as_tensor(num.sup.row, device=dev)] * val).sum(dim=1)
    loss = (x[:, kt:] ** 2).sum().reshape(())
    return {"x": _wide(x, L), "loss": _wide(loss, L), "grad": _wide(grad, L)}
