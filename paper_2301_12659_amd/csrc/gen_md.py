"""Generate straight-line multiple-double routines (md_gen.inc).

The paper's multiple-double code is generated (Section 1.2 and Section 6:
code generated by CAMPARY, inlined on numbers held in registers).  This script
generates our own routines for L = 2, 4 and 8 limbs (double double, quad
double, octo double) from one scheme, written from the published ideas of
error-free transformations (Knuth's TwoSum, Dekker's FastTwoSum, the
FMA-based TwoProd) and of level-by-level accumulation followed by
renormalization (Hida-Li-Bailey for quad doubles, Joldes-Muller-Popescu for
general expansions):

* every partial product a_p * b_q belongs to "level" p + q (magnitude about
  2^(-53(p+q)) relative to the leading product); its TwoProd error belongs to
  level p + q + 1;
* levels 0 .. L-2 are summed with TwoSum, each rounding error carried to the
  next level, so nothing is lost there; level L-1 is summed with plain
  additions and FMAs (errors below 2^(-53 L) are dropped);
* the L level sums are renormalized with one bottom-up TwoSum pass and one
  top-down TwoSum pass into a nonoverlapping expansion.

Each routine is emitted in static single assignment form so the compiler keeps
every value in a register (the paper stages operands through shared memory
into registers, Section 6).
"""
import sys


# FP64 instructions and flops (a fused multiply-add counts as two flops) of
# each emitted primitive.
COST = {"two_sum": (6, 6), "fast_two_sum": (3, 3), "two_prod": (2, 3), "add": (1, 1), "fma": (1, 2),
        "mul": (1, 1), "neg": (0, 0)}


class Emitter:
    def __init__(self):
        self.lines = []
        self.k = 0
        self.instr = 0
        self.flops = 0

    def _count(self, what):
        i, f = COST[what]
        self.instr += i
        self.flops += f

    def tmp(self):
        self.k += 1
        return f"t{self.k}"

    def emit(self, s):
        self.lines.append("    " + s)

    def two_sum(self, a, b):
        if a == "0.0":
            return b, "0.0"
        if b == "0.0":
            return a, "0.0"
        s, e = self.tmp(), self.tmp()
        self.emit(f"double {s}, {e}; two_sum({a}, {b}, {s}, {e});")
        self._count("two_sum")
        return s, e

    def fast_two_sum(self, a, b):
        if b == "0.0":
            return a, "0.0"
        if a == "0.0":
            return b, "0.0"
        s, e = self.tmp(), self.tmp()
        self.emit(f"double {s}, {e}; fast_two_sum({a}, {b}, {s}, {e});")
        self._count("fast_two_sum")
        return s, e

    def two_prod(self, a, b):
        p, e = self.tmp(), self.tmp()
        self.emit(f"double {p}, {e}; two_prod({a}, {b}, {p}, {e});")
        self._count("two_prod")
        return p, e

    def add(self, a, b):
        if a == "0.0":
            return b
        if b == "0.0":
            return a
        t = self.tmp()
        self.emit(f"const double {t} = {a} + {b};")
        self._count("add")
        return t

    def fma(self, a, b, c):
        t = self.tmp()
        if c == "0.0":
            self.emit(f"const double {t} = {a} * {b};")
            self._count("mul")
        else:
            self.emit(f"const double {t} = __builtin_fma({a}, {b}, {c});")
            self._count("fma")
        return t


def level_sums(E, L, terms, last_products):
    """terms[g]: names at level g (g < L); last_products: (x, y) pairs whose
    product belongs to level L-1.  Returns L level sums."""
    out = []
    carries = []
    for g in range(L):
        cur = [t for t in terms[g] + carries if t != "0.0"]
        carries = []
        if g < L - 1:
            if not cur:
                out.append("0.0")
                continue
            acc = cur[0]
            for t in cur[1:]:
                acc, c = E.two_sum(acc, t)
                if c != "0.0":
                    carries.append(c)
            out.append(acc)
        else:
            acc = "0.0"
            for t in cur:
                acc = E.add(acc, t)
            for (x, y) in last_products:
                acc = E.fma(x, y, acc)
            out.append(acc)
    return out


def renorm(E, u, L, first_dominant=False):
    """Renormalize level sums u[0..m-1] (m >= 1) into L limbs."""
    u = list(u)
    m = len(u)
    if m == 1:
        return u + ["0.0"] * (L - 1)
    # bottom-up pass
    e = [None] * m
    s = u[m - 1]
    for i in range(m - 2, -1, -1):
        if i == 0 and first_dominant:
            s, e[i + 1] = E.fast_two_sum(u[i], s)
        else:
            s, e[i + 1] = E.two_sum(u[i], s)
    e[0] = s
    if m == 2:
        r = [e[0], e[1]]
    else:
        # top-down pass; |e1| <= ulp(e0)/2 so the first step is a FastTwoSum
        r = []
        r0, eps = E.fast_two_sum(e[0], e[1])
        r.append(r0)
        for i in range(2, m):
            ri, eps = E.two_sum(eps, e[i])
            r.append(ri)
        r.append(eps)
    out = r[:L]
    while len(out) < L:
        out.append("0.0")
    tail = "0.0"
    for t in r[L:]:
        tail = E.add(tail, t)
    if tail != "0.0":
        out[L - 1] = E.add(out[L - 1], tail)
    return out


def product_terms(E, L, a, b, scalar_b=False):
    """Level lists of a*b (b a double when scalar_b)."""
    terms = [[] for _ in range(L)]
    last = []
    for p in range(L):
        qs = [0] if scalar_b else range(L)
        for q in qs:
            g = p + q
            bq = b if scalar_b else b[q]
            if g < L - 1:
                hi, lo = E.two_prod(a[p], bq)
                terms[g].append(hi)
                terms[g + 1].append(lo)
            elif g == L - 1:
                last.append((a[p], bq))
    return terms, last


def gen_add(L, sub=False):
    """a + b (or a - b) by level sums: the error is of the size 2^(-53 L)
    (|a| + |b|), the bound of a sum of terms, which is how the reductions,
    butterflies and assembly sums use it (several terms, error measured
    against their magnitudes).  add_acc is accurate relative to the result."""
    E = Emitter()
    a = [f"a[{i}]" for i in range(L)]
    b = [(f"-b[{i}]" if sub else f"b[{i}]") for i in range(L)]
    if sub:
        nb = []
        for i in range(L):
            t = E.tmp()
            E.emit(f"const double {t} = -b[{i}];")
            nb.append(t)
        b = nb
    terms = [[a[g], b[g]] for g in range(L)]
    u = level_sums(E, L, terms, [])
    r = renorm(E, u, L)
    return E, r


def level_sums_exact(E, L, terms):
    """Like level_sums, but levels 0 .. L-1 are all summed with TwoSum; the
    rounding errors of level L-1 form level L, which is summed with plain
    additions.  Returns L + 1 level sums."""
    out = []
    carries = []
    for g in range(L + 1):
        cur = [t for t in (terms[g] if g < L else []) + carries if t != "0.0"]
        carries = []
        if g < L:
            if not cur:
                out.append("0.0")
                continue
            acc = cur[0]
            for t in cur[1:]:
                acc, c = E.two_sum(acc, t)
                if c != "0.0":
                    carries.append(c)
            out.append(acc)
        else:
            acc = "0.0"
            for t in cur:
                acc = E.add(acc, t)
            out.append(acc)
    return out


def renorm_all(E, u):
    """One bottom-up and one top-down TwoSum pass over u[0..m-1] (m >= 2),
    keeping all m + 1 outputs: an error-free transformation."""
    m = len(u)
    e = [None] * m
    s = u[m - 1]
    for i in range(m - 2, -1, -1):
        s, e[i + 1] = E.two_sum(u[i], s)
    e[0] = s
    r = []
    r0, eps = E.two_sum(e[0], e[1])
    r.append(r0)
    for i in range(2, m):
        ri, eps = E.two_sum(eps, e[i])
        r.append(ri)
    r.append(eps)
    return r


def gen_add_acc(L, sub=False):
    """a + b (or a - b) accurate relative to the result, also when the
    leading limbs cancel.  The level sums of add drop the rounding errors of
    their last level, which are of the size 2^(-53 L) |a|, so a sum that
    cancels to much less than |a| loses its relative accuracy.  Here every
    level 0 .. L-1 is summed with TwoSum and only the rounding errors of the
    last level's TwoSums are added plainly; where leading limbs cancel,
    Sterbenz's lemma makes their sum exact and the carries that reach the last
    level vanish.  Cancellation moves significant bits to lower levels, so
    the level sums are renormalized twice: once keeping every term, then into
    L limbs.  (Checked against exact rationals with engineered cancellation
    at every depth: relative error below 2^(-53 L) of the result.)"""
    E = Emitter()
    a = [f"a[{i}]" for i in range(L)]
    if sub:
        b = []
        for i in range(L):
            t = E.tmp()
            E.emit(f"const double {t} = -b[{i}];")
            b.append(t)
    else:
        b = [f"b[{i}]" for i in range(L)]
    if L == 1:  # one rounded addition is the correctly rounded sum
        return E, [E.add(a[0], b[0])]
    terms = [[a[g], b[g]] for g in range(L)]
    u = level_sums_exact(E, L, terms)
    r = renorm(E, renorm_all(E, u), L)
    return E, r


def gen_mul(L):
    E = Emitter()
    a = [f"a[{i}]" for i in range(L)]
    b = [f"b[{i}]" for i in range(L)]
    terms, last = product_terms(E, L, a, b)
    u = level_sums(E, L, terms, last)
    r = renorm(E, u, L, first_dominant=True)
    return E, r


def gen_mul_d(L):
    E = Emitter()
    a = [f"a[{i}]" for i in range(L)]
    terms, last = product_terms(E, L, a, "d", scalar_b=True)
    u = level_sums(E, L, terms, last)
    r = renorm(E, u, L, first_dominant=True)
    return E, r


def gen_fma(L, negate=False):
    """c := c + a*b (or c - a*b)."""
    E = Emitter()
    a = [f"a[{i}]" for i in range(L)]
    if negate:
        b = []
        for i in range(L):
            t = E.tmp()
            E.emit(f"const double {t} = -b[{i}];")
            b.append(t)
    else:
        b = [f"b[{i}]" for i in range(L)]
    terms, last = product_terms(E, L, a, b)
    for g in range(L):
        terms[g].insert(0, f"c[{g}]")
    u = level_sums(E, L, terms, last)
    r = renorm(E, u, L)
    return E, r


def gen_fma_lazy(L):
    """u := u + a*b on level sums u[0..L-1] (no renormalization): the
    accumulator of a dot product, renormalized once at its end."""
    E = Emitter()
    a = [f"a[{i}]" for i in range(L)]
    b = [f"b[{i}]" for i in range(L)]
    terms, last = product_terms(E, L, a, b)
    for g in range(L):
        terms[g].insert(0, f"u[{g}]")
    u = level_sums(E, L, terms, last)
    return E, u


def gen_fma_lazy_h(L):
    """fma_lazy with an operand a of L - 1 limbs (a's products of level L - 1
    and above with b's L limbs included)."""
    E = Emitter()
    a = [f"a[{i}]" for i in range(L - 1)]
    b = [f"b[{i}]" for i in range(L)]
    terms, last = [[] for _ in range(L)], []
    for p in range(L - 1):
        for q in range(L - p):
            if p + q < L - 1:
                hi, lo = E.two_prod(a[p], b[q])
                terms[p + q].append(hi)
                terms[p + q + 1].append(lo)
            else:
                last.append((a[p], b[q]))
    for g in range(L):
        terms[g].insert(0, f"u[{g}]")
    return E, level_sums(E, L, terms, last)


def gen_add_lazy(L):
    """u := u + w for two accumulators of level sums (no renormalization):
    the step of a reduction tree over lazily accumulated partial sums."""
    E = Emitter()
    terms = [[f"u[{g}]", f"w[{g}]"] for g in range(L)]
    u = level_sums(E, L, terms, [])
    return E, u


def gen_renorm(L):
    """Renormalize L level sums x[0..L-1] into L limbs."""
    E = Emitter()
    u = [f"x[{i}]" for i in range(L)]
    r = renorm(E, u, L)
    return E, r


def gen_renorm_extra(L):
    """Renormalize L+1 level-ordered terms x[0..L] into L limbs."""
    E = Emitter()
    u = [f"x[{i}]" for i in range(L + 1)]
    r = renorm(E, u, L)
    return E, r


def body(E, r, outname, L):
    lines = list(E.lines)
    for i in range(L):
        lines.append(f"    {outname}[{i}] = {r[i]};")
    return "\n".join(lines)


def generate(counts=None):
    out = []
    out.append("// GENERATED by gen_md.py -- do not edit by hand.")
    out.append("// Multiple-double routines for L = 1, 2, 4, 8 limbs (see gen_md.py for the scheme; one limb is")
    out.append("// plain double arithmetic, the paper's D precision).")
    out.append("")
    # 3, 5 and 9 limbs: what a residual with one limb beyond a precision's
    # own takes (the refinement of the inverse of A_0)
    for L in (1, 2, 3, 4, 5, 8, 9):
        out.append(f"template <> struct MD<{L}> {{")
        out.append(f"  static constexpr int L = {L};")
        defs = [
            ("add", "const double (&a)[L], const double (&b)[L], double (&r)[L]", gen_add(L), "r"),
            ("sub", "const double (&a)[L], const double (&b)[L], double (&r)[L]", gen_add(L, sub=True), "r"),
            ("add_acc", "const double (&a)[L], const double (&b)[L], double (&r)[L]", gen_add_acc(L), "r"),
            ("sub_acc", "const double (&a)[L], const double (&b)[L], double (&r)[L]", gen_add_acc(L, sub=True), "r"),
            ("mul", "const double (&a)[L], const double (&b)[L], double (&r)[L]", gen_mul(L), "r"),
            ("mul_d", "const double (&a)[L], const double d, double (&r)[L]", gen_mul_d(L), "r"),
            ("fma", "double (&c)[L], const double (&a)[L], const double (&b)[L]", gen_fma(L), "c"),
            ("fms", "double (&c)[L], const double (&a)[L], const double (&b)[L]", gen_fma(L, negate=True), "c"),
            ("renorm_extra", "const double (&x)[L + 1], double (&r)[L]", gen_renorm_extra(L), "r"),
            ("fma_lazy", "double (&u)[L], const double (&a)[L], const double (&b)[L]", gen_fma_lazy(L), "u"),
            ("add_lazy", "double (&u)[L], const double (&w)[L]", gen_add_lazy(L), "u"),
            ("renorm", "const double (&x)[L], double (&r)[L]", gen_renorm(L), "r"),
        ]
        if L in (3, 5, 9):
            defs = [d for d in defs if d[0] in ("add", "add_lazy", "renorm")]
            defs.append(("fma_lazy_h", "double (&u)[L], const double (&a)[L - 1], const double (&b)[L]",
                         gen_fma_lazy_h(L), "u"))
        for name, sig, (E, r), outname in defs:
            if counts is not None:
                counts.setdefault(str(L), {})[name] = {"instr": E.instr, "flops": E.flops}
            out.append(f"  static MD_INLINE void {name}({sig}) {{")
            out.append(body(E, r, outname, L))
            out.append("  }")
        out.append("};")
        out.append("")
    return "\n".join(out) + "\n"


if __name__ == "__main__":
    import json
    import os

    counts = {}
    text = generate(counts)
    path = sys.argv[1] if len(sys.argv) > 1 else "md_gen.inc"
    with open(path, "w") as f:
        f.write(text)
    # FP64 instruction and flop counts per routine, used to express
    # multiple-double operation counts as double flops
    with open(os.path.join(os.path.dirname(os.path.abspath(path)), "md_counts.json"), "w") as f:
        json.dump(counts, f, indent=1, sort_keys=True)
