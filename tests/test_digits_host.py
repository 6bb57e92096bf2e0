"""Digits of multiple doubles (digits.hpp), compiled for the host: dot products
against exact rationals."""
import math
import os
import shutil
import subprocess
from fractions import Fraction

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    path = str(tmp_path_factory.mktemp("digits") / "digits_host_check")
    cmd = [HIPCC, "-x", "hip", "-O2", "-ffp-contract=off", "-fno-fast-math", "--offload-arch=gfx950",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           os.path.join(HERE, "digits_host_check.cpp"), "-o", path]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return subprocess.run([path], capture_output=True, text=True, timeout=120, check=True).stdout.splitlines()


def test_dot_products(lines):
    """Within one unit of the precision, 2^(-53 L), of the sum of the sizes of
    the terms, whatever their range."""
    checked = 0
    for line in lines:
        p = line.split()
        if p[0] == "nonfinite":
            continue
        L, n = int(p[0]), int(p[1])
        v = [Fraction(float.fromhex(x)) for x in p[3:]]
        md = lambda q: sum(v[q * L:(q + 1) * L])
        terms = [md(2 * i) * md(2 * i + 1) for i in range(n)]
        err = abs(md(2 * n) - sum(terms)) / sum(abs(t) for t in terms)
        assert err <= Fraction(1, 2 ** (53 * L)), (L, n, p[2], math.log2(err))
        checked += 1
    assert checked == 360


def test_nonfinite(lines):
    assert "nonfinite 1" in lines
