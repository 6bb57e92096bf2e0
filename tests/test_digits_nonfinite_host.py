"""Digits of values that are not finite (digits.hpp), compiled for the host: a
sum of products is a not-a-number exactly where double arithmetic makes it one."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_sums_of_two_products(tmp_path):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "digits_nonfinite_host_check")
    cmd = [HIPCC, "-x", "hip", "-O2", "-ffp-contract=off", "-fno-fast-math", "--offload-arch=gfx950",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           os.path.join(HERE, "digits_nonfinite_host_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = subprocess.run([exe], capture_output=True, text=True, timeout=120, check=True).stdout.splitlines()
    assert len(lines) == 4 * 4 * 5 * 5
    for line in lines:
        kinds, got = line.split()
        # (a digit form holds no infinity: every value that is not finite becomes a
        # not-a-number; an entry outside the series counts for nothing)
        terms = [t for t in (kinds[:2], kinds[2:]) if "m" not in t]
        assert int(got) == int(any(c in "ni" for t in terms for c in t)), line
