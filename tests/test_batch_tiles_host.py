"""The LDS of the batched assembly (batch_tiles.hpp), compiled for the host:
paths of any two orders in one launch stay within it."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_tiles_of_mixed_orders_fit(tmp_path):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "batch_tiles_host_check")
    cmd = [HIPCC, "-x", "hip", "-O1", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", os.path.join(HERE, "batch_tiles_host_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    rows = [tuple(map(int, line.split())) for line in
            subprocess.run([exe], capture_output=True, text=True, timeout=120, check=True).stdout.splitlines()]
    assert len(rows) == 2 * 128 * 128
    assert [r for r in rows if r[3] >= r[4]] == []
    assert max(r[4] for r in rows) * 8 <= 64 * 1024  # (no attribute for larger LDS is asked for)
