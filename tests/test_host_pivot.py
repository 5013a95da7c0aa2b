"""The square root and quotients of a Cholesky pivot, compiled for the host,
against sqrt and division over the range that the source states."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="ROCm compiler not found")
@pytest.mark.timeout(300)
def test_pivot_arithmetic(tmp_path):
    exe = str(tmp_path / "pivot")
    r = subprocess.run(
        [HIPCC, "-O2", "-std=c++17", "--offload-arch=gfx950", "-x", "hip", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"),
         "-I", os.path.join(ROOT, "paper_2511_06600_amd", "csrc"),
         os.path.join(ROOT, "tests", "host_pivot_check.cpp"), "-o", exe],
        capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=200)
    assert r.returncode == 0, r.stderr[-2000:]
    print(r.stdout)
    v = {k: int(x) for k, x in re.findall(r"(\w+) (\d+)", r.stdout)}
    assert v["pivots"] == 4000000
    assert v["root_off"] == 0           # the root is sqrt's, to the bit
    assert v["inv_ulps"] <= 1
    assert v["div_ulps"] <= 1           # a quotient is the division's or next to it
