"""The tables of the multi-step kernels (tiles bit-sliced across subtrees, a block
per lane, bit rows) on the CPU: a host program built from the kernels' own headers
runs the first two word by word through the kernels' memory layout and compares
every step their ring covers with brute force (tests/host/check_run_tables.hip)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_run_tables_give_every_covered_step():
    hipcc = shutil.which("hipcc") or ("/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else None)
    if not hipcc:
        pytest.skip("hipcc not available")
    out = os.path.join(ROOT, "_build", "host")
    os.makedirs(out, exist_ok=True)
    exe = os.path.join(out, "check_run_tables")
    csrc = os.path.join(ROOT, "paper_2201_00613_amd", "csrc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-O2", "-D_GLIBCXX_ASSERTIONS",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "host", "check_run_tables.hip"), os.path.join(csrc, "host_tables.cpp"),
                    "-o", exe], check=True, capture_output=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert "all checks passed" in res.stdout, res.stdout[-2000:]
