"""Launch plans (how a run of many steps is cut into launches) on the CPU, under
AddressSanitizer and UndefinedBehaviorSanitizer (tests/host/check_plans.cpp)."""
import os
import subprocess

from test_host_sanitizers import OUT, ROOT, SAN, _need_gcc


def test_launch_plans_under_sanitizers():
    _need_gcc()
    os.makedirs(OUT, exist_ok=True)
    exe = os.path.join(OUT, "check_plans")
    csrc = os.path.join(ROOT, "paper_2201_00613_amd", "csrc")
    subprocess.run(["g++", *SAN, "-std=c++17", "-Wall", "-Wextra", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "host", "check_plans.cpp"), os.path.join(csrc, "host_tables.cpp"),
                    "-o", exe], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=600,
                         env=dict(os.environ, ASAN_OPTIONS="abort_on_error=1", UBSAN_OPTIONS="print_stacktrace=1"))
    assert res.returncode == 0, (res.stdout + res.stderr)[-4000:]
    assert "all checks passed" in res.stdout
