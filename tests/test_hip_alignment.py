"""The HIP sources promise no more alignment than a caller's buffer has: no access
through a vector type goes by a function or template that drops the type's
declared alignment (the compiler's -Walign-mismatch, as an error)."""
import os
from concurrent.futures import ThreadPoolExecutor
import subprocess

import pytest

import paper_2201_00613_amd.build as build


def test_no_access_assumes_more_alignment_than_declared():
    if not os.path.exists(build.hipcc()):
        pytest.skip("hipcc not available")

    def check(src):
        cmd = [build.hipcc(), *build._common_flags(), "--cuda-device-only", "-fsyntax-only", "-Werror=align-mismatch",
               os.path.join(build.CSRC, src)]
        return src, subprocess.run(cmd, capture_output=True, text=True)

    with ThreadPoolExecutor(4) as ex:
        for src, res in ex.map(check, build.SOURCES):
            assert res.returncode == 0, (src, res.stderr[-3000:])
