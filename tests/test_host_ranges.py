"""The shared point ranges of the x-direction passes (csrc/pgx_ranges.hpp) on
the CPU, one thread per lane (tests/host/ranges_check.cpp), under
AddressSanitizer and UndefinedBehaviorSanitizer: totals beyond 2^31, as a
catalogue of 2^31 - 1 pairs makes them when one group of lines reads each
point several times."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_point_ranges_on_the_cpu(tmp_path):
    exe = str(tmp_path / "ranges_check")
    cmd = ["g++", "-std=c++20", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(HERE, "host", "emu"), "-o", exe, os.path.join(HERE, "host", "ranges_check.cpp"),
           "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "point range checks passed" in r.stdout
