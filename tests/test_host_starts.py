"""Range starts of sorted keys (csrc/pgx_starts.hpp) on the CPU under
AddressSanitizer and UndefinedBehaviorSanitizer (tests/host/starts_check.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_range_starts_on_the_cpu(tmp_path):
    exe = str(tmp_path / "starts_check")
    cmd = ["g++", "-std=c++20", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(HERE, "host", "emu"), "-o", exe, os.path.join(HERE, "host", "starts_check.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "range start checks passed" in r.stdout
