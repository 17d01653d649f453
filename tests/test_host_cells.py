"""Size of the pair search's cell list (tests/host/cells_check.cpp) on the CPU
under UndefinedBehaviorSanitizer (host pass only)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_cell_index_fits_for_every_separation(tmp_path):
    exe = str(tmp_path / "cells_check")
    cmd = [HIPCC, "-std=c++17", "-O1", "-g", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-sanitize-recover=all", "-I", os.path.dirname(HERE), "-o", exe,
           os.path.join(HERE, "host", "cells_check.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "cell list checks passed" in r.stdout
