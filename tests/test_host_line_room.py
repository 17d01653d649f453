"""LDS room of one line (csrc/pgx_fft.hpp), checked by the compiler: FP32 lines
that are transformed in FP64 (64 points) are held twice as long, every other
line, FP64 grids' among them, at its own length plus padding."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
@pytest.mark.parametrize("typ,size", [("float", 4), ("double", 8)])
def test_line_room_by_type(typ, size):
    body = "#include \"../paper_1705_03464_amd/csrc/pgx_fft.hpp\"\n"
    for n in (64, 128, 256, 512, 1024):
        own = n + n // 16 + 1
        body += f"static_assert(sizeof(pgx::C<{typ}>) == {2 * size}, \"\");\n"
        body += f"static_assert(pgx::lds_line_elems<{n}, {typ}>() == {2 * own if (n, size) == (64, 4) else own}, \"\");\n"
    cmd = ["g++", "-std=c++20", "-fsyntax-only", "-I", os.path.join(HERE, "host", "emu"), "-I", HERE, "-x", "c++", "-"]
    r = subprocess.run(cmd, input=body, capture_output=True, text=True, timeout=120, cwd=HERE)
    assert r.returncode == 0, r.stderr[-3000:]
