"""The pair emission also zeroes the tiles' ranges: its grid has to be wide enough
for them where there are few pairs and many tiles (CPU; the launch is recorded,
not made)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_emission_grid(tmp_path):
    out = str(tmp_path / "libemit_grid.so")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                        "-Wno-unused-result", "-Wno-unused-value", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "host", "emit_grid_host_test.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    # pairs; words: ranges of one small frame up to those of 32 views of 2048 x 2048, tiles of 8
    cases = [(p, w) for p in (0, 1, 1024, 1025, 5000, 4_000_000) for w in (0, 256, 4096, 4097, 1 << 20, 32 << 17)]
    code = (f"import ctypes as C; f = C.CDLL({out!r}).lgs_emit_grid; f.argtypes = [C.c_int64] * 2; "
            f"raise SystemExit(sum(f(p, w) for p, w in {cases!r}))")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
