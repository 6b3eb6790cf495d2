"""The workspace pool where device memory is short (CPU): tests/host/
pool_host_test.hip models a card's memory under the runtime's own allocation
code.  A call that fits has to be taken: without the pool's rounding, in blocks
of their own where no block holds a stage's buffers, with fewer feature groups
side by side; and a request that was met in the end leaves no error behind."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_short_memory(tmp_path):
    from paper_2511_16144_amd import binding as B
    if not os.path.exists(B.LIB_PATH):
        pytest.skip("the library is not built")
    out = str(tmp_path / "libpool_host_test.so")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                        "-Wno-unused-result", "-Wno-unused-value", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "host", "pool_host_test.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    # (the built library answers for the kernels' launchers, none of which is called)
    code = (f"import ctypes as C; C.CDLL({B.LIB_PATH!r}, mode=C.RTLD_GLOBAL); "
            f"raise SystemExit(C.CDLL({out!r}).lgs_pool_selftest())")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
