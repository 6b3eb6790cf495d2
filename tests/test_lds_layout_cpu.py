"""LDS objects that are read or written by wider types than their own (CPU: hipcc
cross-compiles gfx950 here): they have to be declared with the wider access's
alignment, and where words are cleared that are then counted in halves, a fence
has to keep the two in order, since distinct types may not alias.  Looked up in
the code as written, before any optimisation (which may raise alignments by
itself)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_16144_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")


def _ir(src, tmp_path):
    out = str(tmp_path / "out.ll")
    subprocess.run([HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes", "--cuda-device-only",
                    "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, src), "-o", out], check=True,
                   capture_output=True)
    return open(out).read()


@pytest.mark.parametrize("src,objects", [
    ("binning.hip", ["k_small_front.*1S"]),
    ("radix_sort.hip", ["k_scatter.*3cnt"]),
    ("raster.hip", ["lds_f", "lds_z"]),
    ("decoder.hip", ["k_decoderI.*2f[AT]", "k_decoderI.*2rC", "k_decoderI.*3dfr"]),
])
def test_wide_accesses_are_aligned(src, objects, tmp_path):
    ir = _ir(src, tmp_path)
    for o in objects:
        got = re.findall(r"^@(\S*%s\S*) = .*addrspace\(3\) global .*, align (\d+)$" % o, ir, re.M)
        assert got, o
        assert all(int(a) % 16 == 0 for _, a in got), got


def test_cleared_words_come_before_counted_halves(tmp_path):
    ir = _ir("radix_sort.hip", tmp_path)
    bodies = [b for b in re.findall(r"^define .*?^}", ir, re.M | re.S)
              if "k_scatter" in b.split("{", 1)[0] and "amdgcn.wave.barrier" in b]   # (those that count)
    assert len(bodies) >= 3
    for b in bodies:
        assert 'fence syncscope("wavefront") acq_rel' in b
