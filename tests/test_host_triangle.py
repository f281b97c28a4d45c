"""The packing of V+- as upper triangles and as the rows of streaming steps, and the reads of the
contractions over them, replayed on the CPU through the index functions that the kernels call
(tests/native/triangle_check.cpp), under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.slow


def test_triangle_replay(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "triangle_check")
    r = subprocess.run([cxx, "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                        "-I", os.path.join(ROOT, "paper_2603_20912_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "triangle_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "triangle checks: 0 of" in r.stdout, (r.stdout + r.stderr)[-4000:]
