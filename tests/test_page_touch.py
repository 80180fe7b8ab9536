"""The pages of an output array are touched ahead of the copy into it without a change to what it holds, so
that a state export that fails half way leaves its later arrays as they were."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("extra", [0, 8, 4096 * 3 + 24])
def test_touch_keeps_the_contents(tmp_path, extra):
    cxx = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("g++")) if c and os.path.exists(c)), None)
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "touch")
    subprocess.run([cxx, "-O2", "-std=c++17", "-Wall", "-x", "c++", "-pthread", "-I", os.path.join(ROOT, "paper_1710_05155_amd", "csrc"),
                    os.path.join(ROOT, "tests", "page_touch.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, str(extra)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
