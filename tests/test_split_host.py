"""The three-way bf16 split of fp32 convolutions (csrc/split3.h) on the CPU:
exact over its range, and the six products that are kept within the stated
bound, at the operands that reach it too."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_split_and_products(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "split_test")
    cmd = [cxx, "-std=c++17", "-O2", "-Wall", "-fno-fast-math", f"-I{os.path.join(ROOT, 'paper_2112_10603_amd', 'csrc')}",
           os.path.join(ROOT, "tests", "native", "split_test.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]
    assert "all passed" in r.stdout
    print(r.stdout)
