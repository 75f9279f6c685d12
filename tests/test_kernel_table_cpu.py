"""Every pass kernel of a size, those of the energy measurement among them, gets its dynamic-LDS limit: the walk
over the kernel table that sets it, on a table of distinct entries."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_walk_over_the_kernel_table_is_complete(tmp_path):
    gxx = shutil.which("g++")
    src = os.path.join(ROOT, "tests", "native", "kernel_table_check.cpp")
    if gxx is None or not os.path.exists(src):
        pytest.skip("g++ or the native driver is not here")
    exe = tmp_path / "kernel_table_check"
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-I",
           os.path.join(ROOT, "paper_2211_10185_amd", "csrc"), src, "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and ", 0 failures" in r.stdout, r.stdout + r.stderr
