"""The single-step H_K^(0) stencil reads nothing outside the lattice, whatever part of its 64 x 16 tiles lies past
it: the conditions of its loads over every size, tile and lane."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_single_step_stencil_loads_stay_in_the_lattice(tmp_path):
    gxx = shutil.which("g++")
    src = os.path.join(ROOT, "tests", "native", "stencil_rows_check.cpp")
    if gxx is None or not os.path.exists(src):
        pytest.skip("g++ or the native driver is not here")
    exe = tmp_path / "stencil_rows_check"
    cmd = [gxx, "-std=c++17", "-O2", "-Wall", "-Werror", "-I",
           os.path.join(ROOT, "paper_2211_10185_amd", "csrc"), src, "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and ", 0 failures" in r.stdout, r.stdout + r.stderr
