"""Native check of the library's limits, on the CPU: the launch shape of the edge
gradients (tests/native/edge_grid_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")
CSRC = os.path.join(ROOT, "paper_2208_00001_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.mark.parametrize("check", ["edge_grid_check"])
def test_native_check(check, tmp_path):
    exe = str(tmp_path / check)
    subprocess.run(["g++", "-O2", "-Wall", "-I", CSRC, "-o", exe, os.path.join(NATIVE, check + ".cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout
