"""Host check of the plan that splits Jacobi iterations over launches: compiled
for the host and run over grids from a point to the tallest the tiled kernel
takes (thin ones and 24000 x 24000 among them) and iteration counts from one
on.  Every launch runs at least one iteration and fits the kernel, and the
iterations add up.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1811_03882_amd", "csrc")
DRIVER = os.path.join(ROOT, "tests", "native", "jacobi_plan_check.cpp")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_launches_fit_and_add_up(tmp_path):
    exe = tmp_path / "jacobi_plan_check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, DRIVER, "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0, out.stdout
