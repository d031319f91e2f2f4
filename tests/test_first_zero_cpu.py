"""Host check of the counter clearing in the first-layer kernel: the statement
that stores the zeros (conv_direct.hip) is compiled for the host and run for
the workgroups of grids up to the largest that a launch takes.  Every word is
cleared once, and no workgroup writes past the words, before them, or at all
where there is nothing to clear.  No GPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = os.path.join(ROOT, "tests", "native", "first_zero_check.cpp")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_only_the_words_are_cleared(tmp_path):
    src = open(os.path.join(ROOT, "paper_1811_03882_amd", "csrc", "conv_direct.hip")).read()
    stores = re.findall(r"^ *[^\n]*a\.zero\[[^\n]*\n", src, flags=re.M)
    assert len(stores) == 1
    (tmp_path / "first_zero.h").write_text(stores[0])
    exe = tmp_path / "first_zero_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", str(tmp_path), DRIVER, "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0, out.stdout
