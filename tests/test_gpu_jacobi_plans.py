"""Jacobi launches at the sizes where the plan takes each form, against the
oracle, bit for bit: the whole grid and the last iteration's change."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import jacobi as oj
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def check(n, m, iters):
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    u0 = np.random.default_rng([n, m, iters]).random((n, m))
    ref, change = oj.solve(u0, iters)
    u = torch.from_numpy(u0).cuda()
    work = torch.full_like(u, float("nan"))  # scratch: what it holds must not matter
    mc = torch.full((1,), -1.0, dtype=torch.float64, device="cuda")
    dn.jacobi(u, work, n, m, iters, mc)
    np.testing.assert_array_equal(u.cpu().numpy(), ref)
    assert mc.item() == change


def test_large_grid_with_an_odd_count_of_iterations():
    """One iteration per launch pays on a grid this large, and three launches
    end in the partner buffer."""
    check(160350, 497, 3)


# rows per wave that the plan takes, with several patches each way where not in place
@pytest.mark.parametrize("n,m,iters,rows", [
    (130, 257, 17, 4), (300, 300, 64, 8), (1000, 1500, 17, 12), (1000, 1500, 64, 12), (1200, 1500, 33, 16),
    (30, 128, 17, 4), (64, 128, 17, 8), (96, 100, 17, 12), (97, 128, 17, 16), (128, 128, 17, 16),
])
def test_every_patch_height(n, m, iters, rows, tmp_path):
    plan_rows = _plan_rows(tmp_path, n, m, iters)
    if plan_rows is not None:
        assert plan_rows == rows  # else this case does not test what it says
    check(n, m, iters)


def _plan_rows(tmp_path, n, m, iters):
    if shutil.which("g++") is None:
        return None
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text('#include <cstdio>\n#include "jacobi_plan.h"\n'
                   'int main() { std::printf("%%d", dnk::jacobi_plan(%d, %d, %d).rows); }\n' % (n, m, iters))
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(root, "paper_1811_03882_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    return int(subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout)


def test_bands_of_a_large_grid_from_its_start():
    """4096 x 4096 on 16-row waves: rows after nine iterations, from the
    initial grid's rows around them."""
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    n, iters = 4096, 9
    u0 = np.random.default_rng([n, iters]).random((n, n))
    u = torch.from_numpy(u0).cuda()
    dn.jacobi(u, torch.empty_like(u), n, n, iters)
    got = u.cpu().numpy()
    for r in (0, 1, 100, 117, 127, 128, 1000, 2047, 4000, 4094, 4095):
        lo, hi = max(0, r - iters), min(n, r + iters + 1)
        band, _ = oj.solve(u0[lo:hi], iters)  # the band's own edge rows stay: wrong from there on, a row an iteration
        np.testing.assert_array_equal(got[r], band[r - lo])
