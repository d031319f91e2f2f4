"""Jacobi launches at the sizes where the plan takes each form, against the
oracle, bit for bit: the whole grid and the last iteration's change."""
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
