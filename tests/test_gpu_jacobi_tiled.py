"""The Jacobi launches that run several iterations each, against the oracle,
bit for bit: grids at the edges of one patch (64 x 128) and of the overlapping
patches, odd widths, and every remainder of the iterations per launch."""
import numpy as np
import pytest

from oracle import jacobi as oj
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRIDS = [(1, 1), (2, 3), (3, 128), (64, 128), (64, 129), (65, 128), (65, 127), (113, 225), (130, 257)]


@pytest.mark.parametrize("iters", [1, 2, 3, 8, 9, 17])
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "%dx%d" % g)
def test_bits_match_the_oracle(grid, iters):
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    n, m = grid
    u0 = np.random.default_rng([n, m, iters]).standard_normal((n, m))
    ref, change = oj.solve(u0, iters)
    u = torch.from_numpy(u0.copy()).cuda()
    work = torch.full_like(u, float("nan"))  # scratch: what it holds must not matter
    mc = torch.full((1,), -1.0, dtype=torch.float64, device="cuda")
    dn.jacobi(u, work, n, m, iters, mc)
    np.testing.assert_array_equal(u.cpu().numpy(), ref)
    assert mc.item() == change
