"""Max pools of windows of two at the edges of their input: sides of one,
windows cut at one or both edges, strides that skip input, and values of -inf,
which must win only where a window holds nothing else."""
import numpy as np
import pytest

import oracle
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp8"])
@pytest.mark.parametrize("h,w,stride", [(1, 1, 1), (1, 7, 1), (6, 1, 2), (5, 8, 3), (13, 13, 1), (9, 10, 2)])
def test_windows_of_two(dtype, h, w, stride):
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    x = synth.make_tensor((3, 20, h, w), 12, w, -2.0, -0.5)
    if dtype != dn.FP8:  # no infinities in that type
        x[:, :, : (h + 1) // 2, : (w + 1) // 2] = -np.inf
    xb = G.to_storage(dn, dtype, x)
    xs = G.from_storage(dn, dtype, xb, *x.shape)  # values the storage type holds
    ho, wo = (h - 1) // stride + 1, (w - 1) // stride + 1
    y = G.empty_bytes(G.nhwc_bytes(dn, dtype, 3, 20, ho, wo))
    dn.maxpool(3, h, w, 20, 2, stride, dtype, xb, y)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(G.from_storage(dn, dtype, y, 3, 20, ho, wo), oracle.maxpool(xs, 2, stride))
