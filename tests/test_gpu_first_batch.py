"""The first-layer kernel past 2^23 workgroups (one 4x4 image each), where a
32-bit count of its threads would change sign: images from the whole batch
against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def test_more_than_two_to_the_23_images():
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    b, s = (1 << 23) + 9, 4
    p = synth.make_params(synth.Net("t", 1, s, s, [synth.conv(4, 3)]), 17)[0]
    d = dn.conv_desc(b, s, s, 1, 4, 3, 1, 1, 1, 0.1, 0, 0, dn.F32, 1.0, 1.0, 1.0, -1, 0, 1)
    wb, vb, wsb = dn.conv_sizes(d)
    assert wsb == 0
    w, bias, scale = G.empty_bytes(wb), G.empty_bytes(vb), G.empty_bytes(vb)
    dn.conv_pack(d, p.w, p.bias, p.mean, p.var, p.gamma, p.beta, 1e-5, w, bias, scale)
    x = torch.rand((b, 1, s, s), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    y = torch.full((b, s, s, 4), float("nan"), device="cuda")
    dn.conv2d(d, x, w, bias, scale, None, y, None, 0)
    torch.cuda.synchronize()
    pick = torch.tensor([0, 1, 4095, 1 << 22, (1 << 23) - 1, 1 << 23, (1 << 23) + 1, b - 1], device="cuda")
    xs = x[pick].double().cpu().numpy()
    ref = oracle.leaky(oracle.batchnorm(oracle.add_bias(oracle.conv2d(xs, p.w, 1, 1), p.bias), p.mean, p.var, p.gamma,
                                        p.beta, 1e-5), 0.1)
    assert G.rel_l2(y[pick].permute(0, 3, 1, 2).cpu().numpy(), ref) < G.GATE[dn.F32]
    assert not torch.isnan(y).any()
