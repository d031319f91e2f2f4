"""Input gradients through convs whose pool ran fused, at the shapes where the
one-kernel form of that backward (unpool + few-channel conv + image egress) has
edges: outputs that leave ragged 16 x 32 tiles, widths that are no multiple of
four, filters and paddings other than 3 and 1, one and several channel
segments, linear activations, and shapes past its limits, which take the
separate kernels.  The full-size gradient in front of the conv, which that
kernel only forms tile by tile, is still read back; the conv of that gradient
by the standalone entry point has to give the image's gradient bit for bit."""
import numpy as np
import pytest

import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# (in_c, cout, k, pad, act, h, w)
SHAPES = [
    (3, 16, 3, 1, 1, 32, 64),    # whole tiles
    (3, 16, 3, 1, 1, 34, 66),    # one row and two columns into new tiles; width % 4 != 0
    (1, 8, 3, 1, 0, 14, 30),     # one tile, linear, one BF16 segment
    (4, 16, 2, 1, 1, 17, 35),    # 2x2 filter: output one larger than the input
    (3, 24, 1, 0, 1, 18, 34),    # 1x1, three segments
    (16, 32, 3, 1, 1, 20, 36),   # sixteen channels out; past the FP32 limit
    (3, 16, 4, 0, 1, 21, 39),    # 4x4 unpadded
    (3, 40, 3, 1, 1, 16, 32),    # past the BF16 limit too
]


@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "c%d_co%d_k%d_p%d_a%d_%dx%d" % s)
def test_image_gradient_equals_the_conv_of_the_full_gradient(dtype, shape):
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    in_c, cout, k, pad, act, h, w = shape
    layers = [synth.Layer(synth.CONV, cout=cout, ksize=k, pad=pad, batchnorm=True, activation=act), synth.maxpool(2, 2)]
    net = synth.Net("t", in_c, h, w, layers)
    params = synth.make_params(net, 77)
    b = 2
    n = dn.Net(layers, in_c, h, w, b, dtype=dtype, leaky_slope=0.1, bn_eps=1e-5)
    n.load_params(params)
    nbytes = n.input_gradient_arena_bytes(1, b, h, w)
    arena = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")  # nothing may rest on its contents
    x = G.dev(synth.make_input(net, b, 78).astype(np.float32))
    grad = torch.full((b, in_c, h, w), float("nan"), device="cuda")
    n.input_gradient_arena(arena, nbytes, 1, x, b, h, w, grad)
    ho, wo = h + 2 * pad - k + 1, w + 2 * pad - k + 1
    full = torch.empty((b, cout, ho, wo), device="cuda")
    assert n.input_gradient_readback(arena, nbytes, 1, b, h, w, 0, 2, full, full.numel() * 4)
    codes = torch.empty((b, ho // 2, wo // 2, dn.channel_pad(dtype, cout)), dtype=torch.uint8, device="cuda")
    assert n.input_gradient_readback(arena, nbytes, 1, b, h, w, 1, 1, codes, codes.numel())
    torch.cuda.synchronize()
    # one element per window carries the gradient, the one its code names
    f = full.view(b, cout, ho // 2, 2, wo // 2, 2).permute(0, 2, 4, 1, 3, 5).reshape(b, ho // 2, wo // 2, cout, 4)
    at = codes[..., :cout].long()
    others = f.clone()
    others.scatter_(-1, at.unsqueeze(-1), 0.0)
    assert (others == 0).all() and (f.gather(-1, at.unsqueeze(-1)) != 0).float().mean() > 0.9
    # the same conv by the standalone entry point on that gradient
    d = dn.conv_desc(b, h, w, in_c, cout, k, 1, pad, act, 0.1, 0, 0, dtype)
    wb, vb, wsb = dn.conv_backward_sizes(d)
    wp, zb, us, ws = G.empty_bytes(wb), G.empty_bytes(vb), G.empty_bytes(vb), G.empty_bytes(wsb)
    p = params[0]
    dn.conv_pack_backward(d, p.w, p.mean, p.var, p.gamma, 1e-5, wp, zb, us)
    dy = G.to_storage(dn, dtype, full.cpu().numpy().astype(np.float64))
    dx = G.empty_bytes(G.nhwc_bytes(dn, dtype, b, in_c, h, w))
    dn.conv_backward_data(d, dy, wp, zb, us, 0, dx, ws, wsb)
    want = G.from_storage(dn, dtype, dx, b, in_c, h, w)
    np.testing.assert_array_equal(grad.cpu().numpy().astype(np.float64), want)
