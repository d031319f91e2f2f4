"""The persistent halo kernel's instances with the window's layout built in
(BF16, 3x3, stride 1, 16 and 32 channels in) against the register-staged GEMM
tile: the same 16x16 MFMA steps in the same order, so the same bits.

Sizes at the edges of their 32-pixel-wide tiles and of the transfers' tests:
images narrower than a tile, one column into the next, one to two rows into
the next, no padding and padding that reaches two pixels past the image, more
images than workgroups per die (positions step across images), and enough
tiles for several per workgroup."""
import numpy as np
import pytest

import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

HALO2_TILE = 101
# (batch, H, W, pad, pool, residual)
SHAPES = [
    (1, 4, 5, 1, 0, 0),
    (2, 7, 33, 1, 0, 1),
    (3, 18, 66, 1, 1, 0),
    (2, 34, 34, 0, 1, 0),     # 32 x 32 out: no column leaves the image
    (1, 9, 31, 2, 0, 0),      # 11 x 33 out
    (40, 6, 10, 1, 1, 0),     # one tile an image
    (20, 70, 100, 1, 1, 0),   # several tiles a workgroup, ragged both ways
    (20, 70, 100, 1, 0, 0),
]


# 32 channels in: the window fits only at the 8-row tiles of 64 channels out
@pytest.mark.parametrize("cin,cout", [(16, 8), (16, 32), (16, 64), (32, 56), (32, 64)])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "b%d_%dx%d_p%d_pool%d_res%d" % s)
def test_same_bits_as_the_register_staged_tile(shape, cin, cout):
    from paper_1811_03882_amd import dn
    b, h, w, pad, pool, res = shape
    p = synth.make_params(synth.Net("t", cin, h, w, [synth.conv(cout, 3)]), 31)[0]
    x = synth.make_tensor((b, cin, h, w), 32, cin)
    r = synth.make_tensor((b, cout, h + 2 * pad - 2, w + 2 * pad - 2), 33, 1) if res else None
    ref = G.run_conv(dn, dn.BF16, x, p, 3, 1, pad, 1, pool=pool, res=r, tile=0, splits=1)
    got = G.run_conv(dn, dn.BF16, x, p, 3, 1, pad, 1, pool=pool, res=r, tile=HALO2_TILE, splits=1)
    np.testing.assert_array_equal(got, ref)


@pytest.mark.parametrize("cin,cout", [(16, 40), (24, 48), (32, 34), (32, 32), (32, 8), (24, 32)])
@pytest.mark.parametrize("shape", [(1, 4, 6, 1, 1, 0), (2, 9, 33, 1, 0, 1), (20, 70, 100, 1, 1, 0), (20, 70, 100, 1, 0, 1)],
                         ids=lambda s: "b%d_%dx%d_p%d_pool%d_res%d" % s)
def test_fewer_channel_blocks_run_as_four(shape, cin, cout):
    """Three blocks of channels out, and one or two whose window does not fit
    the taller tiles, by the library's own choice: the halo kernel at the
    larger sizes, a GEMM tile with its own split at the smaller ones."""
    from paper_1811_03882_amd import dn
    b, h, w, pad, pool, res = shape
    p = synth.make_params(synth.Net("t", cin, h, w, [synth.conv(cout, 3)]), 34)[0]
    x = synth.make_tensor((b, cin, h, w), 35, cin)
    r = synth.make_tensor((b, cout, h + 2 * pad - 2, w + 2 * pad - 2), 36, 1) if res else None
    ref = G.run_conv(dn, dn.BF16, x, p, 3, 1, pad, 1, pool=pool, res=r, tile=0, splits=1)
    got = G.run_conv(dn, dn.BF16, x, p, 3, 1, pad, 1, pool=pool, res=r)
    if b < 20:  # a split's sum: equal before the last rounding to 2^-8
        assert G.rel_l2(got, ref) < 2.0 ** -8
    else:
        np.testing.assert_array_equal(got, ref)
