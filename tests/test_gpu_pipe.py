"""The pipelined GEMM conv tiles against the register-staged tile of the same
sums: both form every output from the same 16x16 MFMA steps in the same
order, so the results are equal bit for bit, at any split count.

Shapes at the edges of the tiles: rows and channels that leave ragged tiles,
one K-tile, fewer K-tiles than pipeline stages, splits without a K-tile,
strides, 1x1, 2x2 and 5x5 filters, padding wider than the image, pooling and
residual epilogues.  One shape per dtype is also held to the FP64 oracle.
"""
import numpy as np
import pytest

import oracle
import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

FIRST_PIPE, TILES = 48, 10


@pytest.fixture(scope="module")
def dn():
    from paper_1811_03882_amd import dn as _dn
    G.torch_cuda()
    assert _dn.tile_count() == FIRST_PIPE + TILES
    return _dn


# (batch, H, W, Cin in 128-byte blocks, Cout, k, stride, pad, pool, residual, splits)
SHAPES = [
    (1, 5, 7, 1, 8, 1, 1, 0, 0, 0, 1),       # one K-tile, fewer rows and channels than any tile
    (2, 9, 11, 2, 40, 1, 1, 0, 0, 1, 1),     # two K-tiles, residual
    (3, 13, 13, 1, 125, 3, 1, 1, 0, 0, 1),   # nine K-tiles, odd channels, M = 507
    (1, 16, 16, 3, 264, 3, 1, 1, 0, 1, 2),   # N past 256, split with residual
    (2, 14, 10, 1, 72, 3, 1, 1, 2, 0, 1),    # pooled
    (2, 14, 10, 2, 72, 3, 1, 1, 2, 0, 4),    # pooled and split
    (2, 17, 15, 1, 64, 3, 2, 1, 0, 0, 1),    # stride 2
    (1, 6, 9, 2, 48, 2, 1, 0, 0, 0, 3),      # 2x2 filter, 8 K-tiles over 3 splits
    (1, 7, 7, 1, 32, 5, 1, 2, 0, 0, 7),      # 5x5: 25 K-tiles over 7 splits, the last one short
    (1, 3, 2, 1, 16, 3, 1, 2, 0, 0, 4),      # padding past the image; 9 K-tiles over 4 splits of 3: one empty
]


def _run(dn, dtype, shape, tile):
    torch = G.torch_cuda()
    b, h, w, blocks, cout, k, st, pad, pool, res, splits = shape
    cin = blocks * 128 // dn.ESIZE[dtype]
    p = synth.make_params(synth.Net("t", cin, h, w, [synth.conv(cout, k)]), 7 + k)[0]
    ho, wo = (h + 2 * pad - k) // st + 1, (w + 2 * pad - k) // st + 1
    x = synth.make_tensor((b, cin, h, w), 3, cin)
    r = synth.make_tensor((b, cout, ho, wo), 4, cout) if res else None
    got = G.run_conv(dn, dtype, x, p, k, st, pad, 1, pool=pool, res=r, in_scale=1.0 / 448, res_scale=1.0 / 448,
                     out_scale=8.0 / 448, tile=tile, splits=splits)
    torch.cuda.synchronize()
    return got, (x, p, r)


@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp8"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "b%d_%dx%d_cb%d_co%d_k%d_s%d_p%d_pool%d_res%d_sp%d" % s)
def test_same_bits_as_the_register_staged_tile(dn, dtype, shape):
    ref, _ = _run(dn, dtype, shape, 0)
    for t in range(FIRST_PIPE, FIRST_PIPE + TILES):
        got, _ = _run(dn, dtype, shape, t)
        np.testing.assert_array_equal(got, ref, err_msg="tile %d" % t)


@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp8"])
def test_against_the_oracle(dn, dtype):
    shape = (3, 13, 13, 1, 125, 3, 1, 1, 0, 0, 1)
    got, (x, p, _) = _run(dn, dtype, shape, FIRST_PIPE + 1)
    ref = oracle.leaky(oracle.batchnorm(oracle.add_bias(oracle.conv2d(x, p.w, 1, 1), p.bias), p.mean, p.var, p.gamma,
                                        p.beta, 1e-5), 0.1)
    assert G.rel_l2(got, ref) < G.GATE[dtype]


def test_shapes_the_kernel_does_not_take_still_run(dn):
    """A pipelined tile asked for where channels are not whole 128-byte blocks
    runs the register-staged kernel: same bits as tile 0."""
    torch = G.torch_cuda()
    p = synth.make_params(synth.Net("t", 24, 9, 9, [synth.conv(40, 3)]), 5)[0]
    x = synth.make_tensor((2, 24, 9, 9), 3, 1)
    ref = G.run_conv(dn, dn.BF16, x, p, 3, 1, 1, 1, tile=0)
    got = G.run_conv(dn, dn.BF16, x, p, 3, 1, 1, 1, tile=FIRST_PIPE + 4)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got, ref)


# batch-16 shapes whose default choice the library's rule makes itself
@pytest.mark.parametrize("cin,cout,side,k", [(64, 64, 13, 3), (256, 512, 8, 1), (512, 256, 7, 3)])
def test_default_choice_within_the_gate(dn, cin, cout, side, k):
    p = synth.make_params(synth.Net("t", cin, side, side, [synth.conv(cout, k)]), 9)[0]
    x = synth.make_tensor((2, cin, side, side), 3, cin)
    ref = oracle.leaky(oracle.batchnorm(oracle.add_bias(oracle.conv2d(x, p.w, 1, k // 2), p.bias), p.mean, p.var,
                                        p.gamma, p.beta, 1e-5), 0.1)
    for dtype in (dn.F32, dn.BF16):
        assert G.rel_l2(G.run_conv(dn, dtype, x, p, k, 1, k // 2, 1), ref) < G.GATE[dtype]
