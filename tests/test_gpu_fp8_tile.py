"""The library's own choice for FP8 never is the number of the 256x256 tile,
whose kernel FP8 does not have: a layer that this tile would cover in one round
(16384 x 1024), in a net's plan; and the number itself still runs, with the
bits of the tile that stands in for it."""
import numpy as np
import pytest

import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def test_plan_and_number():
    from paper_1811_03882_amd import dn
    G.torch_cuda()
    layers = [synth.conv(512, 1), synth.conv(1024, 3)]
    n = dn.Net(layers, 3, 32, 32, 16, dtype=dn.FP8)
    n.load_params(synth.make_params(synth.Net("t", 3, 32, 32, layers), 3))
    x = G.dev(synth.make_tensor((16, 3, 32, 32), 3, 1).astype(np.float32))
    n.calibrate(x, 16, 32, 32)
    tile = n.layer_plan(1, 16, 32, 32)["tile"]
    print("tile", tile)
    assert 48 < tile < 58
    n.close()
    p = synth.make_params(synth.Net("t", 128, 9, 9, [synth.conv(264, 3)]), 5)[0]
    t = synth.make_tensor((3, 128, 9, 9), 3, 1)
    got = [G.run_conv(dn, dn.FP8, t, p, 3, 1, 1, 1, in_scale=1.0 / 448, out_scale=8.0 / 448, tile=k) for k in (48, 49)]
    np.testing.assert_array_equal(got[0], got[1])
