"""Suppression at a threshold of zero where the overlap's quotient is too small
for a float: a box of 1e-14 x 1e-15 inside one of 1e10 x 1e7.  Their IoU is
1e-46, which rounds to 0 in FP32, and decisions are taken in FP32: neither box
suppresses the other, at few candidates (one wave) and at many."""
import numpy as np
import pytest

from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [1, 40, 100, 200])  # 2 to 400 candidates
@pytest.mark.parametrize("nms", [0.0, 1e-40, 1e-20])
def test_quotient_below_the_smallest_float(pairs, nms):
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    A, side = 2, 16
    y = np.zeros((1, A, 6, side, side), np.float32)
    y[:, :, 4] = -40.0  # no object
    y[:, :, 0:2] = -80.0  # centres at their cells' corners
    cells = np.arange(side * side)[:pairs]
    i, j = cells // side, cells % side
    y[0, 0, 4, i, j] = 2.0 - cells / 1024.0
    y[0, 1, 4, i, j] = 1.0 - cells / 1024.0
    y[0, :, 2:4, i, j] = -60.0  # points: no area, no overlap
    y[0, 0, 2, 0, 0], y[0, 0, 3, 0, 0] = np.log(1e10 * side), np.log(1e7 * side)
    y[0, 1, 2, 0, 0], y[0, 1, 3, 0, 0] = np.log(1e-14 * side), np.log(1e-15 * side)
    yd = torch.from_numpy(y.reshape(1, A * 6, side, side)).cuda()
    wsb = dn.detect_workspace(1, A, 1, side, side)
    ws = G.empty_bytes(wsb)
    cap = 2 * pairs + 3
    dets = torch.zeros((1, 1, cap, 5), device="cuda")
    idx = torch.zeros((1, 1, cap), dtype=torch.int32, device="cuda")
    cnt = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
    dn.detect(yd, 1, A, 1, side, side, [1.0] * (2 * A), 0.1, nms, cap, ws, wsb, dets, idx, cnt)
    torch.cuda.synchronize()
    b = dets[0, 0].cpu().numpy()
    big = b[idx[0, 0].cpu().numpy() == 0][0]
    # one pair's quotient as FP32 forms it
    inter, uni = np.float32(1e-14) * np.float32(1e-15), big[3] * big[4]
    assert inter > 0 and np.float32(inter / uni) == 0
    assert cnt.item() == 2 * pairs
