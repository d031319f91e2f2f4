"""The halo kernel's window with its layout built in, where the padding below
the image takes window offsets past 1 GB: rows of the result that lie outside
the image hold the bias alone, whatever the image holds."""
import numpy as np
import pytest

import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def test_rows_far_below_a_large_image():
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    h, w, c, pad = 900, 32768, 16, 140
    ho, wo = h + 2 * pad - 2, w + 2 * pad - 2
    p = synth.make_params(synth.Net("t", c, h, w, [synth.conv(c, 3, bn=False)]), 5)[0]
    d = dn.conv_desc(1, h, w, c, c, 3, 1, pad, 0, 0.1, 0, 0, dn.BF16)
    wb, vb, wsb = dn.conv_sizes(d)
    assert wsb == 0  # the halo kernel's: no split
    wbuf, bias, scale = G.empty_bytes(wb), G.empty_bytes(vb), G.empty_bytes(vb)
    dn.conv_pack(d, p.w, p.bias, None, None, None, None, 1e-5, wbuf, bias, scale)
    x = torch.zeros((1, h, w, c), dtype=torch.bfloat16, device="cuda")
    x[:, :40] = float("inf")  # where offsets from 1 GB on would land if they wrapped
    y = torch.empty((1, ho, wo, c), dtype=torch.bfloat16, device="cuda")
    dn.conv2d(d, x, wbuf, bias, scale, None, y, None, 0)
    torch.cuda.synchronize()
    want = torch.from_numpy(p.bias.astype(np.float32)).to(torch.bfloat16).cuda()
    assert (y[:, h + pad:] == want).all()
