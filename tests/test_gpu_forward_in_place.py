"""A resident forward whose result goes over its image: a net of one conv as
wide as its input, with the same buffer for both, with a result that begins
inside the image, and with two buffers side by side; same bits as with a
buffer of its own."""
import numpy as np
import pytest

import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [False, True], ids=["eager", "graph"])
@pytest.mark.parametrize("dtype", [0, 1], ids=["f32", "bf16"])
def test_result_over_the_image(dtype, graph):
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    b, h, w = 16, 130, 190  # many tiles, whose windows overlap
    net = synth.Net("t", 3, h, w, [synth.conv(3, 3)])
    n = dn.Net(net.layers, 3, h, w, b, dtype=dtype, use_graph=graph)
    n.load_params(synth.make_params(net, 3))
    arena = G.empty_bytes(n.arena_bytes(b, h, w))
    n.bind_arena(arena)
    x = G.dev(synth.make_input(net, b, 4).astype(np.float32))
    ref = torch.empty_like(x)
    n.forward(x, b, h, w, ref)
    size = x.numel()
    for shift in (0, 1, 3 * h * w, size):
        buf = torch.empty(size + shift, device="cuda")
        for _ in range(3):
            buf[:size] = x.reshape(-1)
            n.forward(buf[:size], b, h, w, buf[shift:])
            torch.cuda.synchronize()
            assert torch.equal(buf[shift:].view(x.shape), ref), shift
    n.close()
