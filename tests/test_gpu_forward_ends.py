"""The two ends of a resident forward that conv kernels take over: the last
conv writing the caller's FP32 NCHW tensor itself (first-layer kernel,
pipelined tiles unsplit, finished in the kernel and finished apart), and the
first-layer kernel clearing the split-K counters.  The per-layer-transfer mode
runs the same convs with the egress and the clearing as kernels of their own:
same bits where
no value is rounded in between, on every eager and graph replay, on an arena full of garbage, with
nothing written past the output; and within the dtype's gate of the FP64
oracle."""
import numpy as np
import pytest

import synth
from oracle import net as onet
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

C, LIN = synth.conv, synth.LINEAR
# name -> (in_c, h, w, batch, layers)
NETS = {
    "first_alone": (3, 17, 35, 2, [C(10, 3)]),
    "first_pooled": (3, 32, 34, 1, [C(16, 3), synth.maxpool()]),
    "first_one_channel": (1, 7, 5, 3, [C(1, 3, bn=False, act=LIN)]),
    "conv_1x1_odd": (3, 13, 13, 3, [C(128, 3), C(125, 1, bn=False, act=LIN)]),
    "conv_3x3": (3, 9, 11, 2, [C(128, 3), C(72, 3)]),
    "deep_split": (3, 6, 6, 1, [C(128, 3), C(512, 3), C(70, 3)]),
    "residual_last": (3, 12, 10, 2, [C(128, 3), C(128, 3), synth.shortcut(0)]),
    "pooled_last": (3, 12, 20, 2, [C(128, 3), C(40, 3), synth.maxpool()]),
}


@pytest.mark.parametrize("dtype", [0, 1, 2], ids=["f32", "bf16", "fp8"])
@pytest.mark.parametrize("name", list(NETS))
def test_resident_forward_equals_the_per_layer_one(name, dtype):
    from paper_1811_03882_amd import dn
    torch = G.torch_cuda()
    in_c, h, w, b, layers = NETS[name]
    net = synth.Net("t", in_c, h, w, layers)
    params = synth.make_params(net, 41)
    x = synth.make_input(net, b, 42)
    xd = G.dev(x.astype(np.float32))
    want = onet.forward(net, params, x)[-1]
    convs = sum(layer.kind == synth.CONV for layer in layers)
    fused_early = {"residual_last": 0, "pooled_last": 1, "first_pooled": 1}  # same bits up to this dtype
    ref = None
    for mode, graph in ((dn.PER_LAYER, False), (0, False), (0, True)):
        n = dn.Net(layers, in_c, h, w, b, dtype=dtype, mode=mode, leaky_slope=net.leaky_slope, bn_eps=net.bn_eps,
                   use_graph=graph)
        n.load_params(params)
        if dtype == dn.FP8:
            n.calibrate(xd, b, h, w)
        arena = G.empty_bytes(n.arena_bytes(b, h, w))
        n.bind_arena(arena)
        shape = (b,) + tuple(n.output_shape(h, w))
        size = int(np.prod(shape))
        if mode == dn.PER_LAYER:
            if dtype > fused_early.get(name, 2):
                continue  # a value rounded between the conv and the op fused into it
            y = np.empty(shape, np.float32)
            n.forward(np.ascontiguousarray(x, np.float32), b, h, w, y)
            ref = y.astype(np.float64)
            continue
        buf = torch.empty(size + 64, device="cuda")
        y = buf[:size].view(shape)
        for rep in range(3):
            buf.fill_(float("nan"))
            arena.fill_(0x5A + rep)
            n.forward(xd, b, h, w, y)
            torch.cuda.synchronize()
            assert torch.isnan(buf[size:]).all()
            got = y.cpu().numpy().astype(np.float64)
            err = G.rel_l2(got, want)
            print(name, G.NAME[dtype], "graph" if graph else "eager", "rel_l2 %.3e" % err)
            assert err < convs * G.GATE[dtype]  # each conv within its own gate
            ref = got if ref is None else ref
            np.testing.assert_array_equal(got, ref, err_msg="graph %s, pass %d" % (graph, rep))
        n.close()
