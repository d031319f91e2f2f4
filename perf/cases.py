"""The work this library is used for, as cases with a size, inputs and one pass.

Whole calls: a forward or an input gradient through ``Net``, weights loaded
and the arena bound beforehand, tiles by the library's own rule.  Single
layers: the standalone entry points with the weights packed beforehand, tile
and split by the library's own rule.  The sizes are those of the two networks
the repository benchmarks (nine convolutions at 416x416, and the residual
network at 256x256), of its detection and Jacobi benchmarks, and of the
serving trace (sides 160 to 608).
"""
import math
import types

import numpy as np
import torch

from paper_1811_03882_amd import dn

SLOPE, EPS = 0.1, 1e-5
DTYPE = {"f32": dn.F32, "bf16": dn.BF16, "fp8": dn.FP8}
TORCH = {dn.F32: torch.float32, dn.BF16: torch.bfloat16, dn.FP8: torch.float8_e4m3fn}
LABELS = 20        # classes of the detection head
ANCHORS = 5
WEIGHT_SEED = 11   # a program's weights do not change with its inputs


# ---------------------------------------------------------------- cases


def listed():
    return [
        # one small image through the one-block network: latency and launches
        dict(name="block_f32_b1", kind="net", net="block", dtype="f32", batch=1, side=32),
        # one frame through the nine-layer network, FP32: the latency of a frame
        dict(name="net_f32_b1", kind="net", net="plain", dtype="f32", batch=1, side=416),
        # a full batch of frames through the nine-layer network, BF16: throughput
        dict(name="net_bf16_b64", kind="net", net="plain", dtype="bf16", batch=64, side=416),
        # one gradient of the image modification program (forward and backward)
        dict(name="grad_bf16_b16", kind="grad", net="plain", dtype="bf16", batch=16, side=416),
        # the widest layer of the nine-layer network
        dict(name="conv_wide_bf16", kind="conv", dtype="bf16", batch=64, side=13, cin=1024, cout=1024, k=3,
             stride=1, pool=0, res=0, act=1),
        # a high-resolution layer with its 2x2 pool
        dict(name="conv_pool_bf16", kind="conv", dtype="bf16", batch=64, side=104, cin=32, cout=64, k=3,
             stride=1, pool=2, res=0, act=1),
        # the 3x3 half of a residual unit with its shortcut, fourth stage, batch 16
        dict(name="conv_res_bf16", kind="conv", dtype="bf16", batch=16, side=16, cin=256, cout=512, k=3,
             stride=1, pool=0, res=1, act=1),
        # a wide layer in FP8
        dict(name="conv_fp8", kind="conv", dtype="fp8", batch=32, side=13, cin=512, cout=1024, k=3,
             stride=1, pool=0, res=0, act=1),
        # the 1x1 linear head: an odd channel count
        dict(name="conv_head_bf16", kind="conv", dtype="bf16", batch=64, side=13, cin=1024, cout=125, k=1,
             stride=1, pool=0, res=0, act=0),
        # backward-data of a middle layer
        dict(name="conv_bwd_bf16", kind="bwd", dtype="bf16", batch=64, side=52, cin=64, cout=128, k=3,
             stride=1, accumulate=0),
        # boxes from the head's output: decode and per-class suppression
        dict(name="detect_b64", kind="detect", batch=64, grid=13, max_det=50),
        # Jacobi iterations of the Laplace equation on a resident grid
        dict(name="jacobi_1000x1500", kind="jacobi", n=1000, m=1500, iters=64),
    ]


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    def log(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))
    kind = rng.choice(["block", "net_f32", "net_bf16", "grad", "wide", "pool", "res", "fp8", "head", "bwd",
                       "detect", "jacobi"])
    if kind == "block":
        return dict(kind="net", net="block", dtype=rng.choice(["f32", "bf16"]), batch=log(1, 8), side=rng.randint(17, 64))
    if kind == "net_f32":
        return dict(kind="net", net="plain", dtype="f32", batch=log(1, 2), side=rng.randint(160, 415))
    if kind == "net_bf16":
        return dict(kind="net", net="plain", dtype="bf16", batch=log(2, 63), side=16 * rng.randint(10, 26))
    if kind == "grad":
        return dict(kind="grad", net="plain", dtype="bf16", batch=log(1, 15), side=16 * rng.randint(6, 26))
    if kind == "wide":
        return dict(kind="conv", dtype="bf16", batch=log(8, 63), side=rng.randint(7, 13), cin=rng.choice([256, 512, 1024]),
                    cout=rng.choice([256, 512, 768, 1024]), k=3, stride=1, pool=0, res=0, act=1)
    if kind == "pool":
        return dict(kind="conv", dtype="bf16", batch=log(2, 63), side=2 * rng.randint(20, 52), cin=rng.choice([16, 24, 32]),
                    cout=rng.choice([32, 48, 64]), k=3, stride=1, pool=2, res=0, act=1)
    if kind == "res":
        c = rng.choice([128, 256, 512])
        k = rng.choice([1, 3])
        return dict(kind="conv", dtype="bf16", batch=log(1, 15), side=rng.randint(8, 20), cin=c, cout=2 * c, k=k,
                    stride=1, pool=0, res=rng.randint(0, 1), act=1)
    if kind == "fp8":
        return dict(kind="conv", dtype="fp8", batch=log(4, 31), side=rng.randint(7, 13), cin=rng.choice([128, 256, 512]),
                    cout=rng.choice([256, 512, 1024]), k=3, stride=1, pool=0, res=0, act=1)
    if kind == "head":
        return dict(kind="conv", dtype="bf16", batch=log(2, 63), side=rng.randint(5, 13), cin=rng.choice([512, 1024]),
                    cout=rng.choice([75, 125, 255]), k=1, stride=1, pool=0, res=0, act=0)
    if kind == "bwd":
        c = rng.choice([64, 128, 256])
        return dict(kind="bwd", dtype="bf16", batch=log(4, 63), side=rng.randint(13, 52 * 64 // c), cin=c, cout=2 * c,
                    k=3, stride=1, accumulate=rng.randint(0, 1))
    if kind == "detect":
        return dict(kind="detect", batch=log(1, 63), grid=rng.randint(5, 19), max_det=rng.choice([20, 50]))
    return dict(kind="jacobi", n=log(33, 1500), m=log(33, 1500), iters=log(2, 63))


# ---------------------------------------------------------------- networks


def _layer(kind, cout=0, k=0, stride=1, bn=False, act=0):
    return types.SimpleNamespace(kind=kind, cout=cout, ksize=k, stride=stride, pad=k // 2 if kind == dn.CONV else 0,
                                 batchnorm=bn, activation=act, src=-1)


def _layers(net):
    """block: conv3x3(16) + pool.  plain: six conv3x3 + pool of widths 16 to
    512 (the last pool with stride 1), two conv3x3 to 1024, a linear 1x1 to 125."""
    widths = (16,) if net == "block" else (16, 32, 64, 128, 256, 512)
    out = []
    for i, c in enumerate(widths):
        out += [_layer(dn.CONV, c, 3, bn=True, act=1), _layer(dn.MAXPOOL, 0, 2, 1 if i == 5 else 2)]
    if net == "plain":
        out += [_layer(dn.CONV, 1024, 3, bn=True, act=1), _layer(dn.CONV, 1024, 3, bn=True, act=1),
                _layer(dn.CONV, 125, 1)]
    return out


_kept = {}


def _conv_params(key, cout, cin, k, bn):
    """He-initialised FP64 weights and batch-norm statistics, drawn once per shape."""
    key = (key, cout, cin, k, bn)
    if key not in _kept:
        g = torch.Generator().manual_seed(WEIGHT_SEED + 31 * cout + 7 * cin + k + 1009 * len(str(key)))
        rand = lambda *s: torch.rand(*s, generator=g, dtype=torch.float64)  # noqa: E731
        norm = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64)  # noqa: E731
        p = dict(w=(norm(cout, cin, k, k) * math.sqrt(2.0 / (cin * k * k))).numpy(), bias=(0.1 * norm(cout)).numpy(),
                 mean=None, var=None, gamma=None, beta=None)
        if bn:
            p.update(mean=(0.3 * norm(cout)).numpy(), var=(0.5 + rand(cout)).numpy(),
                     gamma=(0.9 + 0.2 * rand(cout)).numpy(), beta=(0.2 * norm(cout)).numpy())
        _kept[key] = p
    return _kept[key]


def _net_params(net):
    out, c = [], 3
    for i, L in enumerate(_layers(net)):
        if L.kind != dn.CONV:
            out.append(None)
            continue
        out.append(types.SimpleNamespace(**_conv_params("%s%d" % (net, i), L.cout, c, L.ksize, L.batchnorm)))
        c = L.cout
    return out


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _image(case, seed):
    return torch.rand((case["batch"], 3, case["side"], case["side"]), generator=_gen(seed), device="cuda")


def _activation(shape, g):
    """What a leaky layer leaves: half of it small and negative."""
    v = torch.randn(shape, generator=g, device="cuda")
    return torch.where(v > 0, v, v * SLOPE)


# ---------------------------------------------------------------- one pass


def prepare(case, seed):
    return {"net": _prepare_net, "grad": _prepare_net, "conv": _prepare_conv, "bwd": _prepare_bwd,
            "detect": _prepare_detect, "jacobi": _prepare_jacobi}[case["kind"]](case, seed)


def _prepare_net(case, seed):
    b, s = case["batch"], case["side"]
    layers = _layers(case["net"])
    # the forward replays a captured graph on its fixed buffers, as the benchmark and the serving slots do
    net = dn.Net(layers, 3, s, s, b, dtype=DTYPE[case["dtype"]], leaky_slope=SLOPE, bn_eps=EPS, use_graph=True)
    net.load_params(_net_params(case["net"]))
    st = types.SimpleNamespace(case=case, net=net, batch=b, side=s, x=_image(case, seed), last=len(layers) - 1)
    if case["kind"] == "grad":
        arena = net.input_gradient_arena_bytes(st.last, b, s, s)
        st.y = torch.empty_like(st.x)
    else:
        arena = net.arena_bytes(b, s, s)
        st.y = torch.empty((b,) + net.output_shape(s, s), device="cuda")
    st.arena = _bytes(arena)
    net.bind_arena(st.arena)
    return st


def _conv_out(case):
    return (case["side"] + 2 * (case["k"] // 2) - case["k"]) // case["stride"] + 1


def _nhwc(v, dtype):
    """[n][h][w][c] values in the storage type, channels padded with zeros."""
    c = v.shape[-1]
    cp = dn.channel_pad(dtype, c)
    if cp != c:
        v = torch.nn.functional.pad(v, (0, cp - c))
    return v.to(TORCH[dtype]).contiguous()


# FP8 activations carry one static scale per tensor; outputs of He-initialised
# layers reach about twice the inputs' range
IN_SCALE, OUT_SCALE = 5.0 / 448.0, 8.0 / 448.0


def _conv_inputs(case, seed):
    dt, g = DTYPE[case["dtype"]], _gen(seed)
    s, o = (IN_SCALE, OUT_SCALE) if dt == dn.FP8 else (1.0, 1.0)
    x = _nhwc((_activation((case["batch"], case["side"], case["side"], case["cin"]), g) / s).clamp_(-448, 448), dt)
    ho = _conv_out(case)
    r = _nhwc(_activation((case["batch"], ho, ho, case["cout"]), g), dt) if case["res"] else None
    return x, r, s, o


def _prepare_conv(case, seed):
    dt = DTYPE[case["dtype"]]
    x, r, s, o = _conv_inputs(case, seed)
    d = dn.conv_desc(case["batch"], case["side"], case["side"], case["cin"], case["cout"], case["k"], case["stride"],
                     case["k"] // 2, case["act"], SLOPE, case["pool"], case["res"], dt, s, 1.0, o)
    wb, vb, ws = dn.conv_sizes(d)
    st = types.SimpleNamespace(case=case, d=d, x=x, r=r, w=_bytes(wb), b=_bytes(vb), s=_bytes(vb),
                               ws=_bytes(ws) if ws else None, ws_bytes=ws)
    p = _conv_params("conv", case["cout"], case["cin"], case["k"], bool(case["act"]))
    dn.conv_pack(d, p["w"], p["bias"], p["mean"], p["var"], p["gamma"], p["beta"], EPS, st.w, st.b, st.s)
    ho = _conv_out(case) // (2 if case["pool"] else 1)
    st.y = torch.empty((case["batch"], ho, ho, dn.channel_pad(dt, case["cout"])), dtype=TORCH[dt], device="cuda")
    return st


def _bwd_inputs(case, seed):
    g, ho = _gen(seed), _conv_out(case)
    dy = _nhwc(torch.randn((case["batch"], ho, ho, case["cout"]), generator=g, device="cuda"), dn.BF16)
    # zeros where nothing was added yet: repeated passes keep adding the same gradient
    dx = torch.zeros((case["batch"], case["side"], case["side"], case["cin"]), dtype=torch.bfloat16, device="cuda")
    return dy, dx


def _prepare_bwd(case, seed):
    dy, dx = _bwd_inputs(case, seed)
    d = dn.conv_desc(case["batch"], case["side"], case["side"], case["cin"], case["cout"], case["k"], case["stride"],
                     case["k"] // 2, dn.LEAKY, SLOPE, 0, 0, dn.BF16)
    wb, vb, ws = dn.conv_backward_sizes(d)
    st = types.SimpleNamespace(case=case, d=d, dy=dy, dx=dx, w=_bytes(wb), b=_bytes(vb), s=_bytes(vb),
                               ws=_bytes(ws) if ws else None, ws_bytes=ws)
    p = _conv_params("conv", case["cout"], case["cin"], case["k"], True)
    dn.conv_pack_backward(d, p["w"], p["mean"], p["var"], p["gamma"], EPS, st.w, st.b, st.s)
    return st


def _anchor_wh():
    return [float(v) for v in np.random.default_rng(6).uniform(0.5, 12.0, 2 * ANCHORS)]


def _head_output(case, seed):
    """A trained head's output: most cells empty, some confident objects that
    their neighbouring cells repeat, so that boxes compete."""
    g, n, s = _gen(seed), case["batch"], case["grid"]
    y = torch.randn((n, ANCHORS, 5 + LABELS, s, s), generator=g, device="cuda")
    y[:, :, 2:4] *= 0.7
    y[:, :, 4] = 1.4 * y[:, :, 4] - 1.0
    y[:, :, 5:] *= 1.4
    r = np.random.default_rng(seed)
    for i in range(n):
        for _ in range(6):
            ci, cj, k = int(r.integers(0, s)), int(r.integers(0, s)), int(r.integers(0, LABELS))
            i0, i1, j0, j1 = max(0, ci - 1), min(s, ci + 2), max(0, cj - 1), min(s, cj + 2)
            y[i, :, 4, i0:i1, j0:j1] += 3.0
            y[i, :, 5 + k, i0:i1, j0:j1] += 6.0
    return y.reshape(n, ANCHORS * (5 + LABELS), s, s).contiguous()


def _prepare_detect(case, seed):
    n, s, m = case["batch"], case["grid"], case["max_det"]
    ws = dn.detect_workspace(n, ANCHORS, LABELS, s, s)
    return types.SimpleNamespace(
        case=case, y=_head_output(case, seed), anchors=_anchor_wh(), ws=_bytes(ws), ws_bytes=ws,
        dets=torch.zeros((n, LABELS, m, 5), device="cuda"),
        index=torch.zeros((n, LABELS, m), dtype=torch.int32, device="cuda"),
        counts=torch.zeros((n, LABELS), dtype=torch.int32, device="cuda"))


def _prepare_jacobi(case, seed):
    u = torch.rand((case["n"], case["m"]), generator=_gen(seed), dtype=torch.float64, device="cuda")
    return types.SimpleNamespace(case=case, u=u, work=torch.empty_like(u),
                                 change=torch.zeros(1, dtype=torch.float64, device="cuda"))


def run(st):
    case = st.case
    kind = case["kind"]
    stream = torch.cuda.current_stream()
    if kind == "net":
        st.net.forward(st.x, st.batch, st.side, st.side, st.y, stream)
        return st.y
    if kind == "grad":
        st.net.input_gradient(st.last, st.x, st.batch, st.side, st.side, st.y, stream)
        return st.y
    if kind == "conv":
        dn.conv2d(st.d, st.x, st.w, st.b, st.s, st.r, st.y, st.ws, st.ws_bytes, stream)
        return st.y
    if kind == "bwd":
        dn.conv_backward_data(st.d, st.dy, st.w, st.b, st.s, case["accumulate"], st.dx, st.ws, st.ws_bytes, stream)
        return st.dx
    if kind == "detect":
        dn.detect(st.y, case["batch"], ANCHORS, LABELS, case["grid"], case["grid"], st.anchors, 0.2, 0.45,
                  case["max_det"], st.ws, st.ws_bytes, st.dets, st.index, st.counts, stream)
        return {"dets": st.dets, "index": st.index, "counts": st.counts}
    dn.jacobi(st.u, st.work, case["n"], case["m"], case["iters"], st.change, stream)
    return {"u": st.u, "change": st.change}


# ---------------------------------------------------------------- what a pass cannot do without


def _net_work(case):
    """(flops, weight elements, output elements) of one forward."""
    c, h, flops, weights = 3, case["side"], 0.0, 0
    for L in _layers(case["net"]):
        if L.kind == dn.CONV:
            flops += 2.0 * case["batch"] * h * h * L.cout * c * L.ksize ** 2
            weights += L.cout * c * L.ksize ** 2
            c = L.cout
        else:
            h = (h - 1) // L.stride + 1
    return flops, weights, case["batch"] * c * h * h


def work(case):
    kind = case["kind"]
    if kind in ("net", "grad"):
        flops, weights, outs = _net_work(case)
        image = case["batch"] * 3 * case["side"] ** 2 * 4
        es = dn.ESIZE[DTYPE[case["dtype"]]]
        if kind == "grad":  # the input gradient costs a second pass of the same products
            return {"bytes": 2 * image + 2 * weights * es, "flops": 2 * flops}
        return {"bytes": image + weights * es + outs * 4, "flops": flops}
    if kind in ("conv", "bwd"):
        es, ho = dn.ESIZE[DTYPE[case["dtype"]]], _conv_out(case)
        b, k2 = case["batch"], case["k"] ** 2
        x, y = b * case["side"] ** 2 * case["cin"], b * ho * ho * case["cout"]
        flops = 2.0 * y * case["cin"] * k2
        if kind == "conv":
            y = y * (1 + case["res"]) // (4 if case["pool"] else 1)
        else:
            x *= 1 + case["accumulate"]
        return {"bytes": (x + y + case["cout"] * case["cin"] * k2) * es, "flops": flops}
    if kind == "detect":
        cells, n = case["grid"] ** 2 * ANCHORS, case["batch"]
        return {"bytes": n * cells * (5 + LABELS) * 4 + n * LABELS * 4, "flops": n * cells * (20.0 + 10.0 * LABELS)}
    return {"bytes": 2 * case["n"] * case["m"] * 8, "flops": 4.0 * case["n"] * case["m"] * case["iters"]}


# ---------------------------------------------------------------- the same in 64 bits


def _fold(p):
    """Weights and bias with the inference batch norm folded in, FP64 on the GPU."""
    t = {k: None if v is None else torch.from_numpy(v).cuda() for k, v in p.items()}
    if t["mean"] is None:
        return t["w"], t["bias"]
    g = t["gamma"] / torch.sqrt(t["var"] + EPS)
    return t["w"] * g[:, None, None, None], (t["bias"] - t["mean"]) * g + t["beta"]


def _conv64(x, w, stride=1):
    """[n][h][w][c] FP64 convolution with padding k // 2: one matrix product per tap."""
    k = w.shape[2]
    ho = (x.shape[1] + 2 * (k // 2) - k) // stride + 1
    wo = (x.shape[2] + 2 * (k // 2) - k) // stride + 1
    xp = torch.nn.functional.pad(x, (0, 0, k // 2, k // 2, k // 2, k // 2))
    y = 0.0
    for r in range(k):
        for s in range(k):
            v = xp[:, r:r + (ho - 1) * stride + 1:stride, s:s + (wo - 1) * stride + 1:stride]
            y = y + (v.reshape(-1, w.shape[1]) @ w[:, :, r, s].t().contiguous()).reshape(x.shape[0], ho, wo, -1)
    return y


def _pool64(x, stride):
    n, h, w, c = x.shape
    ho, wo = (h - 1) // stride + 1, (w - 1) // stride + 1
    v = torch.nn.functional.pad(x, (0, 0, 0, 2, 0, 2), value=-math.inf)
    parts = [v[:, a:a + stride * (ho - 1) + 1:stride, b:b + stride * (wo - 1) + 1:stride] for a in (0, 1) for b in (0, 1)]
    return torch.maximum(torch.maximum(parts[0], parts[1]), torch.maximum(parts[2], parts[3]))


def _leaky64(x, act):
    return torch.where(x > 0, x, x * float(np.float32(SLOPE))) if act else x


def _net64(case, x):
    v = x.double().permute(0, 2, 3, 1)
    for L, p in zip(_layers(case["net"]), _net_params(case["net"])):
        if L.kind == dn.CONV:
            w, b = _fold(vars(p))
            v = _leaky64(_conv64(v, w) + b, L.activation)
        else:
            v = _pool64(v, L.stride)
    return v.permute(0, 3, 1, 2).contiguous()


def exact(case, seed):
    kind = case["kind"]
    if kind == "net":
        x = _image(case, seed)
        return torch.cat([_net64(case, x[i:i + 4]) for i in range(0, case["batch"], 4)])
    if kind == "grad":
        # piecewise linear in the leaky signs and the pools' choices, which 16-bit
        # activations take differently near a tie: no value to hold it to
        return None
    if kind == "conv":
        x, r, s, o = _conv_inputs(case, seed)
        w, b = _fold(_conv_params("conv", case["cout"], case["cin"], case["k"], bool(case["act"])))
        y = _leaky64(_conv64(x[..., :case["cin"]].double() * s, w, case["stride"]) + b, case["act"])
        if r is not None:
            y = y + r[..., :case["cout"]].double()
        if case["pool"]:
            y = _pool64(y, 2)
        y = y / o
        cp = dn.channel_pad(DTYPE[case["dtype"]], case["cout"])
        return torch.nn.functional.pad(y, (0, cp - case["cout"])).contiguous()
    if kind == "bwd":
        dy, dx = _bwd_inputs(case, seed)
        p = _conv_params("conv", case["cout"], case["cin"], case["k"], True)
        g = torch.from_numpy(p["gamma"] / np.sqrt(p["var"] + EPS)).cuda()
        w = torch.from_numpy(p["w"]).cuda() * g[:, None, None, None]
        return _conv64(dy.double(), w.flip(2, 3).transpose(0, 1).contiguous())
    if kind == "detect":
        return _detect64(case, seed)
    u = torch.rand((case["n"], case["m"]), generator=_gen(seed), dtype=torch.float64, device="cuda")
    change = torch.zeros(1, dtype=torch.float64, device="cuda")
    for _ in range(case["iters"]):
        v = u.clone()
        v[1:-1, 1:-1] = 0.25 * (((u[:-2, 1:-1] + u[2:, 1:-1]) + u[1:-1, :-2]) + u[1:-1, 2:])
        change = (v - u).abs().max().reshape(1)
        u = v
    return {"u": u, "change": change}


def _iou64(p, q):
    lo = np.maximum(p[:2] - p[2:] / 2, q[:, :2] - q[:, 2:] / 2)
    hi = np.minimum(p[:2] + p[2:] / 2, q[:, :2] + q[:, 2:] / 2)
    inter = np.prod(np.maximum(0.0, hi - lo), axis=1)
    union = p[2] * p[3] + q[:, 2] * q[:, 3] - inter
    return np.where(union > 0, inter / np.where(union > 0, union, 1.0), 0.0)


def _detect64(case, seed):
    n, s, m = case["batch"], case["grid"], case["max_det"]
    y = _head_output(case, seed).double().cpu().numpy().reshape(n, ANCHORS, 5 + LABELS, s, s)
    y = y.transpose(0, 3, 4, 1, 2).reshape(n, s * s * ANCHORS, 5 + LABELS)  # box index (i*s + j)*ANCHORS + a
    cell = np.arange(s * s * ANCHORS) // ANCHORS
    wh = np.asarray(_anchor_wh(), np.float32).astype(np.float64).reshape(-1, 2)[np.arange(s * s * ANCHORS) % ANCHORS]
    sig = lambda v: 1.0 / (1.0 + np.exp(-v))  # noqa: E731
    box = np.stack([(cell % s + sig(y[..., 0])) / s, (cell // s + sig(y[..., 1])) / s,
                    wh[:, 0] * np.exp(y[..., 2]) / s, wh[:, 1] * np.exp(y[..., 3]) / s], axis=-1)
    e = np.exp(y[..., 5:] - y[..., 5:].max(-1, keepdims=True))
    score = sig(y[..., 4:5]) * (e / e.sum(-1, keepdims=True))
    dets, index, counts = np.zeros((n, LABELS, m, 5)), np.zeros((n, LABELS, m), np.int32), np.zeros((n, LABELS), np.int32)
    for i in range(n):
        for k in range(LABELS):
            c = np.flatnonzero(score[i, :, k] >= float(np.float32(0.2)))
            c = c[np.argsort(-score[i, c, k], kind="stable")]
            while c.size and counts[i, k] < m:
                b, at = c[0], counts[i, k]
                dets[i, k, at] = (score[i, b, k], *box[i, b])
                index[i, k, at] = b
                counts[i, k] += 1
                c = c[1:][_iou64(box[i, b], box[i, c[1:]]) <= float(np.float32(0.45))]
    return {"dets": dets, "index": index, "counts": counts}
