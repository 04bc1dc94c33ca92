"""The work that users of this library have it do, as cases that can be timed.

Every case is one pass through the public entry points with the library's own choice of kernel (variant = -1), operands
resident in HBM under their layouts, weights packed and descriptors made once.  Seven kinds of work:

layers     the five ResNet-50-style convolution layers of workloads/configs.py (3x3 at four stages, and the 1x1 that
           narrows 4*width channels to width), as written by `width` (channels of the first stage) and `size` (its
           images' side); each stage doubles the channels and halves the side.  One alt_conv2d_multi call: on one stream,
           or (`streams`) on five.
stem       the first layer of an image network: 3 channels as images arrive (NCHW), 7x7 stride 2, bias and ReLU, stored
           as the next layer reads it (NHWC).
encoder    the products of a BERT-shaped layer over `seqs` sequences of `seq` tokens: projection, feed-forward up and
           down, and the attention scores of all heads (batched).
product    one large matrix product.
convert    the conversion operator on activation tensors: out of the default layout (to NHWC and to NCHW16c) and back.
mobile     an inverted-residual block in NHWC: 1x1 widening with bias and ReLU, depth-wise 3x3 with bias and ReLU, 1x1
           narrowing with bias, and the residual sum.
operators  the remaining operators on one feature map: 3-D convolution, transposed 2-D and transposed 3-D convolution."""
import math

import torch

import paper_2210_12415_amd as alt

_FIELDS = {"bf16": (alt.BF16, torch.bfloat16, 2), "f32": (alt.F32, torch.float32, 4)}

# As much work as the largest listed case has; drawn cases stay below it.
_MOST_FLOPS = 2.6e11


def listed():
    return [
        # Interactive inference: one image at a time, launch latency and idle compute units.
        dict(name="layers_b1", kind="layers", batch=1, width=64, size=56, layout="NHWC", dtype="bf16", streams=False),
        # The benchmark's own step: batch 16, independent layers on streams of their own.
        dict(name="layers_b16_streams", kind="layers", batch=16, width=64, size=56, layout="NHWC", dtype="bf16", streams=True),
        # Training-sized batch, one layer after the other.
        dict(name="layers_b256", kind="layers", batch=256, width=64, size=56, layout="NHWC", dtype="bf16", streams=False),
        # Tensors left in the layouts that other programs hand over.
        dict(name="layers_b16_default_layout", kind="layers", batch=16, width=64, size=56, layout="NCHW", dtype="bf16", streams=False),
        # Single precision, as in the paper's own evaluation, at an odd batch.
        dict(name="layers_b5_f32", kind="layers", batch=5, width=64, size=56, layout="NHWC", dtype="f32", streams=False),
        # The first layer of ResNet-18 (Table 3 of the paper) on a batch of photographs.
        dict(name="stem_b16", kind="stem", batch=16, channels=64, size=224),
        # BERT-base: 16 sequences of 128 tokens.
        dict(name="encoder_16x128", kind="encoder", seqs=16, seq=128, heads=12, weights="NK"),
        # The same layer for one short query: few rows, odd extents.
        dict(name="encoder_1x37", kind="encoder", seqs=1, seq=37, heads=12, weights="KN"),
        dict(name="product_4096", kind="product", M=4096, N=4096, K=4096, weights="KN"),
        # The three activation shapes the conversion operator is measured on.
        dict(name="convert_b16", kind="convert", batch=16, width=64, size=56, dtype="bf16"),
        # MobileNet-V2's block at 56x56: 24 channels widened six times.
        dict(name="mobile_b16", kind="mobile", batch=16, C=24, expand=6, size=56),
        # ResNet3D-18-shaped volume and decoder-shaped up-sampling layers.
        dict(name="operators_b2", kind="operators", batch=2, C=128, depth=8, size=28),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread evenly over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layers"] * 5 + ["stem", "encoder", "encoder", "product", "convert", "mobile", "operators"])
    while True:
        if kind == "layers":
            layout, dtype = rng.choice([("NHWC", "bf16")] * 3 + [("NCHW", "bf16"), ("NHWC", "f32")])
            most = 256 if layout == "NHWC" and dtype == "bf16" else 32 if dtype == "bf16" else 8
            c = dict(kind=kind, batch=_log(rng, 1, most), width=rng.randrange(32, 129, 8), size=rng.randrange(28, 81),
                     layout=layout, dtype=dtype, streams=rng.random() < 0.3)
        elif kind == "stem":
            c = dict(kind=kind, batch=_log(rng, 1, 64), channels=rng.choice([32, 48, 64, 96]), size=rng.randrange(96, 321))
        elif kind == "encoder":
            c = dict(kind=kind, seqs=_log(rng, 1, 64), seq=_log(rng, 8, 512), heads=rng.randrange(4, 17), weights=rng.choice(["NK", "KN"]))
        elif kind == "product":
            c = dict(kind=kind, M=_log(rng, 256, 8192), N=8 * _log(rng, 32, 1024), K=8 * _log(rng, 32, 1024), weights=rng.choice(["NK", "KN"]))
        elif kind == "convert":
            c = dict(kind=kind, batch=_log(rng, 1, 256), width=16 * rng.randrange(2, 9), size=rng.randrange(28, 81),
                     dtype=rng.choice(["bf16", "f32"]))
        elif kind == "mobile":
            c = dict(kind=kind, batch=_log(rng, 1, 64), C=8 * rng.randrange(2, 13), expand=rng.choice([4, 6]), size=rng.randrange(7, 85))
        else:
            c = dict(kind=kind, batch=_log(rng, 1, 8), C=16 * rng.randrange(2, 13), depth=rng.randrange(2, 13), size=rng.randrange(7, 41))
        w = work(c)
        limit = _MOST_FLOPS if c.get("dtype") != "f32" or kind == "convert" else _MOST_FLOPS / 16
        if w["flops"] <= limit and w["bytes"] <= 9e8:
            return c


# ---- the problems a case stands for ------------------------------------------------------------------------------------

def _half(v, n=1):
    for _ in range(n):
        v = (v + 1) // 2
    return v


def _layers(case):
    """(C, side, K, filter, padding) of the five layers."""
    w, s = case["width"], case["size"]
    return [(w << i, _half(s, i), w << i, 3, 1) for i in range(4)] + [(4 * w, s, w, 1, 0)]


def _products(case):
    """(batch, M, N, K, layout of B) of the products."""
    if case["kind"] == "product":
        return [(1, case["M"], case["N"], case["K"], "KN->" + case["weights"])]
    tokens, hidden, b = case["seqs"] * case["seq"], 64 * case["heads"], "KN->" + case["weights"]
    return [(1, tokens, hidden, hidden, b), (1, tokens, 4 * hidden, hidden, b), (1, tokens, hidden, 4 * hidden, b),
            (case["seqs"] * case["heads"], case["seq"], case["seq"], 64, "KN->NK")]


def _tensors(case):
    """The activation tensors of the conversion case: an early, a middle and a late stage of a network."""
    n, w, s = case["batch"], case["width"], case["size"]
    return [(n, w, s, s), (n, 4 * w, _half(s, 2), _half(s, 2)), (4 * n, 8 * w, _half(s, 3), _half(s, 3))]


def work(case):
    kind = case["kind"]
    if kind == "layers":
        es, n, elems, flops = _FIELDS[case["dtype"]][2], case["batch"], 0, 0
        for C, s, K, r, _ in _layers(case):
            elems += n * s * s * (C + K) + K * C * r * r
            flops += 2 * n * s * s * K * C * r * r
        return {"bytes": es * elems, "flops": flops}
    if kind == "stem":
        n, K, s = case["batch"], case["channels"], case["size"]
        o = (s - 1) // 2 + 1
        return {"bytes": 2 * (n * 3 * s * s + K * 147 + n * K * o * o) + 4 * K, "flops": 2 * n * K * o * o * 147}
    if kind in ("encoder", "product"):
        ps = _products(case)
        return {"bytes": 2 * sum(b * (m * k + k * n + m * n) for b, m, n, k, _ in ps), "flops": 2 * sum(b * m * n * k for b, m, n, k, _ in ps)}
    if kind == "convert":
        # each of the three conversions of a tensor reads it once and writes it once
        return {"bytes": 6 * _FIELDS[case["dtype"]][2] * sum(math.prod(t) for t in _tensors(case)), "flops": 0}
    n, C, s = case["batch"], case["C"], case["size"]
    if kind == "mobile":
        # the calls return their outputs to the program: widened, filtered, narrowed and summed maps
        E, px = C * case["expand"], n * s * s
        elems = px * ((C + E) + (E + E) + (E + C) + 3 * C) + 2 * C * E + 9 * E
        return {"bytes": 2 * elems + 4 * (2 * E + C), "flops": 2 * px * (2 * C * E + 9 * E)}
    D, K = case["depth"], C // 2
    px, vol = n * D * s * s, D * s * s * n
    elems = (vol * 2 * C + 27 * C * C) + (px * (C + 4 * K) + 16 * C * K) + (vol * (C + 8 * K) + 64 * C * K)
    return {"bytes": 2 * elems, "flops": 2 * (vol * 27 * C * C + px * 16 * C * K + vol * 64 * C * K)}


def tolerance(case):
    """Against the same sums in 64 bits, results in bf16 (one rounding of a 32-bit sum) measure a 2-norm error of 1.66e-3 and a
    largest of 3.9e-3 of the value, 32-bit results 1.5e-7 to 2.3e-7 and 1.1e-6; two rounded results are up to one step of
    bf16 (7.8e-3) apart."""
    if case["kind"] == "convert":
        return "exact"
    if case.get("dtype") == "f32":
        return {"rel": 1e-6, "max": 5e-6}
    if case["kind"] == "mobile":
        # four roundings follow one another
        return {"rel": 1e-2, "max": 3e-2}
    return {"rel": 6e-3, "max": 1.2e-2}


# ---- what a program has in hand before the call --------------------------------------------------------------------------

class _Program:
    """The handle and the streams of a program that calls the library."""

    def __init__(self):
        self.handle = alt.Handle()
        self.streams = [torch.cuda.Stream() for _ in range(5)]


_program = None


def _the_program():
    global _program
    if _program is None:
        _program = _Program()
    return _program


class _Maker:
    def __init__(self, seed, dtype):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed))
        self.dtype = dtype

    def normal(self, count, std=1.0, dtype=None):
        """Random normal values; large tensors are drawn in pieces, so that the 32-bit values fit beside them."""
        out = torch.empty(int(count), dtype=dtype or self.dtype, device="cuda")
        step = 1 << 26
        for at in range(0, out.numel(), step):
            piece = out[at:at + step]
            piece.copy_(torch.randn(piece.numel(), generator=self.gen, device="cuda").mul_(std))
        return out

    def empty(self, count, dtype=None):
        return torch.empty(int(count), dtype=dtype or self.dtype, device="cuda")


def _workspace(nbytes):
    return (torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None), nbytes


def _conv_operands(h, make, d, bias):
    """Input, packed weights, bias, output and workspace of one convolution."""
    g = max(1, d.groups)
    w = make.normal(d.K * (d.C // g) * d.R * d.S, 0.05)
    packed = torch.empty_like(w)
    h.pack_weights(d, w, packed)
    ws, nb = _workspace(h.conv2d_workspace_size(d))
    return dict(w=packed, bias=make.normal(d.K, 0.1, torch.float32) if bias else None,
                y=make.empty(math.prod(h.conv2d_output_shape(d))), workspace=ws, ws_bytes=nb)


def prepare(case, seed):
    prog = _the_program()
    h, kind = prog.handle, case["kind"]
    code, dtype, _ = _FIELDS[case.get("dtype", "bf16")]
    make = _Maker(seed, dtype)
    state = {"kind": kind, "h": h}

    def conv(N, C, H, K, R, **options):
        layout = options.pop("layout", "NHWC")
        lay = dict(x_layout="NCHW->" + layout, w_layout="OIHW->OHWI" if layout == "NHWC" else "OIHW->OIHW", y_layout="NCHW->" + layout)
        lay.update(options)
        return alt.conv_desc(N, C, H, H, K, R, R, in_dtype=code, out_dtype=code, **lay)

    if kind == "layers":
        calls = []
        for i, (C, s, K, r, pad) in enumerate(_layers(case)):
            d = conv(case["batch"], C, s, K, r, pad=pad, layout=case["layout"])
            call = dict(d=d, x=make.normal(case["batch"] * C * s * s), **_conv_operands(h, make, d, False))
            if case["streams"]:
                call["stream"] = prog.streams[i]
            calls.append(call)
        state.update(go=h.conv2d_multi_prepared(calls), out=[c["y"] for c in calls])
    elif kind == "stem":
        n, K, s = case["batch"], case["channels"], case["size"]
        d = conv(n, 3, s, K, 7, stride=2, pad=3, epilogue=alt.EPI_BIAS | alt.EPI_RELU, x_layout="NCHW->NCHW")
        call = dict(d=d, x=make.normal(n * 3 * s * s), **_conv_operands(h, make, d, True))
        state.update(go=h.conv2d_prepared(**call), out=call["y"])
    elif kind in ("encoder", "product"):
        calls = []
        for b, m, n, k, lay in _products(case):
            d = alt.gemm_desc(m, n, k, batch=b, in_dtype=code, out_dtype=code, b_layout=lay)
            ws, nb = _workspace(h.gemm_workspace_size(d))
            calls.append(dict(d=d, A=make.normal(b * m * k), B=make.normal(b * k * n, 0.05), C=make.empty(b * m * n), workspace=ws, ws_bytes=nb))
        state.update(calls=calls)
    elif kind == "convert":
        lay = {p: alt.layout_parse("NCHW->" + p) for p in ("NCHW", "NHWC", "NCHW16c")}
        calls, out = [], []
        for shape in _tensors(case):
            x = make.normal(math.prod(shape))
            to = [torch.empty_like(x) for _ in range(3)]
            calls += [(code, shape, lay["NCHW"], x, lay["NHWC"], to[0]), (code, shape, lay["NCHW"], x, lay["NCHW16c"], to[1]),
                      (code, shape, lay["NHWC"], x, lay["NCHW"], to[2])]
            out += to
        state.update(calls=calls, out=out)
    elif kind == "mobile":
        n, C, s = case["batch"], case["C"], case["size"]
        E = C * case["expand"]
        x, y = make.normal(n * s * s * C), make.empty(n * s * s * C)
        relu = alt.EPI_BIAS | alt.EPI_RELU
        descs = [conv(n, C, s, E, 1, epilogue=relu), conv(n, E, s, E, 3, pad=1, groups=E, epilogue=relu), conv(n, E, s, C, 1, epilogue=alt.EPI_BIAS)]
        calls, at = [], x
        for d in descs:
            calls.append(dict(d=d, x=at, **_conv_operands(h, make, d, True)))
            at = calls[-1]["y"]
        state.update(go=[h.conv2d_prepared(**c) for c in calls], add=(code, x.numel(), at, x, y), out=[c["y"] for c in calls] + [y])
    else:
        n, C, D, s = case["batch"], case["C"], case["depth"], case["size"]
        K = C // 2
        lay = dict(x_layout="NCHW->NHWC", w_layout="OIHW->OHWI", y_layout="NCHW->NHWC", in_dtype=code, out_dtype=code)
        d3 = alt.conv3d_desc(n, C, D, s, s, C, 3, 3, 3, stride=1, pad=1, **lay)
        t2 = alt.conv_desc(n * D, C, s, s, K, 4, 4, stride=2, pad=1, **lay)
        t3 = alt.conv3d_desc(n, C, D, s, s, K, 4, 4, 4, stride=2, pad=1, **lay)
        w3, w2, w4 = (make.normal(v, 0.05) for v in (27 * C * C, 16 * C * K, 64 * C * K))
        p3 = torch.empty_like(w3)
        p2, p4 = make.empty(math.prod(h.conv2d_transpose_weight_shape(t2))), make.empty(math.prod(h.conv3d_transpose_weight_shape(t3)))
        h.pack_weights3d(d3, w3, p3)
        h.pack_weights_transpose(t2, w2, p2)
        h.pack_weights3d_transpose(t3, w4, p4)
        calls = []
        for fn, size, shape, d, p in ((h.conv3d, h.conv3d_workspace_size, h.conv3d_output_shape, d3, p3),
                                      (h.conv2d_transpose, h.conv2d_transpose_workspace_size, h.conv2d_transpose_output_shape, t2, p2),
                                      (h.conv3d_transpose, h.conv3d_transpose_workspace_size, h.conv3d_transpose_output_shape, t3, p4)):
            ws, nb = _workspace(size(d))
            calls.append((fn, dict(d=d, x=make.normal(n * D * s * s * C), w=p, y=make.empty(math.prod(shape(d))), workspace=ws, ws_bytes=nb)))
        state.update(calls=calls)
    return state


def run(state):
    kind, h = state["kind"], state["h"]
    if kind in ("layers", "stem"):
        state["go"]()
        return state["out"]
    if kind in ("encoder", "product"):
        for c in state["calls"]:
            h.gemm(**c)
        return [c["C"] for c in state["calls"]]
    if kind == "convert":
        for c in state["calls"]:
            h.layout_transform(*c)
        return state["out"]
    if kind == "mobile":
        for go in state["go"]:
            go()
        h.eltwise_add(*state["add"])
        return state["out"]
    for fn, c in state["calls"]:
        fn(**c)
    return [c["y"] for _, c in state["calls"]]
