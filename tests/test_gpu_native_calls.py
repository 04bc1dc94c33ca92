"""Repeated calls through the native module and through ctypes, on real tensors and streams: the same bits, on the stream that was asked for."""
import math

import pytest
import torch

import paper_2210_12415_amd as alt
from paper_2210_12415_amd import binding

pytestmark = pytest.mark.gpu

QUICK = [n for n in dir(binding) if n.startswith("_quick_")]


def calls(h):
    """name -> (arguments, output) of one call of each of the repeated entry points."""
    torch.manual_seed(5)
    bf = lambda *s: torch.randn(*s, device="cuda").bfloat16()
    new = lambda n: torch.empty(n, dtype=torch.bfloat16, device="cuda")
    nhwc = dict(in_dtype=alt.BF16, out_dtype=alt.BF16, x_layout="NCHW->NHWC", w_layout="OIHW->OHWI", y_layout="NCHW->NHWC")
    out = {}

    def operator(name, d, shape, weights):
        n = math.prod(shape)
        nb = getattr(h, name.replace("_prepared", "") + "_workspace_size")(d)
        out[name] = (dict(d=d, x=bf(2 * 16 * 6 * 9 * 9), w=bf(math.prod(weights)), y=new(n), bias=torch.randn(24, device="cuda"),
                          workspace=torch.empty(max(nb, 1), dtype=torch.uint8, device="cuda"), ws_bytes=nb), "y")

    c2 = alt.conv_desc(12, 16, 9, 9, 24, 3, 3, pad=1, epilogue=3, **nhwc)
    c3 = alt.conv3d_desc(2, 16, 6, 9, 9, 24, 3, 3, 3, pad=1, epilogue=1, **nhwc)
    for name in ("conv2d", "conv2d_prepared"):
        operator(name, c2, h.conv2d_output_shape(c2), (24, 9, 16))
    operator("conv2d_transpose", c2, h.conv2d_transpose_output_shape(c2), h.conv2d_transpose_weight_shape(c2))
    operator("conv3d", c3, h.conv3d_output_shape(c3), (24, 27, 16))
    operator("conv3d_transpose", c3, h.conv3d_transpose_output_shape(c3), h.conv3d_transpose_weight_shape(c3))
    g = alt.gemm_desc(37, 40, 64, in_dtype=alt.BF16, out_dtype=alt.BF16, b_layout="KN->NK")
    out["gemm"] = dict(d=g, A=bf(37 * 64), B=bf(40 * 64), C=new(37 * 40)), "C"
    out["eltwise_add"] = dict(dtype=alt.BF16, numel=5000, a=bf(5000), b=bf(5000), y=new(5000), relu=True), "y"
    out["layout_transform"] = dict(dtype=alt.BF16, shape=(2, 16, 9, 9), src_layout=alt.layout_parse("NCHW->NCHW"), src=bf(2 * 16 * 81),
                                   dst_layout=alt.layout_parse("NCHW->NHWC"), dst=new(2 * 16 * 81)), "dst"
    return out


NAMES = ["conv2d", "conv2d_prepared", "conv2d_transpose", "conv3d", "conv3d_transpose", "gemm", "eltwise_add", "layout_transform"]


@pytest.mark.skipif(binding._native is None, reason="the native module is not built")
@pytest.mark.parametrize("name", NAMES)
def test_native_and_ctypes_calls_agree(name, monkeypatch):
    h = alt.Handle()
    kw, key = calls(h)[name]
    inputs = {k: v.clone() for k, v in kw.items() if isinstance(v, torch.Tensor) and k not in (key, "workspace")}
    side = torch.cuda.Stream()
    big = torch.randn(3000, 3000, device="cuda")
    binding._stream_address(None)             # (the first call for the current stream goes through ctypes, which finds out how to ask for it)
    results = []
    for native in (True, False):
        taken = []
        for n in QUICK:
            f = getattr(binding, n)
            monkeypatch.setattr(binding, n, (lambda *a, f=f: taken.append(f(*a)) or taken[-1]) if native else binding._not_taken)
        for where in ("default", "current", "named"):
            torch.cuda.synchronize()
            kw[key].zero_()
            for k in inputs:
                kw[k].zero_()
            torch.cuda.synchronize()
            on = side if where != "default" else torch.cuda.default_stream()
            with torch.cuda.stream(on):
                for _ in range(6):
                    big = big @ big * 1e-4                 # the inputs are written behind milliseconds of work on the call's stream
                for k, v in inputs.items():
                    kw[k].copy_(v)
                run = getattr(h, name)
                if where == "current" or where == "default":
                    r = run(**kw)
                    r() if name == "conv2d_prepared" else None
            if where == "named":
                r = run(**kw, stream=side)
                r() if name == "conv2d_prepared" else None
            torch.cuda.synchronize()
            results.append(kw[key].clone())
        assert bool(taken) == native and all(t is not None for t in taken)
    assert results[0].float().abs().max() > 0
    for r in results[1:]:
        assert torch.equal(r, results[0])
