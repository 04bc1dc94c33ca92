"""alt_conv2d_multi: independent convolutions on one stream go out as one launch (csrc/group.h).  Small integers, so that every sum is exact
whatever its order: bit for bit the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2210_12415_amd as alt
from gpu_util import canary_dev, canary_ok, dev, from_layout, host, kernels_run, to_layout
from workloads.inputs import f32_to_bf16_bits, small_ints_f32

pytestmark = pytest.mark.gpu

RELU = alt.EPI_BIAS | alt.EPI_RELU
# N, C, H, W, K, filter, padding, epilogue
SETS = {
    # tiles of 64 and 32 columns, one and many taps, sums in slices, rows and columns that end inside a tile
    ("f32", "NHWC"): [(1, 16, 9, 11, 24, 3, 1, 0), (3, 64, 14, 14, 64, 3, 1, RELU), (1, 256, 7, 7, 96, 3, 1, 0), (2, 48, 13, 10, 20, 1, 0, RELU),
                      (1, 4, 5, 5, 4, 3, 0, 0)],
    # slabs with few and many loads of a patch (wide images), K groups (deep layers of few pixels), ragged channels, one tap
    ("bf16", "NHWC"): [(1, 8, 9, 11, 24, 3, 1, 0), (2, 72, 6, 150, 64, 3, 1, RELU), (1, 256, 7, 7, 96, 3, 1, 0), (3, 40, 13, 10, 20, 1, 0, RELU),
                       (1, 64, 30, 60, 64, 3, 1, 0), (1, 16, 5, 100, 8, 3, 0, 0), (20, 24, 20, 20, 128, 1, 0, 0), (1, 8, 1, 1, 4, 1, 0, 0)],
    # whole and broken super-steps, both filters, planes that do not begin at eight pixels
    ("bf16", "NCHW"): [(1, 8, 9, 11, 24, 3, 1, 0), (2, 72, 14, 30, 64, 3, 1, RELU), (1, 256, 7, 7, 96, 3, 1, 0), (3, 40, 13, 10, 20, 1, 0, RELU),
                       (2, 128, 17, 17, 33, 1, 0, 0), (4, 64, 40, 40, 64, 3, 1, 0)],
}


@pytest.fixture(scope="module")
def h():
    return alt.Handle()


def make(h, dtype, layout, problems, seed, out=alt.F32):
    code = alt.F32 if dtype == "f32" else alt.BF16
    np_out = np.float32 if out == alt.F32 else np.uint16
    bits = (lambda a: a) if dtype == "f32" else f32_to_bf16_bits
    wl = "OHWI" if layout == "NHWC" else "OIHW"
    calls, refs, outs = [], [], []
    for i, (N, C, H, W, K, R, pad, epi) in enumerate(problems):
        x, w = small_ints_f32(seed + i, (N, C, H, W), -2, 2), small_ints_f32(seed + 50 + i, (K, C, R, R), -2, 2)
        b = small_ints_f32(seed + 90 + i, (K,), -4, 4)
        ref = oracle.conv2d(x, w, stride=1, pad=pad)
        if epi:
            ref = np.maximum(ref + b[None, :, None, None], 0)
        d = alt.conv_desc(N, C, H, W, K, R, R, pad=pad, in_dtype=code, out_dtype=out, epilogue=epi, x_layout="NCHW->" + layout,
                          w_layout="OIHW->" + wl, y_layout="NCHW->" + layout)
        n = ref.size
        whole, y = canary_dev(n, np_out)
        ws = torch.empty(36 * n, dtype=torch.float32, device="cuda")
        calls.append(dict(d=d, x=dev(to_layout(bits(x), "NCHW", layout)), w=dev(to_layout(bits(w), "OIHW", wl)), bias=dev(b) if epi else None,
                          y=y, workspace=ws, ws_bytes=ws.numel() * 4))
        refs.append(ref if out == alt.F32 else f32_to_bf16_bits(ref))
        outs.append((whole, np_out))
    return calls, refs, outs


def check(calls, refs, outs, layout):
    for c, ref, (whole, np_out) in zip(calls, refs, outs):
        assert canary_ok(whole, ref.size), "wrote outside y"
        assert np.array_equal(from_layout(host(c["y"], np_out), ref.shape, "NCHW", layout), ref)


@pytest.mark.parametrize("out", [alt.F32, alt.BF16], ids=["to_f32", "to_bf16"])
@pytest.mark.parametrize("kind", list(SETS), ids="_".join)
def test_one_launch_for_independent_convolutions(h, kind, out):
    dtype, layout = kind
    calls, refs, outs = make(h, dtype, layout, SETS[kind], 7000, out)
    run = h.conv2d_multi_prepared(calls)
    run()
    names = kernels_run(run)
    assert len(names) == 1 and "group_kernel" in names[0], names
    check(calls, refs, outs, layout)
    assert h.splitk_status().counters_nonzero == 0
    # without a workspace no sum is sliced
    for c, (whole, _) in zip(calls, outs):
        c["y"].zero_()
        c["workspace"], c["ws_bytes"] = None, 0
    h.conv2d_multi(calls)
    check(calls, refs, outs, layout)
    # the same under capture, replayed with eager work between
    side = torch.cuda.Stream()
    for c in calls:
        c["stream"] = side
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        h.conv2d_multi(calls)
    for _ in range(3):
        for c in calls:
            c["y"].zero_()
        torch.cuda.synchronize()
        g.replay()
        check(calls, refs, outs, layout)


def test_calls_that_meet_run_one_after_the_other(h):
    """A call that reads another's output, or shares its output buffer, is issued behind it, as separate calls on the stream are."""
    calls, _, _ = make(h, "bf16", "NHWC", [(2, 32, 12, 12, 32, 3, 1, 0)] * 3, 7300, alt.BF16)
    calls[1]["x"] = calls[0]["y"]
    calls[2]["x"] = calls[1]["y"]
    run = h.conv2d_multi_prepared(calls)
    run()
    assert len(kernels_run(run)) == 3
    got = [host(c["y"], np.uint16).copy() for c in calls]
    for c in calls:
        c["y"].zero_()
        h.conv2d(**c)
    for c, g in zip(calls, got):
        assert np.array_equal(host(c["y"], np.uint16), g)
    shared = [calls[0], dict(calls[0])]
    assert len(kernels_run(h.conv2d_multi_prepared(shared))) == 2


def test_long_lists_explicit_and_failing_calls(h):
    """Nine calls are two launches; a call with a kernel of its own is issued by itself; a failing call stops the list behind the ones before it."""
    nine = [(1, 16 + 8 * i, 10, 10, 24, 3, 1, 0) for i in range(9)]
    calls, refs, outs = make(h, "bf16", "NHWC", nine, 7400)
    run = h.conv2d_multi_prepared(calls)
    run()
    assert len(kernels_run(run)) == 2
    check(calls, refs, outs, "NHWC")
    for c in calls:
        c["y"].zero_()
    bad = dict(calls[2], d=alt.conv_desc(1, 24, 8, 8, 16, 3, 3, pad=1, x_layout="NCHW->NCHW16c"))
    with pytest.raises(alt.AltError):
        h.conv2d_multi([calls[0], calls[1], bad, calls[3]])
    check(calls[:2], refs[:2], outs[:2], "NHWC")
    torch.cuda.synchronize()
    assert not calls[3]["y"].any()
    name = h.conv2d_variant_name(calls[4]["d"], -1)
    count = h.conv2d_variant_count(calls[4]["d"])
    def named(v):
        try:
            return h.conv2d_variant_name(calls[4]["d"], v)
        except alt.AltError:
            return None
    own = next(v for v in range(count) if named(v) == name)
    calls[4]["d"].variant = own
    run = h.conv2d_multi_prepared(calls[4:6])
    run()
    names = kernels_run(run)
    assert len(names) == 2 and not any("group_kernel" in n for n in names)
