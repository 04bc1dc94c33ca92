"""alt_conv2d_multi: independent convolutions on one stream go out as one launch (csrc/group.h).  Small integers, so that every sum is exact
whatever its order: bit for bit the oracle's."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2210_12415_amd as alt
from gpu_util import canary_dev, canary_ok, dev, from_layout, host, kernels_run, to_layout
from workloads.inputs import f32_to_bf16_bits, small_ints_f32

pytestmark = pytest.mark.gpu

RELU = alt.EPI_BIAS | alt.EPI_RELU
# N, C, H, W, K, filter, padding, epilogue[, stride, dilation]
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


# Lists that bring the tile bodies which those above do not (test_group_plan_cpu.py holds them to it), strides and dilations.
MORE = {
    ("f32", "NHWC"): [
        # whole 64-row tiles of one tap, alone and in slices; of nine taps in one slice
        [(2, 16, 12, 95, 88, 1, 0, RELU), (7, 160, 3, 3, 8, 1, 0, 0, 2), (3, 128, 3, 3, 116, 1, 0, RELU)],
        [(7, 48, 5, 56, 8, 3, 1, 0), (7, 8, 20, 34, 48, 3, 1, 0)],
        [(2, 8, 21, 53, 12, 3, 2, RELU, 2, 2), (2, 96, 20, 27, 40, 1, 0, RELU), (1, 32, 17, 23, 64, 3, 2, 0, 1, 2)]],
    ("bf16", "NHWC"): [
        # K groups with few loads of a patch; tall tiles with many; one tap in slices
        [(7, 152, 18, 77, 8, 1, 0, RELU), (8, 144, 5, 5, 104, 1, 0, RELU, 2), (8, 248, 14, 4, 4, 3, 1, 0)],
        [(4, 256, 27, 39, 68, 1, 0, RELU, 2), (3, 8, 34, 102, 16, 3, 1, 0), (6, 56, 6, 6, 40, 1, 0, RELU)],
        [(8, 32, 10, 10, 48, 1, 0, 0), (8, 168, 7, 7, 16, 1, 0, RELU)],
        [(1, 8, 36, 36, 80, 3, 2, 0, 1, 2), (1, 40, 17, 17, 80, 1, 0, RELU)],
        [(1, 40, 20, 20, 16, 3, 2, RELU, 1, 2), (8, 64, 6, 6, 40, 1, 0, RELU)]],
    ("bf16", "NCHW"): [
        # 256 rows of one tap and of nine; the smallest tile of one tap
        [(1, 248, 3, 3, 96, 3, 1, RELU), (8, 80, 5, 5, 48, 1, 0, RELU), (4, 48, 9, 9, 32, 1, 0, 0)],
        [(3, 56, 5, 46, 62, 3, 1, 0), (2, 256, 38, 6, 128, 3, 1, 0, 2)],
        [(2, 136, 4, 7, 120, 1, 0, RELU), (8, 48, 6, 6, 15, 1, 0, RELU, 2)],
        [(4, 160, 12, 12, 24, 1, 0, 0), (1, 48, 3, 3, 136, 3, 2, RELU, 1, 2)]],
}


@pytest.fixture(scope="module")
def h():
    return alt.Handle()


def describe(dtype, layout, problem, out):
    """The problem's descriptor and the elements of its workspace."""
    N, C, H, W, K, R, pad, epi, stride, dil = problem + (1, 1)[len(problem) - 8:]
    code = alt.F32 if dtype == "f32" else alt.BF16
    d = alt.conv_desc(N, C, H, W, K, R, R, stride=stride, pad=pad, dil=dil, in_dtype=code, out_dtype=out, epilogue=epi, x_layout="NCHW->" + layout,
                      w_layout="OIHW->" + ("OHWI" if layout == "NHWC" else "OIHW"), y_layout="NCHW->" + layout)
    size = lambda e: (e + 2 * pad - dil * (R - 1) - 1) // stride + 1
    return d, 36 * N * K * size(H) * size(W)


def make(h, dtype, layout, problems, seed, out=alt.F32):
    np_out = np.float32 if out == alt.F32 else np.uint16
    bits = (lambda a: a) if dtype == "f32" else f32_to_bf16_bits
    wl = "OHWI" if layout == "NHWC" else "OIHW"
    calls, refs, outs = [], [], []
    for i, problem in enumerate(problems):
        N, C, H, W, K, R, pad, epi, stride, dil = problem + (1, 1)[len(problem) - 8:]
        x, w = small_ints_f32(seed + i, (N, C, H, W), -2, 2), small_ints_f32(seed + 50 + i, (K, C, R, R), -2, 2)
        b = small_ints_f32(seed + 90 + i, (K,), -4, 4)
        ref = oracle.conv2d(x, w, stride=stride, pad=pad, dil=dil)
        if epi:
            ref = np.maximum(ref + b[None, :, None, None], 0)
        d, ws_elems = describe(dtype, layout, problem, out)
        n = ref.size
        whole, y = canary_dev(n, np_out)
        ws = torch.empty(ws_elems, dtype=torch.float32, device="cuda")
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


@pytest.mark.parametrize("kind,which", [(k, i) for k, l in MORE.items() for i in range(len(l))], ids=lambda v: v if isinstance(v, int) else "_".join(v))
def test_every_tile_body(h, kind, which):
    dtype, layout = kind
    calls, refs, outs = make(h, dtype, layout, MORE[kind][which], 7100 + 10 * which, alt.BF16 if dtype == "bf16" else alt.F32)
    run = h.conv2d_multi_prepared(calls)
    run()
    names = kernels_run(run)
    assert len(names) == 1 and "group_kernel" in names[0], names
    check(calls, refs, outs, layout)
    assert h.splitk_status().counters_nonzero == 0


def test_more_lists_than_are_kept(h):
    """Seventy lists in turn, twice: 64 launches are kept."""
    N, C, K = 1, 16, 24
    x, w = small_ints_f32(7200, (N, C, 80, 5), -2, 2), small_ints_f32(7201, (K, C, 3, 3), -2, 2)
    refs = [oracle.conv2d(x[:, :, :4 + i], w, pad=1) for i in range(71)]
    xs = [dev(to_layout(f32_to_bf16_bits(np.ascontiguousarray(x[:, :, :4 + i])), "NCHW", "NHWC")) for i in range(71)]
    wd = dev(to_layout(f32_to_bf16_bits(w), "OIHW", "OHWI"))
    y = [torch.empty(refs[70].size, dtype=torch.float32, device="cuda") for _ in range(2)]
    descs = [alt.conv_desc(N, C, 4 + i, 5, K, 3, 3, pad=1, in_dtype=alt.BF16, out_dtype=alt.F32, x_layout="NCHW->NHWC", w_layout="OIHW->OHWI",
                           y_layout="NCHW->NHWC") for i in range(71)]
    for again in (0, 1):
        for i in range(70):
            calls = [dict(d=descs[i + j], x=xs[i + j], w=wd, y=y[j][:refs[i + j].size]) for j in (0, 1)]
            h.conv2d_multi(calls)
            if i % 23 == 0:
                assert [p.family for p in h.conv2d_multi_plan(calls)] == [2, 2]
            for j in (0, 1):
                assert np.array_equal(from_layout(host(calls[j]["y"], np.float32), refs[i + j].shape, "NCHW", "NHWC"), refs[i + j]), (again, i, j)


def test_sliced_lists_without_a_free_counter_set(h):
    """Every counter set bound to a stream, and a list whose sums are planned in slices under capture on one more: its calls go out one by one, unsliced."""
    hip = ctypes.CDLL("libamdhip64.so")

    def stream():
        out = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(out), 1) == 0
        return torch.cuda.ExternalStream(out.value)

    calls, refs, outs = make(h, "f32", "NHWC", SETS["f32", "NHWC"], 7250)
    streams = []
    while h.splitk_status().streams_bound < 64:
        streams.append(stream())
        for c in calls:
            c["stream"] = streams[-1]
        h.conv2d_multi(calls)
        streams[-1].synchronize()
    assert any(p.slices > 1 for p in h.conv2d_multi_plan(calls))
    side = stream()
    for c in calls:
        c["stream"] = side
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        h.conv2d_multi(calls)
    for _ in range(3):
        for c in calls:
            c["y"].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        check(calls, refs, outs, "NHWC")
    h.conv2d_multi(calls)                       # outside capture: the sets are released
    torch.cuda.synchronize()
    check(calls, refs, outs, "NHWC")
    st = h.splitk_status()
    assert st.streams_bound < 64 and st.counters_nonzero == 0


def test_a_tuned_call_runs_its_kernel():
    """A list beside a tuned problem goes out one by one, with the tuned kernel, and together again when the plans are cleared."""
    h = alt.Handle()
    calls, refs, outs = make(h, "bf16", "NHWC", [(1, 16 + 8 * i, 10, 10, 24, 3, 1, 0) for i in range(3)], 7270)
    assert len(kernels_run(h.conv2d_multi_prepared(calls))) == 1
    arena = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    tuned = alt.ConvDesc.from_buffer_copy(bytes(calls[1]["d"]))
    h.tune_conv2d_variants(tuned, arena, arena.numel(), max_trials=12, warmup=1, reps=3)
    for clear in (False, True):
        if clear:
            h.cache_clear()
        for c in calls:
            c["y"].zero_()
        names = kernels_run(h.conv2d_multi_prepared(calls))
        assert any("group_kernel" in n for n in names) == clear and (len(names) == 1 if clear else len(names) >= 3), names
        check(calls, refs, outs, "NHWC")


@pytest.mark.parametrize("kind", [("f32", "NHWC"), ("bf16", "NCHW")], ids="_".join)
def test_chains_in_the_other_families(h, kind):
    dtype, layout = kind
    out, bits = (alt.F32, np.float32) if dtype == "f32" else (alt.BF16, np.uint16)
    calls, _, _ = make(h, dtype, layout, [(2, 32, 12, 12, 32, 3, 1, 0)] * 3, 7350, out)
    for i in (1, 2):
        calls[i]["x"] = calls[i - 1]["y"]
    assert len(kernels_run(h.conv2d_multi_prepared(calls))) == 3
    got = [host(c["y"], bits).copy() for c in calls]
    for c in calls:
        c["y"].zero_()
        h.conv2d(**c)
    for c, g in zip(calls, got):
        assert np.array_equal(host(c["y"], bits), g)


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
