"""NaN and infinite operands: they reach exactly the outputs whose sums contain them, as what the sum makes of them, on every
kernel variant and with every element type.  The finite operands are small integers, so the comparison is exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2210_12415_amd as alt
from gpu_util import applicable_variants, canary_dev, canary_ok, dev, from_layout, host, to_layout
from workloads import f32_to_bf16_bits, small_ints_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    return alt.Handle()


def f32(a):
    return (a.astype(np.uint32) << 16).view(np.float32) if a.dtype == np.uint16 else a


def conv(h, d, x, w, b, layouts, ref):
    """One convolution of the logical arrays; whether the result is the reference's, NaN for NaN."""
    bits = lambda a: f32_to_bf16_bits(a) if d.in_dtype == alt.BF16 else a
    np_out = np.uint16 if d.out_dtype == alt.BF16 else np.float32
    whole, y = canary_dev(ref.size, np_out)
    ws_bytes = h.conv2d_workspace_size(d)
    h.conv2d(d, dev(to_layout(bits(x), "NCHW", layouts[0])), dev(to_layout(bits(w), "OIHW", layouts[1])), y, bias=dev(b),
             workspace=dev(np.zeros(max(1, ws_bytes // 4), np.float32)), ws_bytes=ws_bytes)
    got = f32(from_layout(host(y, np_out), ref.shape, "NCHW", layouts[2]))
    return canary_ok(whole, ref.size) and np.array_equal(got, f32(ref), equal_nan=True)


@pytest.mark.parametrize("out_dtype", [alt.BF16, alt.F32])
@pytest.mark.parametrize("N,C,H,W,K,R,stride,dtype,layouts", [
    (2, 64, 9, 7, 64, 3, 1, alt.BF16, ("NHWC", "OHWI", "NHWC")), (1, 24, 9, 8, 40, 3, 1, alt.BF16, ("NHWC", "OHWI", "NHWC")),
    (2, 128, 6, 7, 64, 1, 1, alt.BF16, ("NHWC", "OHWI", "NHWC")), (1, 64, 9, 8, 32, 3, 1, alt.BF16, ("NCHW", "OIHW", "NCHW")),
    (1, 64, 8, 7, 64, 3, 1, alt.BF16, ("NCHW16c", "OHWI", "NCHW16c")), (2, 3, 20, 23, 40, 7, 2, alt.BF16, ("NCHW", "OIHW", "NHWC")),
    (1, 72, 9, 8, 36, 3, 1, alt.F32, ("NHWC", "OHWI", "NHWC")), (1, 5, 9, 8, 7, 3, 2, alt.F32, ("NCHW", "OIHW", "NCHW"))])
def test_convolutions_keep_nan_and_infinity(h, N, C, H, W, K, R, stride, dtype, layouts, out_dtype):
    x, w = small_ints_f32(61, (N, C, H, W), -3, 3), small_ints_f32(62, (K, C, R, R), -3, 3)
    b = small_ints_f32(63, (K,), -20, 20)
    x[0, C // 2, 3, 2], x[N - 1, C - 1, H - 2, W - 2], b[K // 2] = np.nan, np.inf, np.nan
    ref = oracle.conv2d(x, w, stride=stride, pad=R // 2, bias=b, out_bf16=out_dtype == alt.BF16)
    assert 0 < np.isnan(f32(ref)).mean() < 0.9 and np.isinf(f32(ref)).any()
    d = alt.conv_desc(N, C, H, W, K, R, R, stride=stride, pad=R // 2, in_dtype=dtype, out_dtype=out_dtype, epilogue=alt.EPI_BIAS,
                      x_layout="NCHW->" + layouts[0], w_layout="OIHW->" + layouts[1], y_layout="NCHW->" + layouts[2])
    wrong = []
    for d.variant, name in [(-1, "default")] + applicable_variants(h, d):
        if not conv(h, d, x, w, b, layouts, ref):
            wrong.append(name)
    assert not wrong


@pytest.mark.parametrize("dtype", [alt.BF16, alt.F32])
def test_element_wise_sum_keeps_nan_and_infinity(h, dtype):
    n = 1037
    a, b = small_ints_f32(64, (n,), -30, 30), small_ints_f32(65, (n,), -30, 30)
    a[::7], b[::11], b[::13] = np.nan, np.inf, -np.inf
    with np.errstate(invalid="ignore"):
        ref = a + b
    bits = lambda v: f32_to_bf16_bits(v) if dtype == alt.BF16 else v
    np_t = np.uint16 if dtype == alt.BF16 else np.float32
    whole, y = canary_dev(n, np_t)
    h.eltwise_add(dtype, n, dev(bits(a)), dev(bits(b)), y)
    assert canary_ok(whole, n) and np.array_equal(f32(host(y, np_t)), ref, equal_nan=True)


# a filter value that meets nothing but the surroundings of the image leaves no trace at the border, whatever it is; one row, one
# column and one image corner per case are covered by no more than a tap or two
@pytest.mark.parametrize("out_dtype", [alt.BF16, alt.F32])
@pytest.mark.parametrize("wl", ["OHWI", "OIHW", "HWIO"])
@pytest.mark.parametrize("N,C,H,W,R,stride,pad", [(2, 24, 7, 9, 3, 1, 1), (2, 256, 65, 61, 3, 1, 1), (1, 16, 8, 13, 3, 2, 2), (2, 8, 6, 6, 5, 1, 2)])
def test_depthwise_taps_outside_the_image_do_not_count(h, N, C, H, W, R, stride, pad, wl, out_dtype):
    x, w = small_ints_f32(66, (N, C, H, W), -3, 3), small_ints_f32(67, (C, 1, R, R), -3, 3)
    b = small_ints_f32(68, (C,), -20, 20)
    w[::5, 0, 0, 0], w[1::5, 0, R - 1, R // 2], w[2::5, 0, R // 2, R - 1], x[0, C - 1, 2, 3] = np.inf, -np.inf, np.nan, np.nan
    ref = oracle.conv2d(x, w, stride=stride, pad=pad, groups=C, bias=b, out_bf16=out_dtype == alt.BF16)
    assert np.isinf(f32(ref)).any() and np.isnan(f32(ref)).any() and np.isfinite(f32(ref)[:, ::5]).any()
    layouts = ("NHWC", wl, "NHWC")
    d = alt.conv_desc(N, C, H, W, C, R, R, stride=stride, pad=pad, groups=C, in_dtype=alt.BF16, out_dtype=out_dtype, epilogue=alt.EPI_BIAS,
                      x_layout="NCHW->NHWC", w_layout="OIHW->" + wl, y_layout="NCHW->NHWC")
    assert conv(h, d, x, w, b, layouts, ref)


# ... and costs little: a launch whose NaN sums at the border were taken again one element at a time took 27 times as long as others.
# The bound leaves room for a second pass over the windows (9.9 and 22.5 us against 8.9 at 144 channels).
@pytest.mark.parametrize("C,H,stride,wl", [(144, 56, 1, "HWIO"), (144, 56, 1, "OHWI"), (96, 112, 2, "HWIO"), (96, 112, 2, "OHWI")])
def test_depthwise_nan_operands_are_not_slow(h, C, H, stride, wl):
    d = alt.conv_desc(16, C, H, H, C, 3, 3, stride=stride, pad=1, groups=C, in_dtype=alt.BF16, out_dtype=alt.BF16, epilogue=alt.EPI_BIAS,
                      x_layout="NCHW->NHWC", w_layout="OIHW->" + wl, y_layout="NCHW->NHWC")
    y, b = torch.empty(16 * C * (H // stride) ** 2, dtype=torch.int16, device="cuda"), torch.zeros(C, device="cuda")
    x, w = [torch.randn(n, device="cuda").bfloat16() for n in (16 * C * H * H, C * 9)]

    def fastest():
        us = []
        for _ in range(12):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                h.conv2d(d, x.view(torch.int16), w.view(torch.int16), y, bias=b)
            end.record()
            end.synchronize()
            us.append(start.elapsed_time(end) * 100)
        return min(us)

    plain = fastest()
    x[::97] = float("nan")
    x_nan = fastest()
    w[:] = float("nan")
    w_nan = fastest()
    assert y.view(torch.bfloat16).isnan().all()
    assert x_nan < 2 * plain and w_nan < 5 * plain, (plain, x_nan, w_nan)
