"""GPU parity at the edges of the kernels' ranges: remainders of tiles, the smallest and the largest extents, every branch
of a dispatch rule.  Integer-valued inputs make every partial sum exact, so results are compared bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2210_12415_amd as alt
from gpu_util import applicable_variants, canary_dev, canary_ok, dev, from_layout, host, to_layout
from workloads import f32_to_bf16_bits, small_ints_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    return alt.Handle()


def check_conv(h, N, C, H, W, K, R, stride=1, pad=0, dil=1, groups=1, layouts=("NHWC", "OHWI", "NHWC"), dtype=alt.BF16,
               out_dtype=None, epilogue=True, variant=-1, S=None):
    """One convolution of small integers under the library's own choice of kernel (or `variant`), against the oracle."""
    S = R if S is None else S
    out_dtype = dtype if out_dtype is None else out_dtype
    bits = lambda a: f32_to_bf16_bits(a) if dtype == alt.BF16 else a
    x, w = small_ints_f32(41, (N, C, H, W), -3, 3), small_ints_f32(42, (K, C // groups, R, S), -3, 3)
    b = small_ints_f32(43, (K,), -20, 20)
    more = dict(bias=b, relu=True) if epilogue else {}
    ref = oracle.conv2d(x, w, stride=stride, pad=pad, dil=dil, groups=groups, out_bf16=out_dtype == alt.BF16, **more)
    xl, wl, yl = layouts
    d = alt.conv_desc(N, C, H, W, K, R, S, stride=stride, dil=dil, in_dtype=dtype, out_dtype=out_dtype, groups=groups,
                      epilogue=alt.EPI_BIAS | alt.EPI_RELU if epilogue else 0, variant=variant, x_layout="NCHW->" + xl,
                      w_layout="OIHW->" + wl, y_layout="NCHW->" + yl)
    d.pad_h, d.pad_w = pad if isinstance(pad, tuple) else (pad, pad)
    np_out = np.uint16 if out_dtype == alt.BF16 else np.float32
    whole, y = canary_dev(ref.size, np_out)
    ws_bytes = h.conv2d_workspace_size(d)
    ws = dev(np.zeros(max(1, ws_bytes // 4), np.float32))
    print("conv", N, C, H, W, K, R, S, stride, pad, dil, groups, layouts, flush=True)
    h.conv2d(d, dev(to_layout(bits(x), "NCHW", xl)), dev(to_layout(bits(w), "OIHW", wl)), y, bias=dev(b) if epilogue else None,
             workspace=ws if ws_bytes else None, ws_bytes=ws_bytes)
    got = from_layout(host(y, np_out), ref.shape, "NCHW", yl)
    assert canary_ok(whole, ref.size), "wrote outside y"
    assert np.array_equal(got, ref)


# widths of 4 * n and with one column over, one or two rows per thread (two from 65536 threads on), an odd last row, one
# vector of channels; 5x5 runs on the general vector kernel
@pytest.mark.parametrize("N,C,H,W,R,stride,pad", [
    (2, 8, 7, 9, 3, 1, 1), (1, 24, 6, 4, 3, 1, (0, 1)), (2, 256, 65, 61, 3, 1, 1), (3, 40, 8, 13, 3, 2, 1), (1, 16, 3, 3, 3, 1, 0),
    (2, 24, 9, 10, 5, 1, 2), (1, 72, 11, 7, 3, 2, (1, 0))])
@pytest.mark.parametrize("wl", ["OHWI", "OIHW", "HWIO"])
def test_depthwise_vector_kernels(h, N, C, H, W, R, stride, pad, wl):
    check_conv(h, N, C, H, W, C, R, stride, pad, groups=C, layouts=("NHWC", wl, "NHWC"))


TAPS_CASES = [
    # N, C, H, W, K, R, S, stride, pad, dil
    (2, 64, 9, 7, 64, 3, 3, 1, 1, 1),          # one K step per tap, rows that end inside a tile
    (1, 24, 12, 11, 40, 3, 3, 1, 1, 1),        # a chunk column crosses taps inside a K step
    (3, 8, 5, 6, 12, 3, 3, 2, 1, 1),           # one chunk per tap, stride 2, narrow output
    (2, 40, 10, 9, 72, 1, 1, 1, 0, 1),         # 1x1, K of 1.25 steps
    (2, 24, 7, 9, 144, 1, 1, 2, 0, 1),         # 1x1 at stride 2
    (1, 96, 8, 8, 100, 5, 5, 1, 4, 2),         # dilation, more padding than same-size
    (1, 128, 6, 5, 256, 1, 7, 1, (0, 3), 1),   # one-dimensional filter
    (1, 16, 4, 4, 32, 3, 3, 1, 8, 8),          # a filter that reaches past the whole image
    (1, 192, 16, 15, 132, 3, 3, 1, 1, 1),
    (4, 160, 1, 1, 36, 1, 1, 1, 0, 1),         # a handful of rows
]


@pytest.mark.parametrize("dtype", [alt.BF16, alt.F32])
@pytest.mark.parametrize("case", TAPS_CASES, ids=lambda c: "_".join(str(v) for v in c))
def test_tap_kernels_every_variant(h, case, dtype):
    """The streaming kernels over filter taps (names with _taps_ or _rtaps_): every tile shape that takes the problem, without
    and with the smallest split-K factor, bit for bit."""
    N, C, H, W, K, R, S, stride, pad, dil = case
    d = alt.conv_desc(N, C, H, W, K, R, S, stride=stride, dil=dil, in_dtype=dtype, out_dtype=dtype, x_layout="NCHW->NHWC",
                      w_layout="OIHW->OHWI", y_layout="NCHW->NHWC")
    d.pad_h, d.pad_w = pad if isinstance(pad, tuple) else (pad, pad)
    seen = set()
    for v, name in applicable_variants(h, d):
        base, k = name.rsplit("_k", 1)
        if "taps_" not in name or (base, k != "1") in seen:
            continue
        seen.add((base, k != "1"))
        check_conv(h, N, C, H, W, K, R, stride, pad, dil, S=S, dtype=dtype, variant=v)
    assert len(seen) >= 3


@pytest.mark.parametrize("bl", ["NK", "KN"])
@pytest.mark.parametrize("M,N,K", [(70, 64, 8), (129, 136, 72), (37, 200, 1304), (300, 72, 104)])
def test_products_with_ragged_depth_every_variant(h, bl, M, N, K):
    """Products whose K is no multiple of a K step on the kernels named _rtaps_ (B as NK) and _rtapskn_ (B as KN)."""
    A, B = small_ints_f32(51, (M, K), -3, 3), small_ints_f32(52, (K, N), -3, 3)
    ref = oracle.gemm(A, B)
    a, b = dev(f32_to_bf16_bits(A)), dev(f32_to_bf16_bits(np.ascontiguousarray(B.T) if bl == "NK" else B))
    d = alt.gemm_desc(M, N, K, b_layout="KN->" + bl)
    seen = 0
    for v, name in applicable_variants(h, d, "gemm"):
        if "rtaps" not in name:
            continue
        seen += 1
        d.variant = v
        ws_bytes = h.gemm_workspace_size(d)
        whole, C = canary_dev(M * N, np.float32)
        print("gemm", M, N, K, bl, name, flush=True)
        h.gemm(d, a, b, C, workspace=dev(np.zeros(max(1, ws_bytes // 4), np.float32)), ws_bytes=ws_bytes)
        got = host(C, np.float32).reshape(M, N)
        assert canary_ok(whole, M * N) and np.array_equal(got, ref), name
    assert seen >= 4


# tiles that end inside an image in both directions, one to four channels, odd and even strides (odd ones read a second, shifted
# copy of the patch), filters of one to eight columns, output channels that leave part of a 32-channel tile empty
@pytest.mark.parametrize("N,C,H,W,K,R,S,stride,pad", [
    (2, 3, 37, 41, 64, 7, 7, 2, 3), (1, 3, 16, 16, 8, 3, 3, 2, 1), (1, 1, 9, 50, 40, 5, 5, 1, 2), (2, 4, 33, 20, 96, 3, 3, 1, 1),
    (1, 3, 70, 66, 104, 7, 7, 2, 3), (1, 2, 21, 23, 32, 3, 8, 2, 4), (3, 3, 8, 8, 64, 1, 1, 1, 0), (1, 2, 40, 36, 48, 5, 6, 3, 0)])
@pytest.mark.parametrize("wl,yl", [("OHWI", "NHWC"), ("OIHW", "NCHW8c")])
def test_few_channel_kernels_every_variant(h, N, C, H, W, K, R, S, stride, pad, wl, yl):
    d = alt.conv_desc(N, C, H, W, K, R, S, stride=stride, pad=pad, in_dtype=alt.BF16, out_dtype=alt.BF16, w_layout="OIHW->" + wl,
                      y_layout="NCHW->" + yl)
    few = [v for v, n in applicable_variants(h, d) if "_few_" in n]
    assert few and "_few_" in h.conv2d_variant_name(d, -1)
    for v in few:
        check_conv(h, N, C, H, W, K, R, stride, pad, S=S, layouts=("NCHW", wl, yl), variant=v)
