"""GPU parity at the edges of the kernels' ranges: remainders of tiles, the smallest and the largest extents, every branch
of a dispatch rule.  Integer-valued inputs make every partial sum exact, so results are compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2210_12415_amd as alt
from gpu_util import applicable_variants, canary_dev, canary_ok, dev, from_layout, host, kernels_run, panel_rows, tile_of, to_layout
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


# depth-wise filters beyond 3x3 on both sides of the rule that chooses between the vector and the element kernel
@pytest.mark.parametrize("N,C,H,W,R,stride,wl,kernel", [
    (1, 24, 9, 10, 5, 1, "OHWI", "elem"), (2, 40, 31, 30, 5, 2, "OIHW", "elem"), (3, 16, 9, 10, 5, 1, "OIHW", "vec8_kernel<true>"),
    (1, 32, 7, 12, 7, 1, "OHWI", "vec8_kernel<true>"), (4, 40, 51, 49, 5, 1, "OHWI", "vec8_kernel<true>"),
    (1, 24, 9, 10, 5, 1, "HWIO", "vec8_kernel<false>"), (4, 40, 51, 49, 5, 1, "HWIO", "vec8_kernel<false>")])
def test_depthwise_kernel_by_filter_layout_and_size(h, N, C, H, W, R, stride, wl, kernel):
    ran = kernels_run(lambda: check_conv(h, N, C, H, W, C, R, stride, R // 2, groups=C, layouts=("NHWC", wl, "NHWC")))
    assert [k for k in ran if "dwconv_" + kernel in k], ran


def test_depthwise_batch_of_more_than_2_gib(h):
    """257 images of 4 M elements: the register-tiled kernel takes them in two launches, each below 2 GiB; every image is what the
    same call makes of a part of the batch, and the images at the seam are the oracle's."""
    N, C, H = 257, 64, 256
    x = torch.empty(N * H * H * C, dtype=torch.bfloat16, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(45)
    for i in range(0, N, 32):
        part = x[i * H * H * C:(i + 32) * H * H * C]
        part.copy_(torch.randint(-3, 4, (part.numel(),), generator=gen, dtype=torch.int32, device="cuda"))
    w = small_ints_f32(46, (C, 1, 3, 3), -3, 3)
    wd, y = dev(f32_to_bf16_bits(to_layout(w, "OIHW", "OHWI"))), torch.empty_like(x)

    def call(first, count, out):
        d = alt.conv_desc(count, C, H, H, C, 3, 3, pad=1, groups=C, in_dtype=alt.BF16, out_dtype=alt.BF16, x_layout="NCHW->NHWC",
                          w_layout="OIHW->OHWI", y_layout="NCHW->NHWC")
        h.conv2d(d, x[first * H * H * C:], wd, out)

    ran = kernels_run(lambda: call(0, N, y))
    assert len(ran) == 2 and all("dwconv_vec8_3x3" in k for k in ran), ran
    for first, count in ((0, 128), (128, 129)):
        part = torch.empty(count * H * H * C, dtype=torch.bfloat16, device="cuda")
        call(first, count, part)
        assert torch.equal(part.view(torch.int16), y[first * H * H * C:(first + count) * H * H * C].view(torch.int16))
    for i in (0, 254, 255, 256):
        image = lambda t: host(t[i * H * H * C:(i + 1) * H * H * C].view(torch.int16), np.uint16)
        xi = from_layout(image(x), (1, C, H, H), "NCHW", "NHWC")
        ref = oracle.conv2d((xi.astype(np.uint32) << 16).view(np.float32), w, pad=1, groups=C, out_bf16=True)
        assert np.array_equal(from_layout(image(y), (1, C, H, H), "NCHW", "NHWC"), ref), i


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


@pytest.mark.parametrize("N,C,H,W,K,R,pad,dil,yl", [
    (2, 8, 9, 7, 12, 3, 1, 1, "NHWC"),         # one chunk of one slab, narrow output
    (3, 40, 10, 11, 72, 3, 1, 1, "NHWC"),      # a slab of eight channels behind a whole one
    (1, 104, 13, 12, 40, 3, 1, 1, "NCHW8c"),   # four slabs (two of 64), blocked output
    (2, 64, 17, 15, 132, 3, 0, 1, "NHWC"),     # no padding: patches of several images' ends
    (1, 72, 19, 18, 64, 3, 2, 2, "NHWC"),      # dilated, same-size
    (5, 96, 4, 4, 32, 3, 1, 1, "NHWC"),        # images smaller than a tile
    (2, 200, 8, 9, 36, 2, 0, 1, "NHWC"),       # 2x2 taps, seven slabs
    (1, 24, 3, 70, 20, 3, 1, 1, "NHWC"),       # long rows
    (1, 16, 1, 1, 16, 3, 1, 1, "NHWC")])       # one pixel, eight of nine taps outside
def test_slab_kernels_every_variant(h, N, C, H, W, K, R, pad, dil, yl):
    d = alt.conv_desc(N, C, H, W, K, R, R, pad=pad, dil=dil, in_dtype=alt.BF16, out_dtype=alt.BF16, x_layout="NCHW->NHWC",
                      w_layout="OIHW->OHWI", y_layout="NCHW->" + yl)
    slab = [(v, n) for v, n in applicable_variants(h, d) if "_slab_" in n]
    assert len(slab) >= 3
    for v, name in slab:
        print(name, flush=True)
        check_conv(h, N, C, H, W, K, R, 1, pad, dil, layouts=("NHWC", "OHWI", yl), variant=v)


# 3-D and transposed convolutions on the kernels over filter taps and over slabs: channel counts of whole and of broken K steps (and of one
# chunk), depth taps beside the channels, output phases of one to four taps per direction, tiles that end inside a phase;
# the last two have taps that these kernels leave to the copying path (a dilated one, phases of unequal taps): several launches
@pytest.mark.parametrize("dtype,out_dtype", [(alt.BF16, alt.F32), (alt.BF16, alt.BF16), (alt.F32, alt.F32)])
@pytest.mark.parametrize("op,N,C,D,H,W,K,T,R,S,stride,pad,dil", [
    ("c3d", 2, 64, 4, 6, 5, 40, 3, 3, 3, 1, 1, 1), ("c3d", 1, 24, 5, 9, 7, 72, 3, 3, 2, (2, 1, 2), (1, 1, 0), 1),
    ("c3d", 3, 8, 2, 4, 4, 12, 2, 1, 1, 1, (1, 0, 0), 1), ("c3d", 1, 96, 7, 5, 6, 132, 3, 3, 3, 1, (2, 2, 2), 2),
    ("t3d", 2, 64, 3, 5, 4, 32, 4, 4, 4, 2, 1, 1), ("t3d", 1, 40, 2, 4, 7, 24, 2, 4, 6, 2, (0, 1, 2), 1),
    ("t3d", 1, 16, 3, 3, 4, 8, 1, 2, 4, (1, 2, 2), (0, 0, 1), 1), ("t3d", 2, 128, 4, 9, 11, 72, 4, 4, 4, 2, 1, 1),
    ("t3d", 1, 32, 3, 4, 5, 16, 3, 3, 3, 1, 1, 1),
    ("t2d", 3, 48, 1, 9, 7, 36, 1, 4, 4, 2, 1, 1), ("t2d", 1, 64, 1, 20, 19, 136, 1, 8, 4, (4, 2), (2, 1), 1),
    ("t2d", 2, 8, 1, 5, 6, 4, 1, 2, 2, 2, 0, 1), ("t2d", 1, 64, 1, 12, 13, 64, 1, 6, 6, 2, 2, 1), ("t2d", 2, 32, 1, 6, 7, 16, 1, 2, 2, 2, 1, 1),
    ("t2d", 1, 32, 1, 6, 7, 16, 1, 2, 2, 2, 1, 3), ("t3d", 1, 16, 3, 4, 5, 16, 3, 3, 3, 2, 1, 1)])
def test_volumes_and_output_phases(h, op, N, C, D, H, W, K, T, R, S, stride, pad, dil, dtype, out_dtype):
    three = op != "t2d"
    x = small_ints_f32(71, (N, C, D, H, W), -3, 3)
    w = small_ints_f32(72, ((K, C) if op == "c3d" else (C, K)) + (T, R, S), -3, 3)
    b = small_ints_f32(73, (K,), -20, 20)
    each = lambda v, first: v if three else (first,) + (v if isinstance(v, tuple) else (v, v))     # a transposed C2D is one slice
    fn = oracle.conv3d if op == "c3d" else oracle.conv3d_transpose
    ref = np.maximum(fn(x, w, stride=each(stride, 1), pad=each(pad, 0), dil=each(dil, 1)) + b[None, :, None, None, None], np.float32(0))
    np_out = np.uint16 if out_dtype == alt.BF16 else np.float32
    ref = f32_to_bf16_bits(ref) if out_dtype == alt.BF16 else ref
    lay = dict(in_dtype=dtype, out_dtype=out_dtype, epilogue=alt.EPI_BIAS | alt.EPI_RELU, x_layout="NCHW->NHWC", w_layout="OIHW->OHWI",
               y_layout="NCHW->NHWC")
    if three:
        d = alt.conv3d_desc(N, C, D, H, W, K, T, R, S, stride=stride, pad=pad, dil=dil, **lay)
    else:
        d = alt.conv_desc(N, C, H, W, K, R, S, dil=dil, **lay)
        d.stride_h, d.stride_w = stride if isinstance(stride, tuple) else (stride, stride)
        d.pad_h, d.pad_w = pad if isinstance(pad, tuple) else (pad, pad)
    name = {"c3d": "conv3d", "t3d": "conv3d_transpose", "t2d": "conv2d_transpose"}[op]
    bits = lambda a: f32_to_bf16_bits(a) if dtype == alt.BF16 else a
    wshape = (K, C * T, R, S) if op == "c3d" else getattr(h, name + "_weight_shape")(d)
    wd = dev(bits(np.zeros(int(np.prod(wshape)), np.float32)))
    {"c3d": h.pack_weights3d, "t3d": h.pack_weights3d_transpose, "t2d": h.pack_weights_transpose}[op](d, dev(bits(w.reshape(-1))), wd)
    whole, y = canary_dev(ref.size, np_out)
    ws_bytes = getattr(h, name + "_workspace_size")(d)
    ws = dev(np.zeros(max(4, ws_bytes // 4), np.float32))
    print(op, N, C, D, H, W, K, T, R, S, stride, pad, dil, flush=True)
    xd, bd = dev(bits(np.ascontiguousarray(np.moveaxis(x, 1, -1)).reshape(-1))), dev(b)
    ran = kernels_run(lambda: getattr(h, name)(d, xd, wd, y, bias=bd, workspace=ws, ws_bytes=ws_bytes))
    if dil == 3 or (op, R, stride) == ("t3d", 3, 2):
        assert len(ran) > 1, ran
    else:
        assert len(ran) == 1 and ("dstream_kernel" in ran[0] or "dslab_kernel" in ran[0]), ran
    got = np.moveaxis(host(y, np_out).reshape(ref.shape[:1] + ref.shape[2:] + (K,)), -1, 1)
    assert canary_ok(whole, ref.size), "wrote outside y"
    assert np.array_equal(got, ref)


# 3x3 layers whose tiles are numbered in panels of rows (order_tiles): patch-resident kernels over all channels, over slabs and for planar
# operands, and those over filter taps; the last column of tiles is eight channels wide
@pytest.mark.parametrize("layouts,families", [(("NHWC", "OHWI", "NHWC"), ("_direct_", "_slab_", "taps_")), (("NCHW", "OIHW", "NCHW"), ("planar_",))])
def test_every_tile_of_a_panel_order_of_layers(h, layouts, families):
    N, C, H, K, R = 40, 512, 16, 72, 3
    x, w = small_ints_f32(61, (N, C, H, H), -3, 3), small_ints_f32(62, (K, C, R, R), -3, 3)
    ref = oracle.conv2d(x, w, stride=1, pad=1)
    xl, wl, yl = layouts
    lay = dict(pad=1, in_dtype=alt.BF16, out_dtype=alt.F32, x_layout="NCHW->" + xl, w_layout="OIHW->" + wl, y_layout="NCHW->" + yl)
    xd, wd = dev(to_layout(f32_to_bf16_bits(x), "NCHW", xl)), dev(to_layout(f32_to_bf16_bits(w), "OIHW", wl))
    seen = set()
    for v, name in applicable_variants(h, alt.conv_desc(N, C, H, H, K, R, R, **lay)):
        family = next((f for f in families if f in name), None)
        bm, bn = tile_of(name)
        if not family or not name.endswith("_k1") or panel_rows(N * H * H, K, bm, bn, 2 * C * bm, 2 * C * 9 * bn) == -(-N * H * H // bm):
            continue
        print(name, flush=True)
        whole, y = canary_dev(ref.size, np.float32)
        h.conv2d(alt.conv_desc(N, C, H, H, K, R, R, variant=v, **lay), xd, wd, y)
        assert canary_ok(whole, ref.size) and np.array_equal(from_layout(host(y, np.float32), ref.shape, "NCHW", yl), ref), name
        seen.add(family)
    assert seen == set(families)


# volumes and output phases large enough for the slab kernels: depth taps outside the volume, a last slab of eight channels, tiles that end
# inside a plane, a phase and an image
@pytest.mark.parametrize("op,N,C,D,H,W,K,T,R,stride,pad,dil", [
    ("c3d", 2, 40, 12, 13, 11, 72, 3, 3, 1, 1, 1), ("c3d", 1, 104, 7, 23, 21, 20, 5, 3, 1, (2, 1, 1), 1),
    ("c3d", 3, 32, 9, 15, 14, 64, 3, 3, 1, (2, 2, 2), 2), ("c3d", 1, 64, 9, 20, 19, 136, 3, 3, 1, (1, 0, 0), 1),
    ("t3d", 2, 24, 8, 24, 23, 20, 4, 4, 2, 1, 1), ("t3d", 3, 72, 7, 19, 21, 64, 4, 4, 2, 1, 1),
    ("t2d", 6, 48, 1, 44, 41, 36, 1, 4, 2, 1, 1), ("t2d", 5, 136, 1, 34, 51, 64, 1, 4, 2, 1, 1)])
@pytest.mark.parametrize("out_dtype", [alt.BF16, alt.F32])
def test_larger_volumes_and_output_phases(h, op, N, C, D, H, W, K, T, R, stride, pad, dil, out_dtype):
    x, b = small_ints_f32(71, (N, C, D, H, W), -3, 3), small_ints_f32(73, (K,), -20, 20)
    w = small_ints_f32(72, ((K, C) if op == "c3d" else (C, K)) + (T, R, R), -3, 3)
    each = lambda v, first: (first, v, v) if op == "t2d" else v
    fn = oracle.conv3d if op == "c3d" else oracle.conv3d_transpose
    ref = np.maximum(fn(x, w, stride=each(stride, 1), pad=each(pad, 0), dil=each(dil, 1)) + b[None, :, None, None, None], np.float32(0))
    lay = dict(in_dtype=alt.BF16, out_dtype=out_dtype, epilogue=alt.EPI_BIAS | alt.EPI_RELU, x_layout="NCHW->NHWC", w_layout="OIHW->OHWI",
               y_layout="NCHW->NHWC", stride=stride, pad=pad, dil=dil)
    d = alt.conv_desc(N, C, H, W, K, R, R, **lay) if op == "t2d" else alt.conv3d_desc(N, C, D, H, W, K, T, R, R, **lay)
    name, pack = {"c3d": ("conv3d", h.pack_weights3d), "t3d": ("conv3d_transpose", h.pack_weights3d_transpose),
                  "t2d": ("conv2d_transpose", h.pack_weights_transpose)}[op]
    wshape = (K, C * T, R, R) if op == "c3d" else getattr(h, name + "_weight_shape")(d)
    wd = dev(np.zeros(int(np.prod(wshape)), np.uint16))
    pack(d, dev(f32_to_bf16_bits(w.reshape(-1))), wd)
    np_out = np.uint16 if out_dtype == alt.BF16 else np.float32
    ref = f32_to_bf16_bits(ref) if out_dtype == alt.BF16 else ref
    whole, y = canary_dev(ref.size, np_out)
    ws_bytes = getattr(h, name + "_workspace_size")(d)
    ws = dev(np.zeros(max(4, ws_bytes // 4), np.float32))
    xd, bd = dev(f32_to_bf16_bits(np.ascontiguousarray(np.moveaxis(x, 1, -1)).reshape(-1))), dev(b)
    print(op, N, C, D, H, W, K, T, R, flush=True)
    ran = kernels_run(lambda: getattr(h, name)(d, xd, wd, y, bias=bd, workspace=ws, ws_bytes=ws_bytes))
    assert len(ran) == 1 and "dslab_kernel" in ran[0], ran
    assert canary_ok(whole, ref.size), "wrote outside y"
    assert np.array_equal(np.moveaxis(host(y, np_out).reshape(ref.shape[:1] + ref.shape[2:] + (K,)), -1, 1), ref)


# single precision: the library's own choice among tiles, K groups and slices (remainders in all of them), with the workspace that
# this choice asks for
@pytest.mark.parametrize("N,C,H,W,K,R", [(5, 64, 21, 19, 64, 3), (1, 512, 7, 7, 512, 3), (3, 72, 9, 11, 76, 3), (1, 256, 30, 31, 36, 1),
                                         (1, 8, 5, 5, 4, 3), (2, 320, 6, 5, 320, 3)])
def test_fp32_default_choice(h, N, C, H, W, K, R):
    d = alt.conv_desc(N, C, H, W, K, R, R, pad=R // 2, in_dtype=alt.F32, out_dtype=alt.F32, x_layout="NCHW->NHWC",
                      w_layout="OIHW->OHWI", y_layout="NCHW->NHWC", epilogue=alt.EPI_BIAS | alt.EPI_RELU)
    assert "_rtaps_" in h.conv2d_variant_name(d, -1)
    check_conv(h, N, C, H, W, K, R, pad=R // 2, dtype=alt.F32)


# products of few rows and long sums: unsplit or in a few slices, never on the patch-resident kernel
@pytest.mark.parametrize("M,N,K", [(37, 768, 3072), (200, 1024, 4096), (810, 384, 1536), (1, 64, 8192), (300, 264, 2048)])
@pytest.mark.parametrize("lay", ["NK", "KN"])
def test_product_default_choice(h, M, N, K, lay):
    a, b = small_ints_f32(81, (M, K), -2, 2), small_ints_f32(82, (K, N), -2, 2)
    A, B = f32_to_bf16_bits(a), f32_to_bf16_bits(b)
    d = alt.gemm_desc(M, N, K, b_layout="KN->" + lay)
    assert "stream" in h.gemm_variant_name(d, -1) or "taps" in h.gemm_variant_name(d, -1)
    ws_bytes = h.gemm_workspace_size(d)
    whole, C = canary_dev(M * N, np.float32)
    h.gemm(d, dev(A), dev(B if lay == "KN" else np.ascontiguousarray(B.T)), C, workspace=dev(np.zeros(max(1, ws_bytes // 4), np.float32)),
           ws_bytes=ws_bytes)
    assert canary_ok(whole, M * N) and np.array_equal(host(C, np.float32).reshape(M, N), oracle.gemm(A, B))


@pytest.mark.parametrize("kind", ["tile", "sliced", "depthwise", "product", "volume"])
def test_later_calls_use_their_own_buffers(h, kind):
    """A launch kept from the first call takes its operands' addresses, stream and workspace from the call."""
    lay = dict(x_layout="NCHW->NHWC", w_layout="OIHW->OHWI", y_layout="NCHW->NHWC", out_dtype=alt.BF16)
    if kind == "product":
        d, call, size, sizes = alt.gemm_desc(100, 96, 128, out_dtype=alt.BF16, b_layout="KN->NK"), h.gemm, h.gemm_workspace_size, (12800, 12288, 9600)
    elif kind == "volume":
        d, call, size = alt.conv3d_desc(1, 16, 3, 6, 6, 16, 3, 3, 3, pad=1, **lay), h.conv3d, h.conv3d_workspace_size
        sizes = (1728, 6912, 1728)
    else:
        C, H, g = (64, 9, 64) if kind == "depthwise" else (64, 9, 1)
        d = alt.conv_desc(2, C, H, H, C, 3, 3, pad=1, groups=g, **lay)
        if kind == "sliced":
            names = applicable_variants(h, d)
            d.variant = next(v for v, n in names if "_64x64x64_taps_" in n and n.endswith("_k3"))
        call, size, sizes = h.conv2d, h.conv2d_workspace_size, (2 * H * H * C, C * C * 9 // g, 2 * H * H * C)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    outs = []
    for s in streams:
        gen = torch.Generator(device="cuda").manual_seed(len(outs))
        x, w = (torch.randint(-4, 5, (n,), generator=gen, device="cuda").to(torch.bfloat16) for n in sizes[:2])
        nb = size(d)
        for _ in range(2):
            y, ws = torch.zeros(sizes[2], dtype=torch.bfloat16, device="cuda"), torch.empty(max(nb, 16), dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            call(d, x, w, y, workspace=ws, ws_bytes=nb, stream=s)
            torch.cuda.synchronize()
            outs.append(y)
        fresh, y = alt.Handle(), torch.zeros_like(y)
        getattr(fresh, call.__name__)(d, x, w, y, workspace=ws, ws_bytes=nb)
        torch.cuda.synchronize()
        assert torch.equal(outs[-1], y) and torch.equal(outs[-2], y) and bool(y.any())
