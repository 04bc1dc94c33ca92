"""Which kernel family the library picks by itself, on both sides of the lines its estimate draws (ops.hip).  Host only."""
import time

import pytest

import paper_2210_12415_amd as alt


@pytest.fixture(scope="module")
def h():
    return alt.Handle()


def conv(h, N, C, H, K, R, stride=1, dtype=alt.BF16):
    return h.conv2d_variant_name(alt.conv_desc(N, C, H, H, K, R, R, stride=stride, pad=R // 2, in_dtype=dtype, out_dtype=dtype,
                                               x_layout="NCHW->NHWC", w_layout="OIHW->OHWI", y_layout="NCHW->NHWC"), -1)


def gemm(h, M, N, K, lay, batch=1, dtype=alt.BF16):
    return h.gemm_variant_name(alt.gemm_desc(M, N, K, batch=batch, in_dtype=dtype, out_dtype=dtype, b_layout="KN->" + lay), -1)


@pytest.mark.parametrize("M,N,K,lay,batch,family", [
    (3220, 208, 800, "NK", 1, "_stream_"), (1865, 584, 1696, "NK", 7, "_stream_"), (542, 1168, 544, "NK", 1, "_stream_"),
    (424, 1680, 160, "NK", 1, "_stream_"), (15, 4048, 96, "KN", 1, "_rtapskn_"), (215, 388, 2912, "NK", 1, "_rtaps_"),
    (300, 264, 1048, "NK", 1, "_rtaps_")])
def test_products_whose_depth_is_an_odd_number_of_half_steps(h, M, N, K, lay, batch, family):
    assert family in gemm(h, M, N, K, lay, batch)


@pytest.mark.parametrize("N,C,H,K,stride,family", [
    (8, 608, 12, 640, 1, "_stream_"), (4, 608, 23, 8, 1, "_stream_"), (16, 256, 56, 64, 1, "_stream_"),
    (17, 512, 17, 244, 2, "taps_"), (21, 256, 22, 92, 2, "taps_"), (3, 128, 42, 108, 2, "taps_")])
def test_one_tap_convolutions(h, N, C, H, K, stride, family):
    assert family in conv(h, N, C, H, K, 1, stride)


@pytest.mark.parametrize("C,H,K,R", [(64, 56, 64, 3), (128, 28, 128, 3), (256, 14, 256, 3), (512, 7, 512, 3), (256, 56, 64, 1)])
def test_single_precision_layers_do_not_change_kernels_with_the_batch(h, C, H, K, R):
    assert all("_rtaps_" in conv(h, n, C, H, K, R, dtype=alt.F32) for n in range(1, 41))


@pytest.mark.parametrize("M,N,K,batch,taps", [(4, 28, 6360, 2, False), (12, 12, 4920, 4, False), (14, 64, 3576, 22, True),
                                              (87, 684, 2280, 18, True), (4, 28, 6360, 1, True)])
def test_single_precision_batches_of_few_tiles_run_in_slices(h, M, N, K, batch, taps):
    name = gemm(h, M, N, K, "NK", batch, alt.F32)
    assert ("_rtaps_" in name) == taps and (taps or not name.endswith("_k1"))


@pytest.mark.parametrize("N,C,H,K,family", [
    (16, 64, 56, 64, "_direct_"), (16, 128, 28, 128, "_direct_"), (16, 512, 7, 512, "_direct_"), (1, 256, 14, 256, "_direct_"),
    (256, 256, 14, 256, "taps_"), (256, 512, 7, 512, "_slab_"), (40, 96, 39, 96, "_slab_"), (6, 208, 15, 208, "_slab_"), (4, 128, 5, 128, "_direct_")])
def test_layers_run_unsliced(h, N, C, H, K, family):
    name = conv(h, N, C, H, K, 3)
    assert family in name and name.endswith("_k1")


def test_choosing_a_kernel_takes_no_longer_for_large_batches(h):
    """The largest patch of any tile is found without a walk over all tiles (here 24000 of them, for dozens of variants: 7 ms)."""
    def us(N):
        d = alt.conv_desc(N, 64, 56, 56, 64, 3, 3, in_dtype=alt.BF16, out_dtype=alt.BF16, x_layout="NCHW->NHWC",
                          w_layout="OIHW->OHWI", y_layout="NCHW->NHWC")
        times = []
        for _ in range(7):
            t = time.perf_counter()
            h.conv2d_variant_name(d, -1)
            times.append(time.perf_counter() - t)
        return min(times)
    assert us(512) < 5 * us(8)


@pytest.mark.parametrize("N,C,D,H,W,K", [(1, 96, 7, 23, 6, 136), (1, 128, 2, 25, 2, 152), (3, 144, 3, 17, 6, 128)])
def test_a_volumes_workspace_holds_the_slices_of_the_kernel_that_runs(h, N, C, D, H, W, K):
    """The kernels over filter taps read the volume in place, in more slices than the depth-unfolded problem takes."""
    d = alt.conv3d_desc(N, C, D, H, W, K, 3, 3, 3, stride=(2, 1, 1), pad=1, in_dtype=alt.BF16, out_dtype=alt.BF16,
                        x_layout="NCHW->NHWC", w_layout="OIHW->OHWI", y_layout="NCHW->NHWC")
    n, k, od, oh, ow = h.conv3d_output_shape(d)
    assert h.conv3d_workspace_size(d) >= 3 * n * k * od * oh * ow * 4


def planar(h, N, C, H, K, R):
    return h.conv2d_variant_name(alt.conv_desc(N, C, H, H, K, R, R, pad=R // 2, in_dtype=alt.BF16, out_dtype=alt.BF16,
                                               x_layout="NCHW->NCHW", w_layout="OIHW->OIHW", y_layout="NCHW->NCHW"), -1)


@pytest.mark.parametrize("widths", [(40, 48, 56, 64), (72, 88, 104, 120, 128)])
def test_planar_layers_of_as_many_channel_steps_run_the_same_tile(h, widths):
    """A step of 64 channels that is filled up with zeros costs what a whole one does."""
    assert len({planar(h, 16, C, 28, 64, 3).replace("rplanar", "planar") for C in widths}) == 1


@pytest.mark.parametrize("M,N,K,family", [(47, 664, 3960, "_gg_"), (170, 1792, 3040, "_gv_"), (112, 1464, 704, "planar_"), (2291, 1600, 608, "planar_")])
def test_products_with_contiguous_rows_of_a(h, M, N, K, family):
    assert family in h.gemm_variant_name(alt.gemm_desc(M, N, K, in_dtype=alt.BF16, out_dtype=alt.BF16, a_layout="MK->KM", b_layout="KN->NK"), -1)


@pytest.mark.parametrize("N,C,H,K,epilogue,short", [
    (46, 248, 76, 296, 3, False), (41, 176, 76, 224, 1, False), (14, 144, 38, 624, 0, False), (12, 200, 61, 568, 3, False), (44, 168, 72, 544, 1, False),
    (4, 160, 81, 160, 1, False), (87, 72, 47, 224, 3, False), (42, 248, 73, 272, 1, False), (46, 88, 37, 208, 1, False),
    (16, 24, 56, 144, 3, True), (16, 144, 56, 24, 1, True), (256, 256, 56, 64, 0, True), (64, 32, 56, 192, 3, True)])
def test_one_tap_layers_of_few_channels(h, N, C, H, K, epilogue, short):
    """The kernels for short reductions run layers with a bias and wide outputs only where they are the faster ones (those above took 1.2 to 1.45 times
    as long as on the tile kernels)."""
    d = alt.conv_desc(N, C, H, H, K, 1, 1, in_dtype=alt.BF16, out_dtype=alt.BF16, epilogue=epilogue,
                      x_layout="NCHW->NHWC", w_layout="OIHW->OHWI", y_layout="NCHW->NHWC")
    assert ("_short_" in h.conv2d_variant_name(d, -1)) == short
