"""The kernel for short reductions (csrc/dshort.h): every tile, edges of rows, columns, chunks and stages, rows of any length and alignment.
Small integers, so that the rounded results are the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2210_12415_amd as alt
from gpu_util import canary_dev, canary_ok, dev, from_layout, host, to_layout
from workloads.inputs import f32_to_bf16_bits, small_ints_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    return alt.Handle()


def short_variants(names):
    return [(v, n) for v, n in names if "_short_" in n]


def variants(h, d, conv):
    count, name = (h.conv2d_variant_count, h.conv2d_variant_name) if conv else (h.gemm_variant_count, h.gemm_variant_name)
    found = []
    for v in range(count(d)):
        try:
            found.append((v, name(d, v)))
        except alt.AltError:
            pass
    return short_variants(found)


# M, N, K, batch: one element; a tile and one more in every direction; every number of stages, whole and broken; many entries, odd rows
PRODUCTS = [(1, 1, 8, 1), (128, 32, 64, 2), (129, 33, 72, 3), (127, 95, 56, 2), (257, 97, 128, 1), (64, 191, 136, 2), (130, 64, 192, 1), (5, 7, 200, 3),
            (131, 65, 256, 2), (37, 37, 64, 12), (15, 15, 64, 301)]


@pytest.mark.parametrize("M,N,K,batch", PRODUCTS)
def test_products(h, M, N, K, batch):
    A, B = small_ints_f32(1, (batch, M, K), -2, 2), small_ints_f32(2, (batch, N, K), -2, 2)
    ref = f32_to_bf16_bits(np.matmul(A, B.transpose(0, 2, 1)))
    d = alt.gemm_desc(M, N, K, batch=batch, in_dtype=alt.BF16, out_dtype=alt.BF16, b_layout="KN->NK")
    found = variants(h, d, False)
    assert len(found) == (3 if K <= 128 else 2)
    a, b = dev(f32_to_bf16_bits(A)), dev(f32_to_bf16_bits(B))
    for v, name in found:
        d.variant = v
        for shift in (0, 1):                     # an output at any even address
            whole, c = canary_dev(ref.size + shift, np.uint16)
            h.gemm(d, a, b, c[shift:])
            assert canary_ok(whole, ref.size + shift), name
            assert np.array_equal(host(c[shift:], np.uint16).reshape(ref.shape), ref), (name, shift)


@pytest.mark.parametrize("N,C,H,K,epilogue", [(2, 24, 13, 144, 3), (1, 144, 9, 24, 1), (3, 256, 7, 64, 0), (1, 8, 1, 4, 3), (2, 72, 12, 100, 2)])
def test_convolutions(h, N, C, H, K, epilogue):
    x, w, b = small_ints_f32(3, (N, C, H, H), -2, 2), small_ints_f32(4, (K, C, 1, 1), -2, 2), small_ints_f32(5, (K,), -4, 4)
    ref = oracle.conv2d(x, w, stride=1, pad=0)
    if epilogue & alt.EPI_BIAS:
        ref = ref + b[None, :, None, None]
    if epilogue & alt.EPI_RELU:
        ref = np.maximum(ref, 0)
    d = alt.conv_desc(N, C, H, H, K, 1, 1, in_dtype=alt.BF16, out_dtype=alt.BF16, epilogue=epilogue, x_layout="NCHW->NHWC", w_layout="OIHW->OHWI", y_layout="NCHW->NHWC")
    xd, wd, bd = dev(to_layout(f32_to_bf16_bits(x), "NCHW", "NHWC")), dev(f32_to_bf16_bits(w)), dev(b)
    found = variants(h, d, True)
    assert found
    for v, name in found:
        d.variant = v
        whole, y = canary_dev(ref.size, np.uint16)
        h.conv2d(d, xd, wd, y, bias=bd)
        assert canary_ok(whole, ref.size), name
        assert np.array_equal(from_layout(host(y, np.uint16), ref.shape, "NCHW", "NHWC"), f32_to_bf16_bits(ref)), name


def test_infinities_and_nan_stay_in_their_rows(h):
    """What lies behind an operand's rows and columns is zeros in LDS: an infinite or NaN element reaches its own row and column alone."""
    M, N, K = 130, 35, 24
    A, B = small_ints_f32(6, (M, K), -2, 2), small_ints_f32(7, (N, K), 1, 3)
    A[129, 23], A[7, 0] = np.inf, np.nan
    with np.errstate(invalid="ignore"):
        ref = A @ B.T
    d = alt.gemm_desc(M, N, K, in_dtype=alt.BF16, out_dtype=alt.BF16, b_layout="KN->NK")
    for v, name in variants(h, d, False):
        d.variant = v
        c = torch.zeros(M * N, dtype=torch.int16, device="cuda")
        h.gemm(d, dev(f32_to_bf16_bits(A)), dev(f32_to_bf16_bits(B)), c)
        got = (host(c, np.uint16).astype(np.uint32) << 16).view(np.float32).reshape(M, N)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~np.isnan(ref)], ref[~np.isnan(ref)]), name
