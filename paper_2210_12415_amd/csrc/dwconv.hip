// Depth-wise 2-D convolution (one filter per channel: groups = C = K), the
// memory-bound member of the C2D family of Section 6.1 of the paper:
//   y[n,c,oh,ow] = sum_{r,s} x[n,c,oh*stride-pad+r*dil, ow*stride-pad+s*dil] * w[c,0,r,s]
// fp32 accumulation over the taps in (r, s) order, then bias, ReLU and the
// output rounding.  There is no reduction over channels, so nothing for the
// matrix cores to do: the kernels are a gather over the filter window, and
// the data layout decides how wide the accesses are.
//
//  * vector kernel: bf16 tensors whose channel is contiguous in runs of at
//    least eight on activations and output (NHWC or NCHW[x]c), with
//    channel-last weights or weights whose taps lie side by side (OHWI, OIHW):
//    a thread owns eight channels of one output pixel, every access to the
//    activations is 16 bytes
//    (3x3 filters without dilation get a register-tiled version of it);
//  * row kernel: bf16 tensors whose width is contiguous on activations and
//    output (NCHW), 3x3 filters with padding 1 along the width: a thread owns
//    four or eight consecutive outputs of one row of one channel plane,
//    reads the input columns under them as 8- or 16-byte vectors (plus the
//    column before them) and stores one such vector;
//  * element kernel: any separable layout; a thread owns one output element,
//    threads run along the output's contiguous dimension.
#include <hip/hip_runtime.h>

#include "igemm_dma.h"
#include "ops.h"

namespace alt {
namespace {

constexpr int kDwThreads = 256;
constexpr int kDwCols = 4;    // output columns per thread of the 3x3 vector kernel

struct DwParams {
    const void *x, *w;
    const float *bias;
    void *y;
    int32_t N, C, H, W, R, S, OH, OW;
    int32_t stride_h, stride_w, pad_h, pad_w, dil_h, dil_w;
    int32_t epilogue, in_bf16, out_bf16, chan_fast;
    Dim2 xn, xc, xh, xw, wo, wr, ws, yn, yk, yh, yw;
    // 3x3 vector kernel: threads, the divisions of a thread's index, sizes of the tensors
    uint32_t items, x_bytes, y_bytes;
    FastDiv fd_c8, fd_owb, fd_ohb;
};

__device__ __forceinline__ float load_elem(const void *p, int64_t off, int bf16)
{
    if (bf16) return __builtin_bit_cast(float, (uint32_t)((const uint16_t *)p)[off] << 16);
    return ((const float *)p)[off];
}

__global__ __launch_bounds__(kDwThreads) void dwconv_elem_kernel(const DwParams p)
{
    const int64_t total = (int64_t)p.N * p.C * p.OH * p.OW;
    for (int64_t e = blockIdx.x * (int64_t)kDwThreads + threadIdx.x; e < total; e += (int64_t)gridDim.x * kDwThreads) {
        int n, c, oh, ow;
        if (total <= 0x7fffffff) {                  // 32-bit divisions cost a fraction of 64-bit ones
            uint32_t r = (uint32_t)e;
            if (p.chan_fast) {
                c = (int)(r % (uint32_t)p.C); r /= (uint32_t)p.C;
                ow = (int)(r % (uint32_t)p.OW); r /= (uint32_t)p.OW;
                oh = (int)(r % (uint32_t)p.OH); n = (int)(r / (uint32_t)p.OH);
            } else {
                ow = (int)(r % (uint32_t)p.OW); r /= (uint32_t)p.OW;
                oh = (int)(r % (uint32_t)p.OH); r /= (uint32_t)p.OH;
                c = (int)(r % (uint32_t)p.C); n = (int)(r / (uint32_t)p.C);
            }
        } else {
            int64_t r = e;
            if (p.chan_fast) {
                c = (int)(r % p.C); r /= p.C;
                ow = (int)(r % p.OW); r /= p.OW;
                oh = (int)(r % p.OH); n = (int)(r / p.OH);
            } else {
                ow = (int)(r % p.OW); r /= p.OW;
                oh = (int)(r % p.OH); r /= p.OH;
                c = (int)(r % p.C); n = (int)(r / p.C);
            }
        }
        const int64_t xb = dim2_off(p.xn, n) + dim2_off(p.xc, c), wb = dim2_off(p.wo, c);
        float acc = 0.f;
        // (H, W, R and S are rarely blocked: then an offset is a multiply, not a division)
        const bool lin = p.xh.f >= p.H && p.xw.f >= p.W && p.wr.f >= p.R && p.ws.f >= p.S;
        for (int fr = 0; fr < p.R; ++fr) {
            const int ih = oh * p.stride_h - p.pad_h + fr * p.dil_h;
            if ((unsigned)ih >= (unsigned)p.H) continue;
            const int64_t xr = xb + (lin ? ih * p.xh.si : dim2_off(p.xh, ih));
            const int64_t wr = wb + (lin ? fr * p.wr.si : dim2_off(p.wr, fr));
            for (int fs = 0; fs < p.S; ++fs) {
                const int iw = ow * p.stride_w - p.pad_w + fs * p.dil_w;
                if ((unsigned)iw >= (unsigned)p.W) continue;
                acc += load_elem(p.x, xr + (lin ? iw * p.xw.si : dim2_off(p.xw, iw)), p.in_bf16) *
                       load_elem(p.w, wr + (lin ? fs * p.ws.si : dim2_off(p.ws, fs)), p.in_bf16);
            }
        }
        if (p.epilogue & ALT_EPI_BIAS) acc += p.bias[c];
        if (p.epilogue & ALT_EPI_RELU) acc = fmaxf(acc, 0.f);
        const int64_t yo = dim2_off(p.yn, n) + dim2_off(p.yk, c) + dim2_off(p.yh, oh) + dim2_off(p.yw, ow);
        if (p.out_bf16) ((uint16_t *)p.y)[yo] = f32_to_bf16_rne(acc);
        else ((float *)p.y)[yo] = acc;
    }
}

// bf16 in and out, eight consecutive channels per thread (one 16-byte access per tensor and tap).  TAPS: the taps of a channel
// lie side by side, so a tap's eight filter values are loaded one by one.  (A template: the choice made inside the loop over
// the taps cost filters with the channel innermost 13 to 20 %, 26 x 568 x 40 x 40 under 5x5 156 us against 133.)
template <bool TAPS>
__global__ __launch_bounds__(kDwThreads) void dwconv_vec8_kernel(const DwParams p)
{
    typedef uint32_t w4_t __attribute__((ext_vector_type(4)));
    typedef float f4_t __attribute__((ext_vector_type(4)));
    const int C8 = p.C >> 3;
    const int64_t total = (int64_t)p.N * p.OH * p.OW * C8;
    for (int64_t e = blockIdx.x * (int64_t)kDwThreads + threadIdx.x; e < total; e += (int64_t)gridDim.x * kDwThreads) {
        int64_t r = e;
        const int c = (int)(r % C8) * 8; r /= C8;
        const int ow = (int)(r % p.OW); r /= p.OW;
        const int oh = (int)(r % p.OH);
        const int n = (int)(r / p.OH);
        const int64_t xb = dim2_off(p.xn, n) + dim2_off(p.xc, c), wb = dim2_off(p.wo, c);
        // even channels of each pair in lo, odd ones in hi (whole-vector arithmetic throughout)
        f4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
        for (int fr = 0; fr < p.R; ++fr) {
            const int ih = oh * p.stride_h - p.pad_h + fr * p.dil_h;
            if ((unsigned)ih >= (unsigned)p.H) continue;
            for (int fs = 0; fs < p.S; ++fs) {
                const int iw = ow * p.stride_w - p.pad_w + fs * p.dil_w;
                if ((unsigned)iw >= (unsigned)p.W) continue;
                const w4_t xv = *(const w4_t *)((const uint16_t *)p.x + xb + dim2_off(p.xh, ih) + dim2_off(p.xw, iw));
                w4_t wv;
                if constexpr (TAPS) {
                    const uint16_t *we = (const uint16_t *)p.w + (int64_t)c * p.R * p.S + fr * p.S + fs;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        wv[q] = (uint32_t)we[(int64_t)2 * q * p.R * p.S] | ((uint32_t)we[(int64_t)(2 * q + 1) * p.R * p.S] << 16);
                } else {
                    wv = *(const w4_t *)((const uint16_t *)p.w + wb + dim2_off(p.wr, fr) + dim2_off(p.ws, fs));
                }
                lo += __builtin_bit_cast(f4_t, xv << 16) * __builtin_bit_cast(f4_t, wv << 16);
                hi += __builtin_bit_cast(f4_t, xv & 0xffff0000u) * __builtin_bit_cast(f4_t, wv & 0xffff0000u);
            }
        }
        if (p.epilogue & ALT_EPI_BIAS) {
            const f4_t b0 = *(const f4_t *)(p.bias + c), b1 = *(const f4_t *)(p.bias + c + 4);
            lo += __builtin_shufflevector(b0, b1, 0, 2, 4, 6);
            hi += __builtin_shufflevector(b0, b1, 1, 3, 5, 7);
        }
        if (p.epilogue & ALT_EPI_RELU) {
            lo = __builtin_elementwise_max(lo, (f4_t){0.f, 0.f, 0.f, 0.f});
            hi = __builtin_elementwise_max(hi, (f4_t){0.f, 0.f, 0.f, 0.f});
        }
        w4_t out;
#pragma unroll
        for (int q = 0; q < 4; ++q) out[q] = f32x2_to_bf16x2(lo[q], hi[q]);
        const int64_t yo = dim2_off(p.yn, n) + dim2_off(p.yk, c) + dim2_off(p.yh, oh) + dim2_off(p.yw, ow);
        *(w4_t *)((uint16_t *)p.y + yo) = out;
    }
}

typedef uint32_t dw_words __attribute__((ext_vector_type(4)));

// The filters of eight channels from c on, tap by tap.  TAPS: tap-contiguous, 72 elements in one run, transposed in registers.
template <bool TAPS>
__device__ __forceinline__ void dw_3x3_filter(const DwParams &p, int c, dw_words (&wv)[9])
{
    typedef dw_words w4_t;
    if constexpr (TAPS) {
        const w4_t *wp = (const w4_t *)((const uint16_t *)p.w + c * 9);
        uint32_t raw[36];
#pragma unroll
        for (int v = 0; v < 9; ++v) {
            const w4_t d = wp[v];
#pragma unroll
            for (int q = 0; q < 4; ++q) raw[v * 4 + q] = d[q];
        }
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {           // channels 2q and 2q + 1 of tap t
                const int a = 2 * q * 9 + t, b = a + 9;
                wv[t][q] = __builtin_amdgcn_perm(raw[b / 2], raw[a / 2], ((b & 1) ? 0x07060000u : 0x05040000u) | ((a & 1) ? 0x0302u : 0x0100u));
            }
    } else {
        const uint16_t *wb = (const uint16_t *)p.w + dim2_off(p.wo, c);
#pragma unroll
        for (int t = 0; t < 9; ++t) wv[t] = *(const w4_t *)(wb + dim2_off(p.wr, t / 3) + dim2_off(p.ws, t % 3));
    }
}

// The outputs of thread `t` of the 3x3 vector kernel once more, over the taps inside the image alone, if it stands at the border and
// its filters hold an infinite or NaN value: the same sums with the filter cleared under taps outside.
// (16 x 144 x 56 x 56 takes 7.5 us, with NaN inputs 8.3, with NaN filters 21.1; one element at a time it took 225, a row of outputs
// at a time 19.1, but those 11 KB of code, never run, cost every pass through several kernels 1 %.)
template <int STRIDE, int TW, int TH, bool TAPS, int POLICY>
__device__ __forceinline__ void dw_3x3_inside(uint32_t t)
{
    // (the item is decoded and the kernel's argument read anew, so that the kernel keeps nothing in registers for this)
    typedef const __attribute__((address_space(4))) DwParams *arg_t;
    arg_t arg = (arg_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(arg), "+v"(t));
    const DwParams &p = *(const DwParams *)arg;
    typedef uint32_t w4_t __attribute__((ext_vector_type(4)));
    typedef float f4_t __attribute__((ext_vector_type(4)));
    const uint32_t e = (uint32_t)igemm_logical_tile((int)gridDim.x) * kDwThreads + t;
    uint32_t r = fast_div(e, p.fd_c8);
    const int c = (int)(e - r * p.fd_c8.d) * 8;
    const uint32_t r2 = fast_div(r, p.fd_owb);
    const int ow0 = (int)(r - r2 * p.fd_owb.d) * TW;
    const int n = (int)fast_div(r2, p.fd_ohb);
    const int oh0 = (int)(r2 - (uint32_t)n * p.fd_ohb.d) * TH;
    const int ih0 = oh0 * STRIDE - p.pad_h, iw0 = ow0 * STRIDE - p.pad_w;
    if (ih0 >= 0 && iw0 >= 0 && ih0 + (TH - 1) * STRIDE + 3 <= p.H && iw0 + (TW - 1) * STRIDE + 3 <= p.W) return;
    w4_t wv[9];
    dw_3x3_filter<TAPS>(p, c, wv);
    typedef uint16_t h8_t __attribute__((ext_vector_type(8)));
    h8_t largest = 0;
#pragma unroll
    for (int f = 0; f < 9; ++f) largest = __builtin_elementwise_max(largest, __builtin_bit_cast(h8_t, wv[f] & 0x7fff7fffu));
    const bool finite = __builtin_reduce_max(largest) < 0x7f80;
    if (finite) return;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc((void *)p.y, 0, (int)p.y_bytes, 0x00020000);
    const int32_t xb = dim2_off32(p.xn, n) + dim2_off32(p.xc, c), yb = dim2_off32(p.yn, n) + dim2_off32(p.yk, c);
    f4_t blo = {0.f, 0.f, 0.f, 0.f}, bhi = {0.f, 0.f, 0.f, 0.f};
    if (p.epilogue & ALT_EPI_BIAS) {
        const f4_t b0 = *(const f4_t *)(p.bias + c), b1 = *(const f4_t *)(p.bias + c + 4);
        blo = __builtin_shufflevector(b0, b1, 0, 2, 4, 6);
        bhi = __builtin_shufflevector(b0, b1, 1, 3, 5, 7);
    }
    const float floor_ = relu_floor(p.epilogue & ALT_EPI_RELU);
#pragma unroll 1
    for (int o = 0; o < TH * TW; ++o) {
        const int oh = oh0 + o / TW, ow = ow0 + o % TW;
        w4_t xv[9];
        uint32_t inside[9];
#pragma unroll
        for (int f = 0; f < 9; ++f) {
            asm volatile("" : "+v"(wv[f]));         // (stays packed from output to output)
            const int ih = oh * STRIDE - p.pad_h + f / 3, iw = ow * STRIDE - p.pad_w + f % 3;
            const bool ok = (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
            inside[f] = ok ? 0xffffffffu : 0u;
            xv[f] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(ok ? (uint32_t)(xb + ih * (int32_t)p.xh.si + iw * (int32_t)p.xw.si) * 2u : kOutOfRange), 0, 0);
        }
        f4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < 9; ++f) {
            const w4_t w = wv[f] & inside[f];
            lo += __builtin_bit_cast(f4_t, xv[f] << 16) * __builtin_bit_cast(f4_t, w << 16);
            hi += __builtin_bit_cast(f4_t, xv[f] & 0xffff0000u) * __builtin_bit_cast(f4_t, w & 0xffff0000u);
        }
        lo = __builtin_elementwise_max(lo + blo, (f4_t){floor_, floor_, floor_, floor_});
        hi = __builtin_elementwise_max(hi + bhi, (f4_t){floor_, floor_, floor_, floor_});
        w4_t out;
#pragma unroll
        for (int q = 0; q < 4; ++q) out[q] = f32x2_to_bf16x2(lo[q], hi[q]);
        const bool ok = ow < p.OW && oh < p.OH;
        __builtin_amdgcn_raw_buffer_store_b128(out, yr, (int)(ok ? (uint32_t)(yb + oh * (int32_t)p.yh.si + ow * (int32_t)p.yw.si) * 2u : kOutOfRange), 0, POLICY);
    }
}

// The common case of the vector kernel: 3x3 filter, dilation 1, H and W not blocked, tensors below 2 GiB a launch.  A
// thread owns eight channels of TH x TW output pixels: the filter is loaded once, and neighbouring outputs share the
// input pixels of their windows, so a thread makes ((TH-1)*STRIDE+3) * ((TW-1)*STRIDE+3) loads for TH*TW outputs.
// The kernel is bound by memory: all its loads go through a buffer descriptor (a pixel outside the image gets an
// out-of-range offset and reads zeros), so no branch keeps them from being in flight together.
// TAPS: the filter lies tap-contiguous (OHWI, OIHW: the nine taps of a channel side by side), so that eight
// channels' taps are one run of 72 elements; they are loaded as nine vectors and transposed in registers.
// Consecutive blocks run on one XCD, so that the rows two blocks share come out of one L2.
// Measured on 16 x 144 x 56 x 56 (29 MB): 7.5 us, 3.9 TB/s; OHWI filters took the element kernel before, 137 us, and
// filters with the channel innermost a version of this one with a branch per load and one row per thread, 13.0 us.
// POLICY: of the stores.  Outputs that the L2s could keep (32 MB) go through to memory as they are written, which leaves nothing to write back
// between this kernel and the next: a block of 16 x 144 x 56 x 56 26.6 us before and 25.3 so, of 15 x 384 x 29 x 29 24.1 and 23.1; larger ones leave
// the L2s anyway (32 x 528 x 43 x 43 102.0 us, through 103.8).
template <int STRIDE, int TW, int TH, bool TAPS, int POLICY>
__global__ __launch_bounds__(kDwThreads, 2) void dwconv_vec8_3x3_kernel(const DwParams p)
{
    typedef uint32_t w4_t __attribute__((ext_vector_type(4)));
    typedef float f4_t __attribute__((ext_vector_type(4)));
    constexpr int NCOL = (TW - 1) * STRIDE + 3, NROW = (TH - 1) * STRIDE + 3;
    const uint32_t e = (uint32_t)igemm_logical_tile((int)gridDim.x) * kDwThreads + threadIdx.x;
    if (e >= p.items) return;
    uint32_t r = fast_div(e, p.fd_c8);
    const int c = (int)(e - r * p.fd_c8.d) * 8;
    const uint32_t r2 = fast_div(r, p.fd_owb);
    const int ow0 = (int)(r - r2 * p.fd_owb.d) * TW;
    const int n = (int)fast_div(r2, p.fd_ohb);
    const int oh0 = (int)(r2 - (uint32_t)n * p.fd_ohb.d) * TH;

    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc((void *)p.y, 0, (int)p.y_bytes, 0x00020000);
    w4_t wv[9];                                     // kept packed: unpacked where used, half the registers
    dw_3x3_filter<TAPS>(p, c, wv);
    f4_t lo[TH][TW], hi[TH][TW];
#pragma unroll
    for (int i = 0; i < TH; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j) { lo[i][j] = (f4_t){0.f, 0.f, 0.f, 0.f}; hi[i][j] = (f4_t){0.f, 0.f, 0.f, 0.f}; }
    const int ih0 = oh0 * STRIDE - p.pad_h, iw0 = ow0 * STRIDE - p.pad_w;
    const int32_t xb = dim2_off32(p.xn, n) + dim2_off32(p.xc, c), sxh = (int32_t)p.xh.si, sxw = (int32_t)p.xw.si;
    uint32_t col[NCOL];                             // byte offset of each input column, out of range outside the image
#pragma unroll
    for (int q = 0; q < NCOL; ++q)
        col[q] = (unsigned)(iw0 + q) < (unsigned)p.W ? (uint32_t)(xb + (iw0 + q) * sxw) * 2u : kOutOfRange;
#pragma unroll
    for (int fr = 0; fr < NROW; ++fr) {
        const int ih = ih0 + fr;
        const bool row_ok = (unsigned)ih < (unsigned)p.H;
        const uint32_t row = (uint32_t)(ih * sxh) * 2u;
        w4_t xv[NCOL];
#pragma unroll
        for (int q = 0; q < NCOL; ++q)
            xv[q] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(row_ok && col[q] != kOutOfRange ? col[q] + row : kOutOfRange), 0, 0);
        f4_t xlo[NCOL], xhi[NCOL];
#pragma unroll
        for (int q = 0; q < NCOL; ++q) {
            xlo[q] = __builtin_bit_cast(f4_t, xv[q] << 16);
            xhi[q] = __builtin_bit_cast(f4_t, xv[q] & 0xffff0000u);
        }
#pragma unroll
        for (int i = 0; i < TH; ++i) {
            const int wr = fr - i * STRIDE;         // this input row's place in output row i's window
            if (wr < 0 || wr >= 3) continue;
#pragma unroll
            for (int fs = 0; fs < 3; ++fs) {
                const f4_t wl = __builtin_bit_cast(f4_t, wv[wr * 3 + fs] << 16);
                const f4_t wh = __builtin_bit_cast(f4_t, wv[wr * 3 + fs] & 0xffff0000u);
#pragma unroll
                for (int j = 0; j < TW; ++j) {
                    lo[i][j] += xlo[j * STRIDE + fs] * wl;
                    hi[i][j] += xhi[j * STRIDE + fs] * wh;
                }
            }
        }
    }
    f4_t blo = {0.f, 0.f, 0.f, 0.f}, bhi = {0.f, 0.f, 0.f, 0.f};
    if (p.epilogue & ALT_EPI_BIAS) {
        const f4_t b0 = *(const f4_t *)(p.bias + c), b1 = *(const f4_t *)(p.bias + c + 4);
        blo = __builtin_shufflevector(b0, b1, 0, 2, 4, 6);
        bhi = __builtin_shufflevector(b0, b1, 1, 3, 5, 7);
    }
    const float floor_ = (p.epilogue & ALT_EPI_RELU) ? 0.f : __builtin_nanf("");     // (relu_floor takes a register too many here)
    const int32_t yb = dim2_off32(p.yn, n) + dim2_off32(p.yk, c), syh = (int32_t)p.yh.si, syw = (int32_t)p.yw.si;
    float probe = 0.f;                              // NaN once a sum is
#pragma unroll
    for (int i = 0; i < TH; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j) {
            const bool ok = ow0 + j < p.OW && oh0 + i < p.OH;
            const f4_t sa = lo[i][j] + blo, sb = hi[i][j] + bhi;
#pragma unroll
            for (int q = 0; q < 4; ++q) probe = __builtin_elementwise_maximum(__builtin_elementwise_maximum(probe, sa[q]), sb[q]);
            const f4_t a = __builtin_elementwise_max(sa, (f4_t){floor_, floor_, floor_, floor_});
            const f4_t b = __builtin_elementwise_max(sb, (f4_t){floor_, floor_, floor_, floor_});
            w4_t out;
#pragma unroll
            for (int q = 0; q < 4; ++q) out[q] = f32x2_to_bf16x2(a[q], b[q]);
            __builtin_amdgcn_raw_buffer_store_b128(out, yr, (int)(ok ? (uint32_t)(yb + (oh0 + i) * syh + (ow0 + j) * syw) * 2u : kOutOfRange), 0, POLICY);
        }
    // A tap outside the image is no part of the sum, but the zeros read for it were multiplied, and zero times an infinite or NaN
    // filter value is NaN.  Where a sum came out NaN, the outputs of a thread at the border are taken again over the taps inside
    // and stored over those above.
    if (probe != probe) dw_3x3_inside<STRIDE, TW, TH, TAPS, POLICY>(threadIdx.x);
}

// bf16 in and out, width contiguous, 3x3 without dilation, padding 1 along the width, W and OW multiples of TW
// (four or eight; checked by the host together with the alignment of every plane and row).  A thread computes
// outputs (oh, ow0 .. ow0+TW-1) of one (n, c) plane from input columns ow0*STRIDE - 1 .. : the columns from
// ow0*STRIDE on come as aligned vectors of TW elements (wholly inside or wholly outside the row), the one before
// them as a scalar.
template <int STRIDE, int TW>
__global__ __launch_bounds__(kDwThreads) void dwconv_rows_3x3_kernel(const DwParams p)
{
    typedef uint32_t wv_t __attribute__((ext_vector_type(TW / 2)));     // TW bf16: 8 bytes (TW = 4) or 16 (TW = 8)
    constexpr int NCOL = (TW - 1) * STRIDE + 3;            // input columns under TW outputs
    constexpr int NV = (NCOL - 1 + TW - 1) / TW;           // vectors that cover columns 1 .. NCOL-1
    const uint32_t OWB = (uint32_t)p.OW / TW;
    const int64_t total = (int64_t)p.N * p.C * p.OH * OWB;
    const int64_t sxh = p.xh.si, syh = p.yh.si;
    for (int64_t e = blockIdx.x * (int64_t)kDwThreads + threadIdx.x; e < total; e += (int64_t)gridDim.x * kDwThreads) {
        int c, ow0, oh, n;
        if (total <= 0x7fffffff) {
            uint32_t r = (uint32_t)e;
            ow0 = (int)(r % OWB) * TW; r /= OWB;
            oh = (int)(r % (uint32_t)p.OH); r /= (uint32_t)p.OH;
            c = (int)(r % (uint32_t)p.C);
            n = (int)(r / (uint32_t)p.C);
        } else {
            int64_t r = e;
            ow0 = (int)(r % OWB) * TW; r /= OWB;
            oh = (int)(r % p.OH); r /= p.OH;
            c = (int)(r % p.C);
            n = (int)(r / p.C);
        }
        const uint16_t *xb = (const uint16_t *)p.x + dim2_off(p.xn, n) + dim2_off(p.xc, c);
        const uint16_t *wb = (const uint16_t *)p.w + dim2_off(p.wo, c);
        float wq[9];
#pragma unroll
        for (int t = 0; t < 9; ++t)
            wq[t] = __builtin_bit_cast(float, (uint32_t)wb[(t / 3) * p.wr.si + (t % 3) * p.ws.si] << 16);
        float acc[TW];
#pragma unroll
        for (int j = 0; j < TW; ++j) acc[j] = 0.f;
        const int ih0 = oh * STRIDE - p.pad_h, iw1 = ow0 * STRIDE;      // column 1 of the window: a multiple of TW
#pragma unroll
        for (int fr = 0; fr < 3; ++fr) {
            const int ih = ih0 + fr;
            if ((unsigned)ih >= (unsigned)p.H) continue;
            const uint16_t *row = xb + ih * sxh;
            float xv[1 + TW * NV];
            xv[0] = iw1 > 0 ? __builtin_bit_cast(float, (uint32_t)row[iw1 - 1] << 16) : 0.f;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                wv_t d;
                __builtin_memset(&d, 0, sizeof d);
                if (iw1 + TW * v < p.W) d = *(const wv_t *)(row + iw1 + TW * v);
#pragma unroll
                for (int q = 0; q < TW / 2; ++q) {
                    xv[1 + TW * v + 2 * q] = __builtin_bit_cast(float, d[q] << 16);
                    xv[2 + TW * v + 2 * q] = __builtin_bit_cast(float, d[q] & 0xffff0000u);
                }
            }
#pragma unroll
            for (int fs = 0; fs < 3; ++fs)
#pragma unroll
                for (int j = 0; j < TW; ++j) acc[j] += xv[j * STRIDE + fs] * wq[fr * 3 + fs];
        }
        const float bias = (p.epilogue & ALT_EPI_BIAS) ? p.bias[c] : 0.f;
        const float floor_ = relu_floor(p.epilogue & ALT_EPI_RELU);
        wv_t out;
#pragma unroll
        for (int q = 0; q < TW / 2; ++q)
            out[q] = f32x2_to_bf16x2(fmaxf(acc[2 * q] + bias, floor_), fmaxf(acc[2 * q + 1] + bias, floor_));
        uint16_t *yb = (uint16_t *)p.y + dim2_off(p.yn, n) + dim2_off(p.yk, c) + oh * syh + ow0;
        *(wv_t *)yb = out;
    }
}

// every offset of a plane or row start is a multiple of m elements
bool rows_of(int m, const Dim2 *d, int n)
{
    for (int i = 0; i < n; ++i)
        if (d[i].so % m || d[i].si % m) return false;
    return true;
}

// eight consecutive channels from a multiple of eight are one contiguous, 16-byte aligned run
bool chan_runs_of_8(const Dim2 &c, int64_t C, const Dim2 *others, int n_others)
{
    const int64_t run = c.f >= C ? C : c.f;
    if (c.si != 1 || run % 8 || C % 8) return false;
    if (c.f < C && c.so % 8) return false;
    for (int i = 0; i < n_others; ++i)
        if (others[i].so % 8 || others[i].si % 8) return false;
    return true;
}

}  // namespace

// pb is the problem of one group (C = K = 1 per group, batch = channels) as conv_problem fills it for
// a depth-wise descriptor; x/w/y Dim2 entries describe the whole tensors.
alt_status_t depthwise_run(alt_handle_t h, const Problem &pb, int64_t N, int64_t C, hipStream_t st)
{
    if (!h->has_gpu) return fail(h, ALT_HIP_ERROR, "no GPU device available");
    const IgemmParams &q = pb.p;
    DwParams p;
    std::memset(&p, 0, sizeof p);
    p.x = q.x; p.w = q.w; p.bias = q.bias; p.y = q.y;
    p.N = (int32_t)N; p.C = (int32_t)C; p.H = q.H; p.W = q.W; p.R = q.R; p.S = q.S; p.OH = q.OH; p.OW = q.OW;
    p.stride_h = q.stride_h; p.stride_w = q.stride_w; p.pad_h = q.pad_h; p.pad_w = q.pad_w;
    p.dil_h = q.dil_h; p.dil_w = q.dil_w;
    p.epilogue = q.epilogue; p.in_bf16 = pb.dtype == ALT_BF16; p.out_bf16 = q.out_bf16;
    p.xn = q.xn; p.xc = q.xc; p.xh = q.xh; p.xw = q.xw;
    p.wo = q.wo; p.wr = q.wr; p.ws = q.ws;
    p.yn = q.yn; p.yk = q.yk; p.yh = q.yh; p.yw = q.yw;
    p.chan_fast = q.yk.si == 1;
    const Dim2 xo[3] = {q.xn, q.xh, q.xw}, wo_[2] = {q.wr, q.ws}, yo[3] = {q.yn, q.yh, q.yw};
    // filters: eight channels a 16-byte run per tap, or (taps) the taps of a channel side by side
    const bool taps = q.wo.f >= C && q.wo.si == q.R * q.S && q.wr.f >= q.R && q.wr.si == q.S && q.ws.f >= q.S && q.ws.si == 1;
    const bool wchan = chan_runs_of_8(q.wo, C, wo_, 2);
    bool vec = p.in_bf16 && p.out_bf16 && chan_runs_of_8(q.xc, C, xo, 3) && (taps || wchan) && chan_runs_of_8(q.yk, C, yo, 3) &&
               (uintptr_t)q.x % 16 == 0 && (uintptr_t)q.w % 16 == 0 && (uintptr_t)q.y % 16 == 0 &&
               (!(q.epilogue & ALT_EPI_BIAS) || (uintptr_t)q.bias % 16 == 0);
    // Images a launch of the 3x3 vector kernel takes: its offsets are 32 bits, so larger batches (outermost, or the images of a
    // launch would not lie together) go in several launches below 2 GiB.
    const int64_t x_image = C * q.H * q.W, y_image = C * q.OH * q.OW;
    int64_t images = std::min(N, ((1 << 30) - 1) / std::max(x_image, y_image));
    if (images < N && !(q.xn.f >= N && q.xn.si == x_image && q.yn.f >= N && q.yn.si == y_image)) images = 0;
    const bool k3x3 = vec && q.R == 3 && q.S == 3 && q.dil_h == 1 && q.dil_w == 1 && q.stride_h == q.stride_w &&
                      (q.stride_h == 1 || q.stride_h == 2) && q.xh.f >= q.H && q.xw.f >= q.W && q.yh.f >= q.OH &&
                      q.yw.f >= q.OW && images > 0;
    if (k3x3) {
        // Rows per thread.  Two share their windows' rows (24 loads for eight outputs against 36) where one row each
        // would make more threads than the chip holds one wave of per SIMD: 16 x 144 x 56 x 56 took 10.0 us with two
        // and 11.5 with one (before outputs were written through), but 1 x 144 x 56 x 56 4.8 and 3.9.  At stride 2 they share one row of three, and the
        // registers they take cost more than that (16 x 96 x 112 x 112: 23 us with two, 12.0 with one).
        const int64_t items1 = N * q.OH * ((q.OW + kDwCols - 1) / kDwCols) * (C / 8);
        const int th = q.stride_h == 1 && items1 >= 65536 ? 2 : 1;
        const uint32_t owb = (uint32_t)(q.OW + kDwCols - 1) / kDwCols, ohb = (uint32_t)(q.OH + th - 1) / th;
        p.fd_c8 = make_fastdiv((uint32_t)C / 8);
        p.fd_owb = make_fastdiv(owb);
        p.fd_ohb = make_fastdiv(ohb);
        auto kernel = [&](auto policy) {
            constexpr int P = decltype(policy)::value;
            return th == 2             ? (taps ? dwconv_vec8_3x3_kernel<1, kDwCols, 2, true, P> : dwconv_vec8_3x3_kernel<1, kDwCols, 2, false, P>)
                 : q.stride_h == 1 ? (taps ? dwconv_vec8_3x3_kernel<1, kDwCols, 1, true, P> : dwconv_vec8_3x3_kernel<1, kDwCols, 1, false, P>)
                                   : (taps ? dwconv_vec8_3x3_kernel<2, kDwCols, 1, true, P> : dwconv_vec8_3x3_kernel<2, kDwCols, 1, false, P>);
        };
        auto kern = N * y_image * 2 <= 32 << 20 ? kernel(std::integral_constant<int, kWriteThrough>{}) : kernel(std::integral_constant<int, 0>{});
        for (int64_t n = 0; n < N; n += images) {
            const int64_t here = std::min(images, N - n);
            p.x = (const uint16_t *)q.x + n * x_image;
            p.y = (uint16_t *)q.y + n * y_image;
            p.items = (uint32_t)(here * ohb * owb * (C / 8));
            p.x_bytes = (uint32_t)(here * x_image * 2);
            p.y_bytes = (uint32_t)(here * y_image * 2);
            hipLaunchKernelGGL(kern, dim3((p.items + kDwThreads - 1) / kDwThreads), dim3(kDwThreads), 0, st, p);
            ALT_CHECK_HIP(h, hipGetLastError());
        }
        return ALT_OK;
    }
    // Filters whose taps lie side by side, beyond 3x3: a thread of the vector kernel loads eight scattered filter values per tap,
    // which pays once the element kernel's eight times as many threads fill the chip (5x5 at stride 2: 1 x 480 x 28 x 28, 11760
    // vectors, 17.4 us against 12.2; 2 x 120 x 75 x 75, 43320, 17.1 and 16.9; 1 x 360 x 70 x 70, 55125, 17.6 and 23.7), or where
    // 8, 16 or 32 channels let a wave's lanes share the values (5 x 8 x 67 x 67, 22445 vectors, 10.0 and 12.3).
    const int64_t vectors = N * q.OH * q.OW * (C / 8);
    if (!wchan && vectors < 49152 && C != 8 && C != 16 && C != 32) vec = false;
    const Dim2 xr[3] = {q.xn, q.xc, q.xh}, yr[3] = {q.yn, q.yk, q.yh};
    const bool rows = !vec && p.in_bf16 && p.out_bf16 && q.R == 3 && q.S == 3 && q.dil_h == 1 && q.dil_w == 1 &&
                      q.stride_h == q.stride_w && (q.stride_h == 1 || q.stride_h == 2) && q.pad_w == 1 && q.xw.si == 1 &&
                      q.xw.f >= q.W && q.xh.f >= q.H && q.yw.si == 1 && q.yw.f >= q.OW && q.yh.f >= q.OH && q.wr.f >= 3 &&
                      q.ws.f >= 3 && q.W % 4 == 0 && q.OW % 4 == 0 && rows_of(4, xr, 3) && rows_of(4, yr, 3) &&
                      (uintptr_t)q.x % 8 == 0 && (uintptr_t)q.y % 8 == 0;
    // eight outputs per thread in 16-byte accesses where the rows allow it
    const bool rows8 = rows && q.W % 8 == 0 && q.OW % 8 == 0 && rows_of(8, xr, 3) && rows_of(8, yr, 3) &&
                       (uintptr_t)q.x % 16 == 0 && (uintptr_t)q.y % 16 == 0;
    const int64_t work = rows ? N * C * q.OH * (q.OW / (rows8 ? 8 : 4))
                            : N * q.OH * q.OW * (vec ? C / 8 : C);
    const unsigned blocks = (unsigned)std::min<int64_t>((work + kDwThreads - 1) / kDwThreads, 256 * 64);
    if (rows8 && q.stride_h == 1) hipLaunchKernelGGL((dwconv_rows_3x3_kernel<1, 8>), dim3(blocks), dim3(kDwThreads), 0, st, p);
    else if (rows8) hipLaunchKernelGGL((dwconv_rows_3x3_kernel<2, 8>), dim3(blocks), dim3(kDwThreads), 0, st, p);
    else if (rows && q.stride_h == 1) hipLaunchKernelGGL((dwconv_rows_3x3_kernel<1, 4>), dim3(blocks), dim3(kDwThreads), 0, st, p);
    else if (rows) hipLaunchKernelGGL((dwconv_rows_3x3_kernel<2, 4>), dim3(blocks), dim3(kDwThreads), 0, st, p);
    else if (vec && wchan) hipLaunchKernelGGL(dwconv_vec8_kernel<false>, dim3(blocks), dim3(kDwThreads), 0, st, p);
    else if (vec) hipLaunchKernelGGL(dwconv_vec8_kernel<true>, dim3(blocks), dim3(kDwThreads), 0, st, p);
    else hipLaunchKernelGGL(dwconv_elem_kernel, dim3(blocks), dim3(kDwThreads), 0, st, p);
    ALT_CHECK_HIP(h, hipGetLastError());
    return ALT_OK;
}

}  // namespace alt
