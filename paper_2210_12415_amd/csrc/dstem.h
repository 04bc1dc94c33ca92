// Direct convolution for images of few channels: the first layer of a network, which reads what a decoder or a camera
// delivers (planar NCHW, one to four channels) and stores what the next layer wants (NHWC or channel-blocked).
//
// The matrix cores take eight consecutive reduction elements of a pixel per lane.  Three channels give no such run, but
// the filter's columns do: the eight input columns from a window's left edge on lie side by side in the image row.  So
// the reduction runs over (channel, filter row) in chunks of eight columns: a chunk of a lane is 16 bytes of the input
// row its pixel's window starts in, read straight out of a patch of image rows in LDS at any even column.  Columns past
// the filter's width are cleared in the fragment and carry zero weights (a 7-wide filter uses 7 of 8).
//
// A workgroup of four waves walks tiles of 16 x 16 output pixels x all or 32 * TN output channels.  The filter stays in
// registers for the whole launch (2 * NKC chunks x TN tiles of 32 channels); per tile the patch of (15 * stride + R)
// rows of each channel comes in through registers while the previous tile computes.  A row tile of the matrix
// instruction is 2 x 16 pixels.  Results are rounded, transposed through LDS, and stored 16 bytes per lane.
//
// 16 images of 3 x 224 x 224, 64 channels of 7 x 7 at stride 2 (30 MB, 3.8 GFLOP): 14.6 us, 2.1 TB/s, against 118 us on the
// element-gather kernel; 64 images 42 us, 2.9 TB/s. What bounds it is what two waves per SIMD cannot hide: per matrix
// instruction 18 vector instructions (window masks, rounding, the transpose, addresses, the filter's way into registers) keep
// the vector units busy a third of the time, LDS is active another third with two of five cycles lost to bank conflicts
// (windows start at any even column), and a wave waits 55 % of its life; the matrix cores are busy 8 %.
#pragma once

#include "dconv.h"

namespace alt {

constexpr int kStemTile = 16;             // output rows and columns of a tile
constexpr int kStemMaxLoads = 8;          // 16-byte pieces of a patch per thread

// LDS bytes: the patch (two copies, one column apart, where odd strides need odd columns) or, before it, the filter's rows;
// beside that zeros, biases, and the output staging or, before the first tile, the filter's chunks
inline int dstem_patch_bytes(int tn, int filter_row, int patch_pieces)
{
    const int rows = (32 * tn * filter_row * 2 + 15) / 16 * 16;
    return patch_pieces * 16 > rows ? patch_pieces * 16 : rows;
}
inline size_t dstem_lds_bytes(int chunks, int tn, int patch_bytes)
{
    const size_t stage = (size_t)4 * 32 * (tn * 64 + 16), filter = (size_t)32 * tn * chunks * 16;
    return (size_t)patch_bytes + 16 + tn * 128 + (stage > filter ? stage : filter);
}

// Patch geometry: pieces of eight columns per row, rows per channel, copies.
inline __host__ __device__ int dstem_pieces(int stride_w) { return ((kStemTile - 1) * stride_w + 8 + 7) / 8; }
inline __host__ __device__ int dstem_rows(int stride_h, int R) { return (kStemTile - 1) * stride_h + R; }
inline __host__ __device__ int dstem_copies(int stride_w) { return stride_w % 2 ? 2 : 1; }

// NL: 16-byte pieces of the patch per thread.
template <int NKC, int TN, int NL>
__global__ __launch_bounds__(256, 2) void dstem_kernel(const DconvParams p)
{
    extern __shared__ uint4 smem_u4[];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int khalf = lane >> 5, px = lane & 31, prow = px >> 4, pcol = px & 15;
    const int chunks = p.C * p.R;                          // chunks of the reduction (<= 2 * NKC)
    const int PCH = dstem_pieces(p.stride_w), PR = dstem_rows(p.stride, p.R), NCP = dstem_copies(p.stride_w);
    const int pitch = PCH * 16;                            // bytes of a patch row
    const int copy_bytes = p.C * PR * pitch;
    const int pieces = NCP * p.C * PR * PCH;
    char *patch = (char *)smem_u4, *zero = patch + p.ncc, *biases = zero + 16, *stage = biases + TN * 128;
    const int n0 = blockIdx.y * (32 * TN);

    // ---- the patch of a tile: piece i = (copy, channel, row, eight columns) ---------------------------------------------
    const uint16_t *xg = (const uint16_t *)p.x;
    const int total = p.in_px * p.C;                       // elements of x (at least eight)
    int rel[NL], place[NL];                                // element offset from the patch's first pixel; row << 16 | column
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const int i = min(l * 256 + t, pieces - 1);
        const uint32_t rest = div32((uint32_t)i, p.d_c16);             // i / PCH
        const int pc = i - (int)rest * PCH;
        const uint32_t plane = div32(rest, p.d_rs);                    // / PR
        const int row = (int)rest - (int)plane * PR;
        const int copy = (int)plane >= p.C, c = (int)plane - (copy ? p.C : 0);
        rel[l] = (c * p.H + row) * p.W + pc * 8 + copy;
        place[l] = row << 16 | (pc * 8 + copy);
    }
    auto tile_at = [&](int tile, int &img, int &oh0, int &ow0) {
        const uint32_t r = div32((uint32_t)tile, p.d_w);   // tiles per row of tiles
        ow0 = (int)((uint32_t)tile - r * (uint32_t)p.tiles_n) * kStemTile;
        const uint32_t im = div32(r, p.d_hw);              // rows of tiles per image
        oh0 = (int)(r - im * (uint32_t)p.splitk) * kStemTile;
        img = (int)im;
    };
    typedef uint32_t w4_t __attribute__((ext_vector_type(4)));
    w4_t in[NL];
    auto load_patch = [&](int tile) {                      // every load inside x, none waits for another
        int img, oh0, ow0;
        tile_at(tile, img, oh0, ow0);
        const int e0 = (img * p.C * p.H + oh0 * p.stride - p.pad_h) * p.W + ow0 * p.stride_w - p.pad_w;
#pragma unroll
        for (int l = 0; l < NL; ++l) __builtin_memcpy(&in[l], xg + max(0, min(e0 + rel[l], total - 8)), 16);
    };
    auto store_patch = [&](int tile) {                     // masked to the image, into LDS
        int img, oh0, ow0;
        tile_at(tile, img, oh0, ow0);
        const int ih0 = oh0 * p.stride - p.pad_h, iw0 = ow0 * p.stride_w - p.pad_w;
        const int e0 = (img * p.C * p.H + ih0) * p.W + iw0;
        const bool border = iw0 < 0 || iw0 + PCH * 8 + 1 > p.W || ih0 < 0 || ih0 + PR > p.H;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int i = l * 256 + t;
            w4_t v = in[l];
            if (border) {
                const int e = e0 + rel[l], d = e - max(0, min(e, total - 8));
                if (d != 0) {                              // moved to stay inside x: back by d elements
                    const uint64_t lo = (uint64_t)v[1] << 32 | v[0], hi = (uint64_t)v[3] << 32 | v[2];
                    uint64_t nlo = 0, nhi = 0;
                    const int k = (d < 0 ? -d : d) * 16;   // bits; 128 and more leave nothing
                    if (d < 0) {
                        if (k < 64) { nlo = lo << k; nhi = hi << k | (lo >> 1) >> (63 - k); }
                        else if (k < 128) nhi = lo << (k - 64);
                    } else {
                        if (k < 64) { nhi = hi >> k; nlo = lo >> k | (hi << 1) << (63 - k); }
                        else if (k < 128) nlo = hi >> (k - 64);
                    }
                    v = (w4_t){(uint32_t)nlo, (uint32_t)(nlo >> 32), (uint32_t)nhi, (uint32_t)(nhi >> 32)};
                }
                const int iw = iw0 + (place[l] & 0xffff);
                const bool row_ok = (unsigned)(ih0 + (place[l] >> 16)) < (unsigned)p.H;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[q] &= (row_ok && (unsigned)(iw + 2 * q) < (unsigned)p.W ? 0xffffu : 0u) |
                            (row_ok && (unsigned)(iw + 2 * q + 1) < (unsigned)p.W ? 0xffff0000u : 0u);
            }
            if (i < pieces) *(w4_t *)(patch + i * 16) = v;
        }
    };
    int tile = blockIdx.x;
    load_patch(tile);

    // ---- the filter: rows as they lie into LDS (coalesced), from there as chunks, into registers ----------------------------
    {
        constexpr int NW = (32 * TN * 2 * NKC + 255) / 256;
        const int row_elems = p.wst_o, valid = min(32 * TN, p.Nc - n0) * row_elems;
        const uint16_t *wg = (const uint16_t *)p.w + n0 * row_elems;
        uint16_t *raw = (uint16_t *)smem_u4;
        for (int i = t * 8; i + 8 <= valid; i += 256 * 8) {
            w4_t v;
            __builtin_memcpy(&v, wg + i, 16);
            *(w4_t *)(raw + i) = v;
        }
        if (t < (valid & 7)) raw[(valid & ~7) + t] = wg[(valid & ~7) + t];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const int i = min(k * 256 + t, 32 * TN * 2 * NKC - 1), q = i / (32 * TN), n = i - q * (32 * TN);
            const bool ok = q < chunks && n0 + n < p.Nc;
            const int qq = ok ? q : 0, nn = ok ? n : 0;
            const uint32_t c = div32((uint32_t)qq, p.d_s); // q / R
            const uint16_t *row = raw + nn * row_elems + (int)c * p.wst_i + (qq - (int)c * p.R) * p.wst_r;
            uint32_t e[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) e[s] = row[min(s, p.S - 1) * p.wst_s];
            w4_t v;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = (ok && 2 * j < p.S ? e[2 * j] : 0u) | (ok && 2 * j + 1 < p.S ? e[2 * j + 1] << 16 : 0u);
            *(w4_t *)(stage + i * 16) = v;
        }
    }
    __syncthreads();                                       // (the rows' place is the patch's)
    if (t == 0) *(uint4 *)zero = make_uint4(0, 0, 0, 0);
    if (t < 32 * TN) ((float *)biases)[t] = (p.flags & ALT_EPI_BIAS) && n0 + t < p.Nc ? p.bias[n0 + t] : 0.f;
    __syncthreads();
    u32x4_t bf[NKC][TN];
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc)
#pragma unroll
        for (int j = 0; j < TN; ++j) bf[kc][j] = *(const u32x4_t *)(stage + ((2 * kc + khalf) * 32 * TN + j * 32 + px) * 16);
    // this lane's chunks: byte offset from the window's first row and channel (past the last chunk: negative)
    int off[NKC];
    u32x4_t mask;                                          // columns past the filter
#pragma unroll
    for (int q = 0; q < 4; ++q) mask[q] = (2 * q < p.S ? 0xffffu : 0u) | (2 * q + 1 < p.S ? 0xffff0000u : 0u);
#pragma unroll
    for (int kc = 0; kc < NKC; ++kc) {
        const int q = 2 * kc + khalf;
        const uint32_t c = div32((uint32_t)q, p.d_s);
        off[kc] = q < chunks ? ((int)c * PR + (q - (int)c * p.R)) * pitch : -1;
    }
    const float floor_ = relu_floor(p.flags & ALT_EPI_RELU);
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(p.y, 0, (int)p.y_bytes, 0x00020000);
    const int odd = (pcol * p.stride_w) & 1;
    constexpr int SP = TN * 64 + 16;                       // staging pitch of a pixel in bytes
    char *stg = stage + wave * (32 * SP);

    for (; tile < p.tiles_m; tile += gridDim.x) {
        __syncthreads();                                   // the previous tile (or the filter) is read
        store_patch(tile);
        __syncthreads();
        int img, oh0, ow0;
        tile_at(tile, img, oh0, ow0);
        if (tile + (int)gridDim.x < p.tiles_m) load_patch(tile + gridDim.x);
#pragma unroll 1
        for (int u = 0; u < 2; ++u) {
            const int orow = (wave * 2 + u) * 2;           // first of the row tile's two output rows
            const char *base = patch + odd * copy_bytes + (orow + prow) * p.stride * pitch + (pcol * p.stride_w - odd) * 2;
            u32x4_t a[NKC];
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc)
                __builtin_memcpy(&a[kc], __builtin_assume_aligned(off[kc] < 0 ? zero : base + off[kc], 4), 16);
            floatx16_t acc[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
#pragma unroll
            for (int kc = 0; kc < NKC; ++kc) {
                a[kc] &= mask;
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, bf[kc][j]), __builtin_bit_cast(bf16x8_t, a[kc]), acc[j], 0, 0, 0);
            }
            // lane: pixel px, channels 8*g + 4*khalf .. + 3 of each 32-channel tile
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4_t b = *(const f32x4_t *)(biases + (j * 32 + g * 8 + khalf * 4) * 4);
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = fmaxf(acc[j][4 * g + e] + b[e], floor_);
                    *(uint2 *)(stg + px * SP + j * 64 + g * 16 + khalf * 8) = make_uint2(f32x2_to_bf16x2(o[0], o[1]), f32x2_to_bf16x2(o[2], o[3]));
                }
            // (a wave reads back only what it wrote; the compiler orders these accesses)
            constexpr int LPP = TN * 4;                    // 16-byte pieces per pixel
#pragma unroll
            for (int it = 0; it < (32 * LPP) / 64; ++it) {
                const int i = it * 64 + lane, q = i / LPP, g = i - q * LPP;
                const u32x4_t ov = *(const u32x4_t *)(stg + q * SP + g * 16);
                const int oh = oh0 + orow + (q >> 4), ow = ow0 + (q & 15), n = n0 + g * 8;
                const bool ok = oh < p.OH && ow < p.OW && n < p.Nc;
                uint32_t el;
                if (p.y_blk == 0) el = (uint32_t)((img * p.OH + oh) * p.OW + ow) * (uint32_t)p.Nc + (uint32_t)n;
                else el = (uint32_t)img * (uint32_t)(p.Nc * p.OH * p.OW) +
                          (((((uint32_t)n >> p.y_blk) * (uint32_t)(p.OH * p.OW) + (uint32_t)(oh * p.OW + ow)) << p.y_blk) | ((uint32_t)n & ((1u << p.y_blk) - 1)));
                __builtin_amdgcn_raw_buffer_store_b128(ov, yr, (int)(ok ? el * 2u : kOutOfRange), 0, kWriteThrough);
            }
        }
    }
}

template <int NKC, int TN>
hipError_t dstem_launch(const DconvParams &p, size_t lds, hipStream_t st)
{
    const unsigned nt = (unsigned)((p.Nc + 32 * TN - 1) / (32 * TN));
    // as many workgroups as the registers let share the compute units: four with one channel tile, two with two
    const unsigned slots = TN == 1 ? 1024u : 512u, most = slots / nt > 0 ? slots / nt : 1u;
    const int pieces = dstem_copies(p.stride_w) * p.C * dstem_rows(p.stride, p.R) * dstem_pieces(p.stride_w);
    auto kern = pieces <= 3 * 256 ? dstem_kernel<NKC, TN, 3> : dstem_kernel<NKC, TN, kStemMaxLoads>;
    hipLaunchKernelGGL(kern, dim3((unsigned)p.tiles_m < most ? (unsigned)p.tiles_m : most, nt), dim3(256), lds, st, p);
    return hipGetLastError();
}

}  // namespace alt
