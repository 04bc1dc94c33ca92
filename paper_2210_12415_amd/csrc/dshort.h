// Products over a short reduction: C[M][N] = A[M][K] * B[N][K]^T with K up to 256, dense, bf16 in and out (the scores of attention heads, and
// 1x1 convolutions over few channels in NHWC), batched or not.
//
// Such a product is bound by its output's and its left operand's way from and to memory, not by matrix instructions, and has no loop worth
// a pipeline.  A workgroup of four waves brings the whole reduction of its 128 x 32 TN tile into LDS at once (direct-to-LDS loads, all in flight
// together), waits once, multiplies, and stores through LDS; what covers the waiting are the other three or so workgroups on the compute
// unit: 20 to 28 KB of LDS each for 64 channels and 32 to 96 columns.
//
// Output rows may have any length: a lane stores eight columns at once, at any even address, and the last ones of a row one by one.
// (The tile kernels of dstream.h store four aligned columns at least; other products ran on register-staged kernels.)
//
// Without this kernel and with it: scores of 12 x 37 x 37 x 64 6.7 us and 3.5, 120 x 367 x 367 x 64 29.8 and 13.0 (40 MB out: 3 TB/s), 260 x 280 x 280 x 64
// 36.7 and 13.7; 16 x 56 x 56, 24 channels to 144 with bias 8.8 and 7.5, 144 to 24 5.9 and 4.3; 256 x 56 x 56, 256 to 64 118 and 113.5 (411 MB fetched and 103 written, 4.5
// TB/s: every kernel tried there ends between 112 and 120; two column tiles ask the L2s for 9.6 M lines, 58 % hits).  Over 5600 random products and 1x1
// layers in its range the choice with this kernel takes 0.74 of the time without.
#pragma once

#include "dplanar.h"

namespace alt {

constexpr int kShortRows = 128;           // rows of a tile: 32 per wave
constexpr int kShortStages = 4;           // most K stages of 64

inline size_t dshort_lds_bytes(int BN, int64_t C)
{
    const size_t stages = (size_t)(C + 63) / 64;
    return std::max(stages * (kShortRows + BN) * 128, (size_t)kShortRows * (BN * 2 + 16));
}

template <int TN, int KS>
__global__ __launch_bounds__(256, TN <= 2 ? 4 : 3) void dshort_kernel(const DconvParams p)
{
    constexpr int BN = 32 * TN, A_STAGE = kShortRows * 128, B_STAGE = BN * 128;
    constexpr int SPB = BN * 2 + 16;                       // staging pitch of a row in bytes
    extern __shared__ uint4 smem_u4[];
    char *smem = (char *)smem_u4;                          // A's stages, B's stages; then the staging
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem_u4;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

    // tiles of an entry one after the other, columns fastest, on one XCD
    const int tiles = p.tiles_m * p.tiles_n, logical = igemm_logical_tile(tiles * p.batch);
    const int entry = (int)div32((uint32_t)logical, p.d_od), tile = logical - entry * tiles;
    const int mt = (int)div32((uint32_t)tile, p.d_tn), nt = tile - mt * p.tiles_n;
    const int m0 = mt * kShortRows, n0 = nt * BN;
    const i32x4_t x_rsrc = make_rsrc((const char *)p.x + (int64_t)entry * p.x_bstride, p.x_bytes);
    const i32x4_t w_rsrc = make_rsrc((const char *)p.w + (int64_t)entry * p.w_bstride, p.w_bytes);

    // slot s of a stage holds chunk (s % 8) ^ (row / 2 % 8) of row s / 8, as in dstream.h; rows past the last one lie behind the operand's end
    // and chunks past a row's are given an offset there: both read zeros
    auto load = [&](i32x4_t rsrc, int row0, int j, int ks, uint32_t lds) {
        const int s = j * 64 + lane, row = s >> 3, chunk = ks * 8 + ((s & 7) ^ ((row >> 1) & 7));
        dma_load16_s(rsrc, chunk < p.c16 ? (uint32_t)(row0 + row) * p.x_pix + (uint32_t)chunk * 16u : kOutOfRange, 0u, lds + (uint32_t)j * 1024u);
    };
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int i = 0; i < 4; ++i) load(x_rsrc, m0, wave * 4 + i, ks, lds0 + ks * A_STAGE);
#pragma unroll
        for (int i = 0; i < TN; ++i) load(w_rsrc, n0, i * 4 + wave, ks, lds0 + KS * A_STAGE + ks * B_STAGE);
    }
    floatx16_t acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
    wait_vmcnt<0>();
    lds_barrier();

    const int r = lane & 31, khalf = lane >> 5;
    const char *a_row = smem + (wave * 32 + r) * 128, *b_row = smem + KS * A_STAGE + r * 128;
    const int swz = ((r >> 1) & 7) * 16;                   // (rows 32 apart have the same)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            const int at = (kc * 32 + khalf * 16) ^ swz;
            const u32x4_t a = *(const u32x4_t *)(a_row + ks * A_STAGE + at);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const u32x4_t b = *(const u32x4_t *)(b_row + ks * B_STAGE + j * (32 * 128) + at);
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, b), __builtin_bit_cast(bf16x8_t, a), acc[j], 0, 0, 0);
            }
        }
    __syncthreads();                                       // every wave is done with the operands

    // lane: row r, columns 8 q + 4 khalf .. + 3 of each 32; a wave reads back only what it wrote
    const float floor_ = relu_floor(p.flags & ALT_EPI_RELU);
    char *stg = smem + wave * (32 * SPB);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = j * 32 + q * 8 + khalf * 4;
            float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
            if ((p.flags & ALT_EPI_BIAS) && n0 + c < p.Nc) b = *(const float4 *)(p.bias + n0 + c);
            const float o0 = fmaxf(acc[j][4 * q] + b.x, floor_), o1 = fmaxf(acc[j][4 * q + 1] + b.y, floor_);
            const float o2 = fmaxf(acc[j][4 * q + 2] + b.z, floor_), o3 = fmaxf(acc[j][4 * q + 3] + b.w, floor_);
            *(uint2 *)(stg + r * SPB + c * 2) = make_uint2(f32x2_to_bf16x2(o0, o1), f32x2_to_bf16x2(o2, o3));
        }
    uint16_t *y = (uint16_t *)((char *)p.y + (int64_t)entry * p.y_bstride);
    constexpr int LPR = BN / 8;                            // lanes per row
#pragma unroll
    for (int it = 0; it < 32 * LPR / 64; ++it) {
        const int i = it * 64 + lane, row = i / LPR, c = (i - row * LPR) * 8;
        const int m = m0 + wave * 32 + row, n = n0 + c;
        const u32x4_t v = *(const u32x4_t *)(stg + row * SPB + c * 2);
        if (m >= p.M || n >= p.Nc) continue;
        uint16_t *dst = y + (int64_t)m * p.Nc + n;
        if (n + 8 <= p.Nc) {
            ((PlanarRun *)dst)->v = v;
        } else {
#pragma unroll
            for (int e = 0; e < 7; ++e)
                if (n + e < p.Nc) dst[e] = (uint16_t)(v[e / 2] >> (e % 2 * 16));
        }
    }
}

template <int TN, int KS>
hipError_t dshort_launch_ks(const DconvParams &p, size_t lds, hipStream_t st)
{
    auto kern = dshort_kernel<TN, KS>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_m * p.tiles_n * p.batch)), dim3(256), lds, st, p);
    return hipGetLastError();
}

template <int TN>
hipError_t dshort_launch(const DconvParams &p, size_t lds, hipStream_t st)
{
    switch ((p.C + 63) / 64) {
    case 1: return dshort_launch_ks<TN, 1>(p, lds, st);
    case 2: return dshort_launch_ks<TN, 2>(p, lds, st);
    case 3: if constexpr (TN <= 2) return dshort_launch_ks<TN, 3>(p, lds, st); break;
    case 4: if constexpr (TN <= 2) return dshort_launch_ks<TN, 4>(p, lds, st); break;
    }
    return hipErrorInvalidValue;
}

}  // namespace alt
