// Patch-resident convolution over slabs of channels, for bf16 on gfx950: NHWC activations, OHWI weights, any number of
// channels that is a multiple of eight, stride 1, 3x3 filters (2-D, or of a 3-D convolution any number of them one behind the
// other in depth) and the output phases of transposed convolutions that have 2x2 taps a slice.
//
// The kernels over filter taps (dstream.h) fetch a pixel once per tap: nine times through L2 for a 3x3 filter, 27 times for
// 3x3x3, and delivery from L2 is what bounds them.  The patch-resident kernel of dconv.h fetches it once, but holds all
// channels of a slice and is unrolled over them, so that it takes 64, 128, 256 or 512 channels only.  Here the reduction is cut
// into slabs of BK channels of one depth tap.  A slab's patch (the tile's BM pixels and the filter's reach) is one of two
// buffers: while the KR x KR taps of a slab run as one straight piece of code, the next slab's patch arrives in the other, a few
// direct-to-LDS loads a step, beside the weights, which stream through a ring of NS stages NS - 1 steps ahead.  A last slab of fewer
// channels, and the slabs that even out K groups, read zeros behind the last channel (in LDS and in the weights).
//
// Depth: the pixels of output plane od all lie over input plane od + t, so a plane outside the volume is one whose pixels are
// zeros in that slab's patch, and the rows' addresses are the same for every depth tap.  A tap outside the image inside a plane
// reads the zero area behind the patch buffer, on the banks of the pixel it replaces, as in dconv.h.
//
// No read from LDS is in flight where slabs meet, so the loop over slabs may branch (see dstream.h).
// K groups (KW): group kg takes slabs kg, kg + KW, ... with a ring and patch buffers of its own; sums as in dconv.h.
#pragma once

#include "dconv.h"

namespace alt {

// Stages of the weight ring.
constexpr int slab_stages(int KR, int BK) { return KR == 3 && BK == 64 ? 3 : KR * KR; }
// Wave-loads of the next patch that a wave issues in step u of a slab, PN in all: over the first steps, so that the last of them
// has landed when the slab ends.  (A kernel issues exactly PN, past the patch's end zeros onto the zero area, so that the waits can
// count; such loads cost as much as real ones, so there is a kernel for each of a few PN: with six where four were needed the phases of a
// transposed 128 -> 64 x 4x4x4 took 26.7 us, not 24.6.)
constexpr int slab_load_steps(int KR) { return KR == 3 ? 6 : 2; }
constexpr int slab_loads(int KR, int PN, int u)
{
    const int steps = slab_load_steps(KR), at = (u + 2 * KR * KR) % (KR * KR);
    return at < steps ? (at + 1) * PN / steps - at * PN / steps : 0;
}
constexpr int kSlabLoads[3] = {4, 6, 9};                   // the PN there are
constexpr int kSlabZero = 1024;                            // bytes of zeros behind a patch buffer: one wave-load

// Bytes of a patch buffer of np pixels, with its zero area.
inline __host__ __device__ uint32_t slab_patch_bytes(int np, int BK)
{
    const uint32_t slots = (uint32_t)np * (uint32_t)(BK / 8 + 1);
    return ((slots + 63) / 64) * 1024u + kSlabZero;
}

// (buffers: 1 where no group has a second slab)
inline size_t dslab_lds_bytes(int BM, int BN, int BK, int KR, int waves_n, int kw, int np, int buffers)
{
    const size_t main_loop = (size_t)kw * ((size_t)slab_stages(KR, BK) * BN * BK * 2 + buffers * (size_t)slab_patch_bytes(np, BK));
    const size_t staging = (size_t)kw * BM * (BN + 8 * waves_n) * 4 + 16;
    return main_loop > staging ? main_loop : staging;
}

// Wave-loads that a wave has issued behind those the barrier of step `tap` waits for: the next step's weights (issued NS - 2 steps
// ago, each step's weights before its share of a patch) and, in a slab's first step, the patch.
template <int KR, int BK, int NLB, int PN>
constexpr int slab_loads_behind(int tap)
{
    constexpr int RS = KR * KR, NS = slab_stages(KR, BK);
    int n = 0;
    for (int u = tap + 2 - NS; u < tap; ++u) n += (u > tap + 2 - NS ? NLB : 0) + slab_loads(KR, PN, u);
    const int patch = (RS - slab_load_steps(KR)) * NLB;
    return tap == 0 && patch < n ? patch : n;
}

template <int BM, int BN, int WGM, int WGN, int KW, int BK, int KR, int PN>
__device__ __forceinline__ void dslab_body(const DconvParams &p, int tiles, int bx, int by)
{
    constexpr int NWG = WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    constexpr int RS = KR * KR, NKC = BK / 16, NG = RS * NKC;   // taps, k chunks of a step and of a slab
    constexpr int CPR = BK / 8, SPP = CPR + 1;                  // 16-byte chunks of a weight row; slots of a patch pixel (one unused)
    constexpr int RP = 256 / (BK * 2);
    constexpr int NS = slab_stages(KR, BK), B_STAGE = BN * BK * 2;
    constexpr int NLB = B_STAGE / 1024 / NWG;
    static_assert(WTM % 32 == 0 && WTN % 32 == 0 && TM >= 1 && TN >= 1, "wave tile");
    static_assert(B_STAGE % (1024 * NWG) == 0 && NLB >= 1, "a weight stage is a whole number of wave-loads per wave");
    static_assert(RS % NS == 0 && NS >= 3, "a slab is whole rounds over the ring");
    static_assert(NS * NLB + 2 * PN < 60, "pipeline depth against the vmcnt range");

    extern __shared__ uint4 smem_u4[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem_u4;

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int kg = wave / NWG, wq = wave % NWG;
    const int wm = wq / WGN, wn = wq % WGN;

    int mt, nt;
    dconv_tile_unsliced(p, tiles, bx, mt, nt);
    const int m0 = mt * BM, n0 = nt * BN;
    int f_d = 0, f_h = 0, f_w = 0;                         // the phase's first tap in the common window
    int64_t y_phase = 0;
    if (p.phases > 1) {
        const uint32_t bz = (uint32_t)by;
        const uint32_t pd = div32(bz, p.d_phw), phw = bz - pd * (uint32_t)(p.ph_sh * p.ph_sw);
        const uint32_t ph = div32(phw, p.d_phs), pw = phw - ph * (uint32_t)p.ph_sw;
        f_d = (int)div32(pd + (uint32_t)p.ph_pad_d, p.d_phd) + p.ph_first_d;
        f_h = (int)div32(ph + (uint32_t)p.ph_pad_h, p.d_phh) + p.ph_first_h;
        f_w = (int)div32(pw + (uint32_t)p.ph_pad_w, p.d_phs) + p.ph_first_w;
        y_phase = (int64_t)(pd * p.y_pd + ph * p.y_ph + pw * p.y_pw) * (p.flags & kDconvOutBf16 ? 2 : 4);
    }
    const i32x4_t x_rsrc = make_rsrc(p.x, p.x_bytes);
    const i32x4_t w_rsrc = make_rsrc((const char *)p.w + (int64_t)by * p.w_bstride, p.w_bytes);

    // ---- the patch: pixels a0 + s_min .. of the planes the tile's outputs lie in (before the depth tap's shift) -----------
    const int HW = p.H * p.W, ohw = p.OH * p.OW;
    auto anchor = [&](int m) {
        const int img = (int)div32((uint32_t)m, p.d_hw), rem = m - img * ohw;
        const int oh = (int)div32((uint32_t)rem, p.d_w);
        return img * HW + oh * p.W + (rem - oh * p.OW);
    };
    const int r0 = f_h * p.dil - p.pad_h, c0 = f_w * p.dil_w - p.pad_w;     // the first tap's row and column from an output's
    const int s_min = r0 * p.W + c0;
    const int a0 = anchor(m0);
    const int np = anchor(min(m0 + BM, p.M) - 1) - a0 + 1 + (KR - 1) * (p.dil * p.W + p.dil_w);
    const int nwl = (np * SPP + 63) >> 6;                  // wave-loads (at most NWG * PN: the host sees to it)
    const uint32_t pbuf = (uint32_t)p.patch_bytes;         // of the largest patch of any tile
    const int ncs = (p.c16 + CPR - 1) / CPR, nslab = ncs * p.T, nq = (nslab + KW - 1) / KW;
    const uint32_t next = nq > 1 ? pbuf : 0u;              // from the first buffer to the second
    const uint32_t ring0 = lds0 + kg * (NS * B_STAGE);
    const uint32_t patch0 = lds0 + KW * (NS * B_STAGE) + kg * (pbuf + next);
    const uint32_t zero0 = patch0 + pbuf - kSlabZero;      // (the second buffer's: `next` further on)
    for (int i = t - kg * (64 * NWG); i < kSlabZero / 16; i += 64 * NWG)
        for (uint32_t b = 0; b <= next; b += pbuf) *(uint4 *)((char *)smem_u4 + (zero0 - lds0) + b + i * 16) = make_uint4(0, 0, 0, 0);

    // wave-load i of a patch by this wave: slot j * 64 + lane, j = i * NWG + wq; its byte offset in slab 0 with the chunk inside the
    // pixel in the low bits (an unused slot's chunk is CPR, which no slab has), and its output plane inside its volume
    uint32_t p_off[PN];
    int p_od[PN];
#pragma unroll
    for (int i = 0; i < PN; ++i) {
        const uint32_t slot = (uint32_t)((i * NWG + wq) * 64 + lane), px = slot / SPP, c = slot - px * SPP;
        const int g = a0 + s_min + (int)px;
        const bool in = (int)px < np && (unsigned)g < (unsigned)p.in_px;
        p_off[i] = (uint32_t)g * p.x_pix + c * 16u + (in ? c : (uint32_t)CPR);
        const uint32_t plane = div32(in ? (uint32_t)g : 0u, p.d_ihw);
        p_od[i] = (int)(plane - div32(plane, p.d_od) * (uint32_t)p.D);
    }
    // weights: slot s = (i*NWG + wq)*64 + lane of a stage holds chunk (s % CPR) ^ swz(row) of row s / CPR, as in dconv.h
    uint32_t b_voff[NLB];
    int b_chunk[NLB];
#pragma unroll
    for (int i = 0; i < NLB; ++i) {
        const int s = (i * NWG + wq) * 64 + lane, row = s / CPR, n = n0 + row;
        b_chunk[i] = (s % CPR) ^ ((row / RP) & (CPR - 1));
        b_voff[i] = n < p.Nc ? (uint32_t)n * p.w_row + (uint32_t)f_d * p.wtap_d + (uint32_t)f_h * p.wtap_h + (uint32_t)f_w * p.wtap_w +
                                   (uint32_t)b_chunk[i] * 16u : kOutOfRange;
    }

    // ---- slab q of this group --------------------------------------------------------------------------------------
    struct Slab {
        uint32_t x_off, w_off;                             // what it adds to the offsets
        int dsh, live;                                     // planes from an output's to its inputs'; chunks of a pixel (0: no such slab)
        bool walked;                                       // (a slab without chunks that evens out the groups is: over zeros)
        uint32_t bv[NLB];                                  // the weight rows' offsets, out of range behind the last channel
    };
    auto slab_of = [&](int q) {
        const int idx = kg + q * KW;
        const int td = (int)div32((uint32_t)idx, p.d_c16), cs = idx - td * ncs;   // (d_c16 divides by ncs here)
        Slab s;
        s.dsh = (f_d + td) * p.dil_d - p.pad_d;
        s.walked = q < nq;
        s.live = idx < nslab ? min(CPR, p.c16 - cs * CPR) : 0;
        s.x_off = (uint32_t)(s.dsh * HW) * p.x_pix + (uint32_t)cs * (BK * 2u);
        s.w_off = idx < nslab ? (uint32_t)td * p.wtap_d + (uint32_t)cs * (BK * 2u) : 0u;
#pragma unroll
        for (int i = 0; i < NLB; ++i) s.bv[i] = b_chunk[i] < s.live ? b_voff[i] : kOutOfRange;
        return s;
    };
    auto load_patch = [&](const Slab &s, int i, uint32_t buffer) {
        const int j = i * NWG + wq, c = (int)(p_off[i] & 15u);
        const bool ok = c < s.live && (unsigned)(p_od[i] + s.dsh) < (unsigned)p.D;
        // (past the last wave-load, and past the last slab: zeros onto the zero area, so that every step issues the same number)
        dma_load16_s(x_rsrc, ok ? (p_off[i] & ~15u) + s.x_off : kOutOfRange, 0u, j < nwl && s.walked ? buffer + j * 1024 : buffer + pbuf - kSlabZero);
    };
    // (the taps' weights one after the other: their offset runs along, so that not all of them sit in scalar registers)
    const uint32_t ring_w = ring0 + wq * 1024, row_step = p.wtap_h - (KR - 1) * p.wtap_w;
    uint32_t w_soff = 0;
    auto load_w = [&](const Slab &s, auto TAP) {
        constexpr int tap = decltype(TAP)::value, st = tap % NS;
        w_soff = tap == 0 ? s.w_off : w_soff + (tap % KR ? p.wtap_w : row_step);
        static_for<NLB>([&](auto I) {
            constexpr int i = decltype(I)::value;
            dma_load16_at<st * B_STAGE + i * (NWG * 1024)>(w_rsrc, s.bv[i], w_soff, ring_w);
        });
    };

    Slab cur = slab_of(0);
#pragma unroll
    for (int i = 0; i < PN; ++i) load_patch(cur, i, patch0);
    // (the steps before the first one: their weights, and as many wave-loads as they would have issued for a patch)
    static_for<NS - 1>([&](auto U) {
        constexpr int u = decltype(U)::value;
        load_w(cur, U);
#pragma unroll
        for (int i = 0; i < slab_loads(KR, PN, u - (NS - 1)); ++i) dma_load16_s(x_rsrc, kOutOfRange, 0u, zero0);
    });

    // ---- operand addresses of this lane ----------------------------------------------------------------------------------
    const uint32_t khalf = (lane >> 5) * 16;
    uint32_t t_row[RS][TM], b_rd[TN][NKC];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * WTM + i * 32 + (lane & 31);
        int oh = -(1 << 20), ow = -(1 << 20), px = 0;
        if (m < p.M) {
            const int img = (int)div32((uint32_t)m, p.d_hw), rem = m - img * ohw;
            oh = (int)div32((uint32_t)rem, p.d_w);
            ow = rem - oh * p.OW;
            px = img * HW + oh * p.W + ow - a0;
        }
#pragma unroll
        for (int tap = 0; tap < RS; ++tap) {
            const int dr = (tap / KR) * p.dil, ds = (tap % KR) * p.dil_w;
            const bool ok = (unsigned)(oh + r0 + dr) < (unsigned)p.H && (unsigned)(ow + c0 + ds) < (unsigned)p.W;
            const uint32_t at = patch0 + (uint32_t)(px + dr * p.W + ds) * (SPP * 16);
            t_row[tap][i] = (ok ? at : zero0 + (at & 255u)) + khalf;
        }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int r = wn * WTN + j * 32 + (lane & 31);
        const uint32_t swz = ((r / RP) & (CPR - 1)) * 16;
#pragma unroll
        for (int kc = 0; kc < NKC; ++kc) b_rd[j][kc] = ring0 + r * (BK * 2) + ((kc * 32 + khalf) ^ swz);
    }

    floatx16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // ---- main loop -------------------------------------------------------------------------------------------------------
    // Step `tap` of a slab: at its barrier every wave has its share of the next step's weights landed (and, in a slab's first step,
    // of the patch), so the operand reads, D chunks ahead, may run into the next step; the stage and, in the first step, the patch
    // buffer that were read last are refilled behind it: weights of NS - 1 steps on, then a few wave-loads of the next patch.
    constexpr int D0 = (TM + TN) * 3 <= 15 ? 3 : (TM + TN) * 2 <= 15 ? 2 : 1;
    constexpr int D = D0 < NKC ? D0 : NKC, NBUF = 4;
    static_assert(D < NBUF, "look-ahead against the register buffers");
    u32x4_t af[NBUF][TM], bf[NBUF][TN];
    auto reads = [&](auto GI) {
        constexpr int g = decltype(GI)::value, tap = g / NKC, kc = g % NKC, buf = g % NBUF;
        static_for<TM>([&](auto ic) { lds_read16_async_at<kc * 32>(af[buf][decltype(ic)::value], t_row[tap][decltype(ic)::value]); });
        static_for<TN>([&](auto jc) { lds_read16_async_at<(tap % NS) * B_STAGE>(bf[buf][decltype(jc)::value], b_rd[decltype(jc)::value][kc]); });
    };
    lds_barrier();                                         // the zero areas
    uint32_t other = next;                                 // from this slab's patch buffer to the other
    for (int q = 0; q < nq; ++q) {
        const Slab nxt = slab_of(q + 1);
        const uint32_t buffer = patch0 + (q & 1 ? 0u : next);
        static_for<RS>([&](auto TC) {
            constexpr int tap = decltype(TC)::value;
            wait_vmcnt<slab_loads_behind<KR, BK, NLB, PN>(tap)>();
            if constexpr (NWG > 1) asm volatile("s_barrier" ::: "memory");
            constexpr int ahead_tap = tap + NS - 1;
            load_w(ahead_tap < RS ? cur : nxt, std::integral_constant<int, ahead_tap % RS>{});
            if constexpr (slab_loads(KR, PN, tap) > 0) {
#pragma unroll
                for (int i = 0; i < slab_loads(KR, PN, tap); ++i) load_patch(nxt, tap * PN / slab_load_steps(KR) + i, buffer);
            }
            if constexpr (tap == 0) static_for<D>([&](auto GI) { reads(GI); });
            static_for<NKC>([&](auto KC) {
                constexpr int g = tap * NKC + decltype(KC)::value, buf = g % NBUF;
                if constexpr (g + D < NG) reads(std::integral_constant<int, g + D>{});
                constexpr int flying = g + D < NG ? D : NG - 1 - g;
                lds_wait<flying * (TM + TN)>(af[buf], bf[buf]);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, bf[buf][j]),
                                                                            __builtin_bit_cast(bf16x8_t, af[buf][i]), acc[i][j], 0, 0, 0);
            });
        });
        cur = nxt;
#pragma unroll
        for (int tap = 0; tap < RS; ++tap)
#pragma unroll
            for (int i = 0; i < TM; ++i) t_row[tap][i] += other;
        other = 0u - other;
    }
    wait_vmcnt<0>();                                       // the loads past the last slab

    dconv_epilogue<BM, BN, WGM, WGN, KW>(p, acc, smem_u4, t, lane, wave, kg, wq, wm, wn, m0, n0, mt, nt, 0, (char *)p.y + y_phase);
}

template <int BM, int BN, int WGM, int WGN, int KW, int BK, int KR, int PN>
__global__ __launch_bounds__(64 * WGM * WGN * KW, ALT_DCONV_MIN_WAVES((BM / WGM) * (BN / WGN) / 64, WGM * WGN * KW))
void dslab_kernel(const DconvParams p)
{
    // (the number of tiles as the grid has it costs a load and saves up to 17 spilled scalar registers: 3x3x3 over 128 channels 16.9 us, 17.1 with
    // the product; 62 x 80 x 17 x 17, 3x3, 11.4 and 11.9.  Layers of 256 images that run 256x128 tiles take 0.5 % longer so.)
    dslab_body<BM, BN, WGM, WGN, KW, BK, KR, PN>(p, BN < 128 ? (int)gridDim.x : p.tiles_m * p.tiles_n, (int)blockIdx.x, (int)blockIdx.y);
}

template <int BM, int BN, int WGM, int WGN, int KW, int BK, int KR, int PN>
hipError_t dslab_launch_pn(const DconvParams &p, size_t lds, hipStream_t st)
{
    auto kern = dslab_kernel<BM, BN, WGM, WGN, KW, BK, KR, PN>;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_m * p.tiles_n), (unsigned)std::max(1, p.phases)), dim3(64 * WGM * WGN * KW), lds, st, p);
    return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int KW, int BK, int KR>
hipError_t dslab_launch_kr(const DconvParams &p, size_t lds, hipStream_t st)
{
    const int loads = (int)(((uint32_t)p.patch_bytes - kSlabZero) / 1024 + WGM * WGN - 1) / (WGM * WGN);
    if (loads <= kSlabLoads[0]) return dslab_launch_pn<BM, BN, WGM, WGN, KW, BK, KR, kSlabLoads[0]>(p, lds, st);
    if (loads <= kSlabLoads[1]) return dslab_launch_pn<BM, BN, WGM, WGN, KW, BK, KR, kSlabLoads[1]>(p, lds, st);
    if (loads <= kSlabLoads[2]) return dslab_launch_pn<BM, BN, WGM, WGN, KW, BK, KR, kSlabLoads[2]>(p, lds, st);
    return hipErrorInvalidValue;
}

template <int BM, int BN, int WGM, int WGN, int KW, int BK>
hipError_t dslab_launch(const DconvParams &p, size_t lds, hipStream_t st)
{
    if (p.bk != BK || p.splitk != 1) return hipErrorInvalidValue;
    if (p.R == 3 && p.S == 3) return dslab_launch_kr<BM, BN, WGM, WGN, KW, BK, 3>(p, lds, st);
    if (p.R == 2 && p.S == 2) return dslab_launch_kr<BM, BN, WGM, WGN, KW, BK, 2>(p, lds, st);
    return hipErrorInvalidValue;
}

}  // namespace alt
