// Host side of the patch-resident direct convolution (dconv.h) and of the
// streaming kernel (dstream.h): which problems each covers, their launch
// parameters, and the arrival counters of the fused split-K reduction.
#include <mutex>

#include "dplanar.h"
#include "dshort.h"
#include "dslab.h"
#include "dstem.h"
#include "dstream.h"
#include "group.h"
#include "ops.h"

namespace alt {

namespace {

// Arrival counters of the fused split-K reduction: zero when the module is
// loaded, and every launch leaves them zero again.  There are kDconvSlots sets;
// a set is bound to the first stream that issues a split-K launch and stays
// with it (launches on one stream run one after the other, so they can share
// a set; launches on different streams never do).
__device__ __align__(256) uint32_t g_dconv_counters[kDconvSlots * kDconvMaxTiles];
constexpr int kMaxDevices = 16;

struct SlotTable {
    hipStream_t stream[kDconvSlots];
    bool used[kDconvSlots], pinned[kDconvSlots];   // pinned: a captured graph carries this set's address
};

struct DeviceState {
    uint32_t *counters = nullptr;
    SlotTable slots{};
};
DeviceState g_dev[kMaxDevices];
std::mutex g_mutex;

bool dense(const Dim2 &d, int64_t extent, int64_t stride)
{
    return extent == 1 || (d.f >= extent && d.si == stride);
}

// Whether four per-dimension maps describe a dense activation tensor with the channels of a pixel contiguous
// (NHWC: *blk = 0) or in blocks of b = 2^*blk >= 8 channels (N C/b H W b, b dividing C).
bool nhwc_or_blocked(const Dim2 &c, const Dim2 &w, const Dim2 &h, const Dim2 &n, int64_t C, int64_t H, int64_t W, int64_t N,
                     int *blk)
{
    if (dense(c, C, 1) && dense(w, W, C) && dense(h, H, W * C) && dense(n, N, H * W * C)) { *blk = 0; return true; }
    const int64_t b = c.f;
    if (c.si != 1 || b < 8 || b >= C || (b & (b - 1)) || C % b || c.so != H * W * b) return false;
    if (!(dense(w, W, b) && dense(h, H, W * b) && dense(n, N, C * H * W))) return false;
    int l = 0;
    while (((int64_t)1 << l) < b) ++l;
    *blk = l;
    return true;
}

DeviceState *device_state()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    return &g_dev[dev];
}

}  // namespace

// Device address of the counters on the current device (looked up once per device).
hipError_t dconv_counters(uint32_t **out)
{
    DeviceState *ds = device_state();
    if (!ds) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_mutex);
    if (!ds->counters) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_dconv_counters));
        if (e != hipSuccess) return e;
        ds->counters = (uint32_t *)ptr;
    }
    *out = ds->counters;
    return hipSuccess;
}

// Counter sets bound to streams on the current device, and how many counters are not zero once
// the device is idle (-1 if they cannot be read): waits for the device.
void dconv_splitk_state(int *slots_bound, int *counters_nonzero)
{
    DeviceState *ds = device_state();
    *slots_bound = 0;
    *counters_nonzero = -1;
    if (!ds) return;
    {
        std::lock_guard<std::mutex> lock(g_mutex);
        for (int i = 0; i < kDconvSlots; ++i) *slots_bound += ds->slots.used[i] ? 1 : 0;
    }
    uint32_t *base = nullptr;
    if (dconv_counters(&base) != hipSuccess || hipDeviceSynchronize() != hipSuccess) return;
    std::vector<uint32_t> host((size_t)kDconvSlots * kDconvMaxTiles);
    if (hipMemcpy(host.data(), base, host.size() * 4, hipMemcpyDeviceToHost) != hipSuccess) return;
    int nz = 0;
    for (uint32_t v : host) nz += v != 0;
    *counters_nonzero = nz;
}

// The counter set of `st` on the current device: the one bound to it, else a free one.  When
// every set is bound the host waits until the device is idle and releases all sets except
// those a captured graph carries the address of.  hipErrorNotReady if that leaves none, or
// if the wait would be needed while `st` is being captured.
static hipError_t counter_slot(DeviceState *ds, hipStream_t st, int *slot)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (st) (void)hipStreamIsCapturing(st, &cap);
    const bool capturing = cap != hipStreamCaptureStatusNone;
    std::lock_guard<std::mutex> lock(g_mutex);
    SlotTable &t = ds->slots;
    int free_slot = -1;
    for (int i = 0; i < kDconvSlots; ++i) {
        if (t.used[i] && t.stream[i] == st) { t.pinned[i] |= capturing; *slot = i; return hipSuccess; }
        if (!t.used[i] && free_slot < 0) free_slot = i;
    }
    if (free_slot < 0) {
        // Every set is bound.  Sets whose address a captured graph carries stay; the others are
        // released once nothing is in flight on the device.
        if (capturing) return hipErrorNotReady;
        hipError_t e = hipDeviceSynchronize();
        if (e != hipSuccess) return e;
        for (int i = 0; i < kDconvSlots; ++i)
            if (!t.pinned[i]) { t.used[i] = false; if (free_slot < 0) free_slot = i; }
        if (free_slot < 0) return hipErrorNotReady;
    }
    t.used[free_slot] = true;
    t.pinned[free_slot] = capturing;
    t.stream[free_slot] = st;
    *slot = free_slot;
    return hipSuccess;
}

// The order in which a launch's tiles are numbered (dconv_tile): rows of tiles per panel.  An XCD works on a window of at most 64
// consecutive tiles at a time (32 compute units of one or two), which covers rows and columns of tiles; the panel is the one whose window
// reads least.  a, b: bytes that a row and a column of tiles read.  All rows are one panel where that reads no more than an eighth
// above the least, or no more than half of an XCD's L2 (4 MB), where it comes in once in any order; and fp32 tiles (dconv_tile).
static void order_tiles(DconvParams *d, double a, double b, bool panels = true)
{
    const int64_t tiles = (int64_t)d->tiles_m * d->tiles_n, share = (tiles * d->splitk + 7) / 8;
    const int window = (int)std::min<int64_t>(std::min<int64_t>(share, tiles), 64);
    auto reads = [&](int pm) {
        const int64_t panel = (int64_t)pm * d->tiles_n;
        const int rows = panel >= window ? std::min(pm, window) : (int)std::min<int64_t>((int64_t)pm * ((window + panel - 1) / panel), d->tiles_m);
        const int cols = panel >= window ? (window + pm - 1) / pm : d->tiles_n;
        return rows * a + cols * b;
    };
    int best = d->tiles_m;
    double least = reads(best) / 1.125;
    if (panels && d->splitk == 1 && reads(best) > 2e6)
        for (int pm = 1; pm <= window && 2 * pm <= d->tiles_m; ++pm)
            if (d->tiles_m % pm == 0 && reads(pm) < least) { least = reads(pm); best = pm; }
    d->flags |= (int32_t)((uint32_t)best << kPanelShift);
    d->d_pm = make_div32((uint32_t)best);
    d->d_tn = make_div32((uint32_t)d->tiles_n);
}

// The same for a streaming kernel (dstream.h): 1x1 filters, stride 1, no padding (a GEMM
// is lowered to that), any number of channels that splits into 64-channel steps.
static bool dstream_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes,
                          std::string *why)
{
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p = pb.p;
    if (pb.dtype != ALT_BF16) return no("streaming kernel is bf16 only");
    if (p.R != 1 || p.S != 1 || p.stride_h != 1 || p.stride_w != 1 || p.pad_h != 0 || p.pad_w != 0)
        return no("streaming kernel needs a 1x1 filter, stride 1, no padding");
    if (p.OH != p.H || p.OW != p.W) return no("streaming kernel needs output size = input size");
    const int64_t C = p.C, H = p.H, W = p.W, K = p.Nc, N = p.M / (H * W);
    // (B first: half of these kernels read the other layout of it)
    if (k.bt) {
        if (!(dense(p.wo, K, 1) && dense(p.wi, C, K))) return no("B is not dense with N contiguous");
        if (K % 8) return no("row-major B is loaded eight columns at a time");
    } else if (!(dense(p.wi, C, 1) && dense(p.wo, K, C))) {
        return no("B is not dense with K contiguous");
    }
    int x_blk = 0, y_blk = 0;
    if (!nhwc_or_blocked(p.xc, p.xw, p.xh, p.xn, C, H, W, N, &x_blk)) return no("A is not dense with K contiguous (whole or in blocks)");
    if (x_blk && k.BK % (1 << x_blk)) return no("channel blocks larger than a K step");
    if (!nhwc_or_blocked(p.yk, p.yw, p.yh, p.yn, K, H, W, N, &y_blk)) return no("output is not dense with N contiguous (whole or in blocks)");
    if ((x_blk || y_blk) && p.batch > 1) return no("blocked tensors are not built for batched problems");
    const int64_t osz = p.out_bf16 ? 2 : 4;
    if ((uintptr_t)p.x % 16 || (uintptr_t)p.w % 16 || (uintptr_t)p.y % 16) return no("operands are not 16-byte aligned");
    if (p.batch > 1 && ((p.x_bstride * 2) % 16 || (p.w_bstride * 2) % 16 || (p.y_bstride * osz) % 16))
        return no("batch entries are not 16-byte aligned");
    if (p.batch > 65535) return no("too many batch entries for one launch");
    if (p.addend && p.batch > 1) return no("the fused sum is not built for batched problems");
    if (splitk < 1 || (splitk > 1 && p.batch > 1)) return no("split-K is not built for batched problems");
    if (C % ((int64_t)k.BK * splitk * k.kw)) return no("K does not split into whole steps per slice and K group");
    if (pb.x_elems * 2 >= 0x7fffffff || pb.w_elems * 2 >= 0x7fffffff || p.y_bytes == 0)
        return no("operand of 2 GiB or more");
    if ((int64_t)p.M * K * 4 >= 0x7fffffff) return no("output too large for 32-bit offsets");
    if (K % 4 || (p.epilogue & ALT_EPI_BIAS && (uintptr_t)p.bias % 16)) return no("streaming kernel stores four output columns at a time");
    const size_t lds = dstream_lds_bytes(k.BM, k.BN, k.BK * 2, k.prefetch + 1, k.wgm, k.wgn, k.kw);
    if (lds > 160 * 1024) return no("stages do not fit LDS");
    if (dstream_banded(k.BM, k.BN, k.wgn, k.kw) && splitk > 1) return no("tiles this large take no split-K");
    const int tiles_m = (p.M + k.BM - 1) / k.BM, tiles_n = (p.Nc + k.BN - 1) / k.BN;
    if (splitk > 1 && (int64_t)tiles_m * tiles_n > kDconvMaxTiles) return no("too many output tiles for the split-K counters");
    if ((int64_t)tiles_m * tiles_n * splitk > 0x7fffffff) return no("grid too large");
    if (lds_bytes) *lds_bytes = lds;
    if (!out) return true;
    DconvParams d;
    std::memset(&d, 0, sizeof d);
    d.x = p.x; d.w = p.w; d.bias = p.bias; d.y = p.y; d.addend = p.addend;
    d.x_bytes = p.x_bytes; d.w_bytes = p.w_bytes; d.y_bytes = p.y_bytes;
    d.partial_bytes = (uint32_t)((int64_t)p.M * K * 4);
    d.M = p.M; d.Nc = p.Nc; d.C = p.C; d.Cs = (int32_t)(C / splitk);
    d.H = p.H; d.W = p.W; d.R = 1; d.S = 1;
    d.tiles_m = tiles_m; d.tiles_n = tiles_n; d.splitk = splitk;
    d.flags = (p.epilogue & (ALT_EPI_BIAS | ALT_EPI_RELU)) | (p.out_bf16 ? kDconvOutBf16 : 0);
    d.d_hw = make_div32((uint32_t)(p.H * p.W));
    d.d_w = make_div32((uint32_t)p.W);
    order_tiles(&d, 2.0 * C / splitk * k.BM, 2.0 * C / splitk * k.BN);
    d.ncc = (int32_t)(C / splitk / k.kw / k.BK);
    d.bk = k.BK;
    d.batch = p.batch;
    d.OH = p.H; d.OW = p.W; d.x_blk = x_blk; d.y_blk = y_blk;
    d.d_ihw = make_div32((uint32_t)(p.H * p.W));
    d.x_bstride = p.x_bstride * 2; d.w_bstride = p.w_bstride * 2; d.y_bstride = p.y_bstride * osz;
    *out = d;
    return true;
}

// The same for a streaming kernel over filter taps (dstream.h, TAPS): any filter of up to ten taps per direction, any
// stride, dilation and padding, dense NHWC activations and output with OHWI weights, a pixel's channels a whole number of
// 16-byte chunks; and matrix products whose K is one, with B as NK or (bt) KN.
static bool dtaps_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes, std::string *why)
{
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p = pb.p;
    const int es = (int)dtype_size(pb.dtype), epc = 16 / es;
    const int64_t C = p.C, H = p.H, W = p.W, OH = p.OH, OW = p.OW, K = p.Nc, R = p.R, S = p.S;
    // (a volume's slices are images; D = OD = T = 1 without one)
    const Volume &v = pb.v;
    const int64_t D = v.T ? v.D : 1, OD = v.T ? v.OD : 1, T = v.T ? v.T : 1, N = p.M / (OH * OW * OD), NX = N * D, NY = N * OD;
    const int sd = v.T ? v.sd : 1, sh = v.T ? v.sh : 1, sw = v.T ? v.sw : 1, phases = sd * sh * sw;
    const int64_t nT = phases > 1 ? v.taps[0] : T, nR = phases > 1 ? v.taps[1] : R, nS = phases > 1 ? v.taps[2] : S;
    if (T > kTapBits || R > kTapBits || S > kTapBits) return no("filters of more than ten taps in one direction");
    if (C % epc) return no("a pixel's channels are not a whole number of 16-byte chunks");
    if (k.bt) {
        if (v.T || R * S != 1 || !(dense(p.wo, K, 1) && dense(p.wi, C, K))) return no("B is not dense with N contiguous");
        if (K % 8) return no("row-major B is loaded eight columns at a time");
    } else if (!(dense(p.wi, T * C, 1) && dense(p.ws, S, T * C) && dense(p.wr, R, S * T * C) && dense(p.wo, phases * K, R * S * T * C))) {
        return no("weights are not dense OHWI");
    }
    int x_blk = 0, y_blk = 0;
    if (!nhwc_or_blocked(p.xc, p.xw, p.xh, p.xn, C, H, W, NX, &x_blk) || x_blk) return no("activations are not dense NHWC");
    if (!nhwc_or_blocked(p.yk, p.yw, p.yh, p.yn, K, OH * sh, OW * sw, NY * sd, &y_blk) || (y_blk && p.batch > 1)) return no("output is not dense NHWC or N K/b H W b");
    const int64_t osz = p.out_bf16 ? 2 : 4;
    if ((uintptr_t)p.x % 16 || (uintptr_t)p.w % 16 || (uintptr_t)p.y % 16) return no("operands are not 16-byte aligned");
    if (p.batch > 1 && ((p.x_bstride * es) % 16 || (p.w_bstride * es) % 16 || (p.y_bstride * osz) % 16))
        return no("batch entries are not 16-byte aligned");
    if (p.batch > 65535) return no("too many batch entries for one launch");
    if (pb.groups > 1) return no("a group's channels are not dense");
    if (p.addend && p.batch > 1) return no("the fused sum is not built for batched problems");
    if (splitk < 1 || (splitk > 1 && p.batch > 1)) return no("split-K is not built for batched problems");
    const int64_t pix = C * es, shift = ((v.T ? v.pad_d * H * W : 0) + (int64_t)p.pad_h * W + p.pad_w) * pix;
    if (pb.x_elems * es + shift >= 0x7fffffff || pb.w_elems * es >= 0x7fffffff || p.y_bytes == 0) return no("operand of 2 GiB or more");
    if ((int64_t)p.M * pix + shift >= 0x7fffffff && R * S == 1 && p.stride_h == 1) return no("operand of 2 GiB or more");
    if ((int64_t)p.M * phases * K * 4 >= 0x7fffffff) return no("output too large for 32-bit offsets");
    if (K % 4 || ((p.epilogue & ALT_EPI_BIAS) && (uintptr_t)p.bias % 16)) return no("streaming kernel stores four output columns at a time");
    const int64_t reach = ((v.T ? (T - 1) * (int64_t)v.dil_d * H * W : 0) + (R - 1) * (int64_t)p.dil_h * W + (S - 1) * (int64_t)p.dil_w) * pix;
    if (reach + shift >= 0x3fffffff) return no("filter reaches too far");
    const int cpr = k.BK * es / 16;
    const int64_t kq = nT * nR * nS * C / epc, steps = (kq + cpr - 1) / cpr, slices = (int64_t)splitk * k.kw;
    if (k.taps == kTapsUniform && (C % k.BK || steps % slices)) return no("K steps do not divide the channels and the slices evenly");
    const int64_t nk = (steps + slices - 1) / slices;
    if ((slices - 1) * nk >= steps) return no("split factor leaves an empty slice");
    const size_t lds = dstream_lds_bytes(k.BM, k.BN, k.BK * es, k.prefetch + 1, k.wgm, k.wgn, k.kw);
    if (lds > 160 * 1024) return no("stages do not fit LDS");
    if (dstream_banded(k.BM, k.BN, k.wgn, k.kw) && splitk > 1) return no("tiles this large take no split-K");
    const int tiles_m = (p.M + k.BM - 1) / k.BM, tiles_n = (p.Nc + k.BN - 1) / k.BN;
    if (splitk > 1 && (int64_t)tiles_m * tiles_n > kDconvMaxTiles) return no("too many output tiles for the split-K counters");
    if ((int64_t)tiles_m * tiles_n * splitk > 0x7fffffff) return no("grid too large");
    if (lds_bytes) *lds_bytes = lds;
    if (!out) return true;
    DconvParams d;
    std::memset(&d, 0, sizeof d);
    d.x = p.x; d.w = p.w; d.bias = p.bias; d.y = p.y; d.addend = p.addend;
    d.x_bytes = p.x_bytes; d.w_bytes = p.w_bytes; d.y_bytes = p.y_bytes;
    d.partial_bytes = (uint32_t)((int64_t)p.M * K * 4);
    d.M = p.M; d.Nc = p.Nc; d.C = p.C; d.Cs = p.C;
    d.H = p.H; d.W = p.W; d.R = (int32_t)nR; d.S = (int32_t)nS; d.pad_h = p.pad_h; d.pad_w = p.pad_w;
    d.OH = p.OH; d.OW = p.OW; d.stride = p.stride_h; d.dil = p.dil_h; d.stride_w = p.stride_w; d.dil_w = p.dil_w;
    d.T = d.D = d.OD = d.stride_d = d.dil_d = 1;
    if (v.T) { d.T = (int32_t)nT; d.D = v.D; d.OD = v.OD; d.stride_d = v.stride_d; d.pad_d = v.pad_d; d.dil_d = v.dil_d; }
    d.tiles_m = tiles_m; d.tiles_n = tiles_n; d.splitk = splitk;
    d.flags = (p.epilogue & (ALT_EPI_BIAS | ALT_EPI_RELU)) | (p.out_bf16 ? kDconvOutBf16 : 0);
    d.d_hw = make_div32((uint32_t)(OH * OW));
    d.d_w = make_div32((uint32_t)OW);
    order_tiles(&d, (double)es * C / splitk * T * k.BM * p.stride_h * p.stride_w, (double)es * C / splitk * T * R * S * k.BN, es == 2);
    d.d_od = make_div32((uint32_t)OD);
    d.ncc = (int32_t)nk;
    d.bk = k.BK;
    d.taps = (int32_t)(nT * nR * nS);
    d.strided = v.T || !(R * S == 1 && OH == H && OW == W && p.stride_h == 1 && p.stride_w == 1 && p.pad_h == 0 && p.pad_w == 0);
    d.c16 = (int32_t)(C / epc); d.kq = (int32_t)kq;
    d.d_c16 = make_div32((uint32_t)d.c16);
    d.d_rs = make_div32((uint32_t)(nR * nS));
    d.d_s = make_div32((uint32_t)nS);
    d.x_pix = (uint32_t)pix;
    d.w_row = (uint32_t)(R * S * T * pix);
    d.tap_h = (uint32_t)(p.dil_h * W * pix);
    d.tap_w = (uint32_t)(p.dil_w * pix);
    if (v.T) d.tap_d = (uint32_t)(v.dil_d * H * W * pix);
    d.wtap_d = (uint32_t)pix;
    d.wtap_h = (uint32_t)(S * T * pix);
    d.wtap_w = (uint32_t)(T * pix);
    d.w_dense = T == 1 && phases == 1;
    d.x_shift = (uint32_t)shift;
    if (phases > 1) {
        d.phases = phases;
        d.ph_sh = sh; d.ph_sw = sw;
        d.ph_pad_d = v.pad[0]; d.ph_pad_h = v.pad[1]; d.ph_pad_w = v.pad[2];
        d.ph_first_d = v.pad_d + 1 - v.taps[0]; d.ph_first_h = p.pad_h + 1 - v.taps[1]; d.ph_first_w = p.pad_w + 1 - v.taps[2];
        d.d_phw = make_div32((uint32_t)(sh * sw)); d.d_phd = make_div32((uint32_t)sd);
        d.d_phh = make_div32((uint32_t)sh); d.d_phs = make_div32((uint32_t)sw);
        d.y_pw = (uint32_t)K; d.y_ph = (uint32_t)(OW * sw * K); d.y_pd = (uint32_t)(OH * sh * OW * sw * K);
        d.y_pix = sw * d.y_pw; d.y_row = sh * d.y_ph; d.y_img = sd * d.y_pd;
        // (the last phase's outputs end where the tensor does)
        d.y_bytes = p.y_bytes - (uint32_t)(((sd - 1) * (int64_t)d.y_pd + (sh - 1) * (int64_t)d.y_ph + (sw - 1) * (int64_t)d.y_pw) * osz);
        y_blk = kOutPhases;
    }
    d.batch = p.batch;
    d.y_blk = y_blk;
    d.d_ihw = make_div32((uint32_t)(H * W));
    d.x_bstride = p.x_bstride * es; d.w_bstride = p.w_bstride * es; d.y_bstride = p.y_bstride * osz;
    *out = d;
    return true;
}

// The same for a patch-resident kernel over slabs of channels (dslab.h): what the kernels over filter taps take, with 3x3 filters
// or output phases of 2x2 taps at stride 1 and an output no larger than the input.
static bool dslab_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes, std::string *why)
{
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p = pb.p;
    const Volume &v = pb.v;
    if (pb.dtype != ALT_BF16) return no("slab kernel is bf16 only");
    if (splitk != 1) return no("slab kernel takes no split-K");
    const int phases = v.T ? v.sd * v.sh * v.sw : 1;
    if (p.batch != phases) return no("slab kernel takes no batch");
    const int kr = phases > 1 ? v.taps[1] : p.R, ks = phases > 1 ? v.taps[2] : p.S;
    if (kr != ks || (kr != 2 && kr != 3)) return no("slab kernel is built for 2x2 and 3x3 taps");
    if (p.stride_h != 1 || p.stride_w != 1 || (v.T && v.stride_d != 1)) return no("slab kernel needs stride 1");
    if (p.dil_h != p.dil_w) return no("slab kernel needs one dilation for rows and columns");
    // (then the input pixel under an output pixel never moves backwards, and a depth tap is a whole number of planes)
    if (p.OH > p.H || p.OW > p.W || (v.T && v.OD != v.D)) return no("output larger than the input, or of another depth");
    if (phases > 1 && (p.OH != p.H || p.OW != p.W)) return no("output phases of another size than the input");
    // (the parameters are built for a launch alone: choosing a kernel asks about seven of these)
    IgemmLaunch t = k;
    t.kw = 1; t.prefetch = 2;
    if (!dtaps_setup(pb, t, 1, nullptr, nullptr, why)) return false;
    const int64_t planes = (int64_t)p.M / ((int64_t)p.OH * p.OW), in_px = planes * p.H * p.W;
    if (in_px > 0x7fffffff) return no("input too large for 32-bit pixel indices");
    const size_t np = dconv_patch_pixels(k.BM, p.M, p.H, p.W, p.OH, p.OW, kr, ks, 0, 0, 1, p.dil_h);
    const int nwg = k.wgm * k.wgn;
    if (np > 8192 || (slab_patch_bytes((int)np, k.BK) - kSlabZero) / 1024 > (uint32_t)(nwg * kSlabLoads[2]))
        return no("patch takes more loads than a slab's steps issue");
    const int64_t ncs = ((int64_t)p.C + k.BK - 1) / k.BK, slabs = ncs * (phases > 1 ? v.taps[0] : v.T ? v.T : 1);
    const size_t lds = dslab_lds_bytes(k.BM, k.BN, k.BK, kr, k.wgn, k.kw, (int)np, slabs > k.kw ? 2 : 1);
    if (lds > 160 * 1024) return no("patches and weight stages do not fit LDS");
    if (lds_bytes) *lds_bytes = lds;
    if (!out) return true;
    DconvParams d;
    if (!dtaps_setup(pb, t, 1, &d, nullptr, why)) return false;
    d.in_px = (int32_t)in_px;
    d.patch_bytes = (int32_t)slab_patch_bytes((int)np, k.BK);
    d.d_c16 = make_div32((uint32_t)ncs);
    *out = d;
    return true;
}

// The same for a channel-planar kernel (dplanar.h): NCHW activations, OIHW weights, NCHW output, all dense.
static bool dplanar_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes,
                          std::string *why)
{
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p = pb.p;
    if (pb.dtype != ALT_BF16) return no("planar kernel is bf16 only");
    if (p.batch != 1) return no("planar kernel takes no batch");
    if (splitk != 1) return no("planar kernel takes no split-K");
    if (p.addend) return no("planar kernel has no fused sum");
    if (!((p.R == 3 && p.S == 3) || (p.R == 1 && p.S == 1))) return no("planar kernel is built for 1x1 and 3x3 filters");
    if (p.stride_h != p.stride_w || (p.stride_h != 1 && p.stride_h != 2) || p.dil_h != p.dil_w || p.dil_h < 1)
        return no("planar kernel needs stride 1 or 2 and one dilation for both directions");
    if (p.pad_h < 0 || p.pad_w < 0 || 2 * p.pad_h > p.dil_h * (p.R - 1) || 2 * p.pad_w > p.dil_w * (p.S - 1))
        return no("planar kernel needs padding between none and same-size");
    const int st_ = p.stride_h;
    if ((int64_t)(p.OH - 1) * st_ >= p.H || (int64_t)(p.OW - 1) * st_ >= p.W) return no("output larger than the strided input");
    const int64_t C = p.C, H = p.H, W = p.W, OH = p.OH, OW = p.OW, K = p.Nc, R = p.R, S = p.S, N = p.M / (OH * OW);
    if (!(dense(p.xw, W, 1) && dense(p.xh, H, W) && dense(p.xc, C, H * W) && dense(p.xn, N, C * H * W)))
        return no("activations are not dense NCHW");
    if (!(dense(p.ws, S, 1) && dense(p.wr, R, S) && dense(p.wi, C, R * S) && dense(p.wo, K, C * R * S)))
        return no("weights are not dense OIHW");
    const bool y_nchw = dense(p.yw, OW, 1) && dense(p.yh, OH, OW) && dense(p.yk, K, OH * OW) && dense(p.yn, N, K * OH * OW);
    const bool y_nhwc = dense(p.yk, K, 1) && dense(p.yw, OW, K) && dense(p.yh, OH, OW * K) && dense(p.yn, N, OH * OW * K);
    if (!y_nchw && !y_nhwc) return no("output is neither dense NCHW nor dense NHWC");
    if (!y_nchw && (K % 8 || (uintptr_t)p.y % 16)) return no("NHWC output is stored eight channels at a time");
    if (C % 8) return no("channels must be a multiple of eight");
    if (!k.ragged && C % 64) return no("channels are no multiple of 64");
    if (H * W < 8) return no("images of fewer than eight pixels");
    if ((uintptr_t)p.w % 16 || (uintptr_t)p.x % 2) return no("weights are not 16-byte aligned");
    if ((p.epilogue & ALT_EPI_BIAS) && (uintptr_t)p.bias % 4) return no("bias is not aligned");
    if (pb.x_elems * 2 >= 0x7fffffff || pb.w_elems * 2 >= 0x7fffffff || p.y_bytes == 0 || (int64_t)p.M * K * 4 >= 0x7fffffff)
        return no("operand of 2 GiB or more");
    if (N * H * W > 0x7fffffff) return no("input too large for 32-bit pixel indices");
    const size_t np = dconv_patch_pixels(k.BM, p.M, p.H, p.W, p.OH, p.OW, p.R, p.S, p.pad_h, p.pad_w, st_, p.dil_h);
    size_t lds = 0;
    const int64_t slab = planar_slab(k.BM, k.BN, k.kw, (int)(R * S), C, np, k.ragged, &lds);
    if (k.ragged && C % 64 == 0 && slab == C && lds <= 160 * 1024) return no("channels fit LDS in whole steps");
    if (lds > 160 * 1024) return no("patch and weight stages do not fit LDS");
    const int tiles_m = (p.M + k.BM - 1) / k.BM, tiles_n = (p.Nc + k.BN - 1) / k.BN;
    if ((int64_t)tiles_m * tiles_n > 0x7fffffff) return no("grid too large");
    if (lds_bytes) *lds_bytes = lds;
    if (!out) return true;
    DconvParams d;
    std::memset(&d, 0, sizeof d);
    d.x = p.x; d.w = p.w; d.bias = p.bias; d.y = p.y;
    d.x_bytes = p.x_bytes; d.w_bytes = p.w_bytes; d.y_bytes = p.y_bytes;
    d.M = p.M; d.Nc = p.Nc; d.C = p.C; d.Cs = (int32_t)slab;
    d.H = p.H; d.W = p.W; d.R = p.R; d.S = p.S; d.pad_h = p.pad_h; d.pad_w = p.pad_w;
    d.tiles_m = tiles_m; d.tiles_n = tiles_n; d.splitk = 1;
    d.flags = (p.epilogue & (ALT_EPI_BIAS | ALT_EPI_RELU)) | (p.out_bf16 ? kDconvOutBf16 : 0) | (y_nchw ? 0 : kPlanarOutNhwc);
    d.OH = p.OH; d.OW = p.OW; d.stride = st_; d.dil = p.dil_h;
    d.in_px = (int32_t)(N * H * W);
    d.d_hw = make_div32((uint32_t)(p.OH * p.OW));
    d.d_w = make_div32((uint32_t)p.OW);
    order_tiles(&d, 2.0 * C * k.BM * st_ * st_, 2.0 * C * p.R * p.S * k.BN);
    d.d_ihw = make_div32((uint32_t)(H * W));
    d.bk = 64;
    *out = d;
    return true;
}

// The same for the kernel over images of few channels (dstem.h): NCHW activations, filters of up to eight columns under any
// unblocked layout, NHWC or channel-blocked bf16 output.
static bool dstem_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes, std::string *why)
{
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p = pb.p;
    if (pb.dtype != ALT_BF16 || !p.out_bf16) return no("kernel for few channels is bf16 in and out");
    if (p.batch != 1 || pb.groups > 1 || splitk != 1 || p.addend) return no("kernel for few channels takes no batch, groups, split-K or fused sum");
    const int64_t C = p.C, H = p.H, W = p.W, OH = p.OH, OW = p.OW, K = p.Nc, R = p.R, S = p.S, N = p.M / (OH * OW);
    if (C > 4 || S > 8 || C * R > 2 * k.prefetch || p.dil_h != 1 || p.dil_w != 1) return no("more channels, taps or dilation than the kernel for few channels holds");
    if (!(dense(p.xw, W, 1) && dense(p.xh, H, W) && dense(p.xc, C, H * W) && dense(p.xn, N, C * H * W))) return no("activations are not dense NCHW");
    if (!dense(p.wo, K, C * R * S) || (K > 1 && p.wo.si != C * R * S) || p.wi.f < C || p.wr.f < R || p.ws.f < S)
        return no("filter is not dense with the output channel outermost");
    int y_blk = 0;
    if (!nhwc_or_blocked(p.yk, p.yw, p.yh, p.yn, K, OH, OW, N, &y_blk)) return no("output is not dense NHWC or N K/b H W b");
    if (K % 8 || (uintptr_t)p.y % 16) return no("output is stored eight channels at a time");
    if (pb.x_elems * 2 >= 0x7fffffff || p.y_bytes == 0 || pb.w_elems >= 0x7fffffff || C * N * H * W > 0x7fffff00) return no("operand of 2 GiB or more");
    if (C * N * H * W < 8 || pb.w_elems > 0x3fffffff) return no("images of fewer than eight elements");
    const int PCH = dstem_pieces(p.stride_w), PR = dstem_rows(p.stride_h, (int)R);
    const int64_t pieces = (int64_t)dstem_copies(p.stride_w) * C * PR * PCH;
    if (pieces > kStemMaxLoads * 256) return no("patch does not fit the registers it is loaded through");
    const int patch = dstem_patch_bytes(k.BN / 32, (int)(C * R * S), (int)pieces);
    const size_t lds = dstem_lds_bytes(2 * k.prefetch, k.BN / 32, patch);
    if (lds > 64 * 1024) return no("patch does not fit LDS");
    const int64_t tw = (OW + kStemTile - 1) / kStemTile, th = (OH + kStemTile - 1) / kStemTile;
    if (tw * th * N > 0x7fffffff - 4096 || (K + k.BN - 1) / k.BN > 65535) return no("grid too large");
    if (lds_bytes) *lds_bytes = lds;
    if (!out) return true;
    DconvParams d;
    std::memset(&d, 0, sizeof d);
    d.x = p.x; d.w = p.w; d.bias = p.bias; d.y = p.y;
    d.y_bytes = p.y_bytes;
    d.M = p.M; d.Nc = p.Nc; d.C = p.C; d.H = p.H; d.W = p.W; d.R = p.R; d.S = p.S; d.pad_h = p.pad_h; d.pad_w = p.pad_w;
    d.OH = p.OH; d.OW = p.OW; d.stride = p.stride_h; d.stride_w = p.stride_w;
    d.in_px = (int32_t)(N * H * W);
    d.flags = (p.epilogue & (ALT_EPI_BIAS | ALT_EPI_RELU)) | kDconvOutBf16;
    d.tiles_m = (int32_t)(tw * th * N); d.tiles_n = (int32_t)tw; d.splitk = (int32_t)th;
    d.d_w = make_div32((uint32_t)tw);
    d.d_hw = make_div32((uint32_t)th);
    d.d_c16 = make_div32((uint32_t)PCH);
    d.d_rs = make_div32((uint32_t)PR);
    d.d_s = make_div32((uint32_t)R);
    d.ncc = patch;
    d.wst_o = (int32_t)(C * R * S); d.wst_i = (int32_t)p.wi.si; d.wst_r = (int32_t)p.wr.si; d.wst_s = (int32_t)p.ws.si;
    d.y_blk = y_blk;
    *out = d;
    return true;
}

// The same for a kernel over a short reduction (dshort.h): 1x1 filters at stride 1 over dense NHWC, and products of contiguous rows.
static bool dshort_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes, std::string *why)
{
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p = pb.p;
    if (pb.dtype != ALT_BF16 || !p.out_bf16) return no("kernel for short reductions is bf16 in and out");
    if (splitk != 1 || pb.groups > 1 || p.addend) return no("kernel for short reductions takes no split-K, groups or fused sum");
    if (p.R != 1 || p.S != 1 || p.stride_h != 1 || p.stride_w != 1 || p.pad_h != 0 || p.pad_w != 0 || p.OH != p.H || p.OW != p.W)
        return no("kernel for short reductions needs a 1x1 filter, stride 1, no padding");
    const int64_t C = p.C, H = p.H, W = p.W, K = p.Nc, N = p.M / (H * W), stages = (C + 63) / 64;
    if (C % 8) return no("a row's reduction is not a whole number of 16-byte chunks");
    if (stages > (k.BN <= 64 ? kShortStages : 2)) return no("reduction does not fit LDS at once");
    if (!(dense(p.xc, C, 1) && dense(p.xw, W, C) && dense(p.xh, H, W * C) && dense(p.xn, N, H * W * C))) return no("A is not dense with K contiguous");
    if (!(dense(p.wi, C, 1) && dense(p.wo, K, C))) return no("B is not dense with K contiguous");
    if (!(dense(p.yk, K, 1) && dense(p.yw, W, K) && dense(p.yh, H, W * K) && dense(p.yn, N, H * W * K))) return no("output is not dense with N contiguous");
    if ((uintptr_t)p.x % 16 || (uintptr_t)p.w % 16 || (uintptr_t)p.y % 2) return no("operands are not 16-byte aligned");
    if (p.batch > 1 && ((p.x_bstride * 2) % 16 || (p.w_bstride * 2) % 16)) return no("batch entries are not 16-byte aligned");
    if ((p.epilogue & ALT_EPI_BIAS) && (K % 4 || (uintptr_t)p.bias % 16)) return no("bias is loaded four columns at a time");
    if (pb.x_elems * 2 >= 0x7fffffff || pb.w_elems * 2 >= 0x7fffffff || p.y_bytes == 0 || ((int64_t)p.M + k.BM) * C * 2 >= 0x7fffffff ||
        (K + k.BN) * C * 2 >= 0x7fffffff)
        return no("operand of 2 GiB or more");
    const size_t lds = dshort_lds_bytes(k.BN, C);
    const int64_t tiles_m = (p.M + k.BM - 1) / k.BM, tiles_n = (K + k.BN - 1) / k.BN;
    if (tiles_m * tiles_n * p.batch > 0x7fffffff) return no("grid too large");
    if (lds_bytes) *lds_bytes = lds;
    if (!out) return true;
    DconvParams d;
    std::memset(&d, 0, sizeof d);
    d.x = p.x; d.w = p.w; d.bias = p.bias; d.y = p.y;
    d.x_bytes = p.x_bytes; d.w_bytes = p.w_bytes; d.y_bytes = p.y_bytes;
    d.M = p.M; d.Nc = p.Nc; d.C = p.C;
    d.tiles_m = (int32_t)tiles_m; d.tiles_n = (int32_t)tiles_n; d.splitk = 1;
    d.flags = (p.epilogue & (ALT_EPI_BIAS | ALT_EPI_RELU)) | kDconvOutBf16;
    d.d_tn = make_div32((uint32_t)tiles_n);
    d.d_od = make_div32((uint32_t)(tiles_m * tiles_n));
    d.c16 = (int32_t)(C / 8);
    d.x_pix = (uint32_t)(C * 2);
    d.bk = 64;
    d.batch = p.batch;
    d.x_bstride = p.x_bstride * 2; d.w_bstride = p.w_bstride * 2; d.y_bstride = p.y_bstride * 2;
    *out = d;
    return true;
}

// Fills the launch parameters of direct kernel `k` for `pb` split into `splitk`
// channel slices, or says why the kernel does not cover the problem.
bool dconv_setup(const Problem &pb, const IgemmLaunch &k, int splitk, DconvParams *out, size_t *lds_bytes, std::string *why)
{
    if (k.stream == 2) return dplanar_setup(pb, k, splitk, out, lds_bytes, why);
    if (k.stream == 3) return dstem_setup(pb, k, splitk, out, lds_bytes, why);
    if (k.stream == 5) return dshort_setup(pb, k, splitk, out, lds_bytes, why);
    if (k.stream == 4) return dslab_setup(pb, k, splitk, out, lds_bytes, why);
    if (k.taps) return dtaps_setup(pb, k, splitk, out, lds_bytes, why);
    if (k.stream) return dstream_setup(pb, k, splitk, out, lds_bytes, why);
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p = pb.p;
    if (pb.dtype != ALT_BF16) return no("direct kernel is bf16 only");
    if (p.batch != 1) return no("direct kernel takes no batch");
    if (p.stride_h != p.stride_w || (p.stride_h != 1 && p.stride_h != 2) || p.dil_h != p.dil_w || p.dil_h < 1)
        return no("direct kernel needs stride 1 or 2 and one dilation for both directions");
    if (p.pad_h < 0 || p.pad_w < 0 || 2 * p.pad_h > p.dil_h * (p.R - 1) || 2 * p.pad_w > p.dil_w * (p.S - 1))
        return no("direct kernel needs padding between none and same-size");
    const int st_ = p.stride_h;
    // (then OH <= ceil(H / stride) and likewise OW: the input pixel under an output pixel never moves backwards)
    if ((int64_t)(p.OH - 1) * st_ >= p.H || (int64_t)(p.OW - 1) * st_ >= p.W) return no("output larger than the strided input");
    const int64_t C = p.C, H = p.H, W = p.W, OH = p.OH, OW = p.OW, K = p.Nc, R = p.R, S = p.S, N = p.M / (OH * OW);
    int x_blk = 0, y_blk = 0;
    if (!nhwc_or_blocked(p.xc, p.xw, p.xh, p.xn, C, H, W, N, &x_blk)) return no("activations are not dense NHWC or N C/b H W b");
    if (!(dense(p.wi, C, 1) && dense(p.ws, S, C) && dense(p.wr, R, S * C) && dense(p.wo, K, R * S * C)))
        return no("weights are not dense OHWI");
    if (!nhwc_or_blocked(p.yk, p.yw, p.yh, p.yn, K, OH, OW, N, &y_blk)) return no("output is not dense NHWC or N K/b H W b");
    if ((uintptr_t)p.x % 16 || (uintptr_t)p.w % 16) return no("operands are not 16-byte aligned");
    if (splitk < 1 || C % splitk) return no("split factor does not divide the channels");
    const int64_t Cs = C / splitk;
    if (Cs % 64 || (Cs & (Cs - 1)) || Cs > 512) return no("channels per slice must be 64, 128, 256 or 512");
    // K groups: each takes Cs / kw channels, in steps of k.BK (64, or 32: built for 3x3 filters over
    // 32 or 64 channels per group)
    const int kw = k.kw, bk = k.BK;
    if (Cs % kw) return no("K groups do not divide the slice");
    const int64_t Csg = Cs / kw;
    if (Csg % bk) return no("too few channels per K group");
    if (bk == 32 && !(R == 3 && S == 3 && Csg <= 64)) return no("32-channel K steps are built for 3x3 filters over 32 or 64 channels per group");
    if (pb.x_elems * 2 >= 0x7fffffff || pb.w_elems * 2 >= 0x7fffffff || p.y_bytes == 0)
        return no("operand of 2 GiB or more");
    if ((int64_t)p.M * K * 4 >= 0x7fffffff) return no("output too large for 32-bit offsets");
    if (K % 4 || (uintptr_t)p.y % 16 || ((p.epilogue & ALT_EPI_BIAS) && (uintptr_t)p.bias % 16))
        return no("direct kernel stores four output channels at a time");
    const size_t lds = dconv_lds_bytes(k.BM, k.BN, k.prefetch + 1, k.wgn, kw, bk, (int)Cs,
                                       dconv_patch_pixels(k.BM, p.M, p.H, p.W, p.OH, p.OW, p.R, p.S, p.pad_h, p.pad_w, st_, p.dil_h));
    if (lds > 160 * 1024) return no("patch does not fit LDS");
    const int tiles_m = (p.M + k.BM - 1) / k.BM, tiles_n = (p.Nc + k.BN - 1) / k.BN;
    if (splitk > 1 && (int64_t)tiles_m * tiles_n > kDconvMaxTiles) return no("too many output tiles for the split-K counters");
    if ((int64_t)tiles_m * tiles_n * splitk > 0x7fffffff) return no("grid too large");
    if (lds_bytes) *lds_bytes = lds;
    if (!out) return true;
    DconvParams d;
    std::memset(&d, 0, sizeof d);
    d.x = p.x; d.w = p.w; d.bias = p.bias; d.y = p.y; d.addend = p.addend;
    d.x_bytes = p.x_bytes; d.w_bytes = p.w_bytes; d.y_bytes = p.y_bytes;
    d.partial_bytes = (uint32_t)((int64_t)p.M * K * 4);
    d.M = p.M; d.Nc = p.Nc; d.C = p.C; d.Cs = (int32_t)Cs;
    d.H = p.H; d.W = p.W; d.R = p.R; d.S = p.S; d.pad_h = p.pad_h; d.pad_w = p.pad_w;
    d.tiles_m = tiles_m; d.tiles_n = tiles_n; d.splitk = splitk;
    d.flags = (p.epilogue & (ALT_EPI_BIAS | ALT_EPI_RELU)) | (p.out_bf16 ? kDconvOutBf16 : 0);
    d.OH = p.OH; d.OW = p.OW; d.stride = st_; d.dil = p.dil_h;
    if (N * H * W > 0x7fffffff) return no("input too large for 32-bit pixel indices");
    d.in_px = (int32_t)(N * H * W);
    d.d_hw = make_div32((uint32_t)(p.OH * p.OW));
    d.d_w = make_div32((uint32_t)p.OW);
    order_tiles(&d, 2.0 * Cs * k.BM * st_ * st_, 2.0 * Cs * p.R * p.S * k.BN);
    int l2 = 0;
    while ((8 << l2) < Cs) ++l2;
    d.log2_cpp = l2;
    d.d_slots = make_div32((uint32_t)(Cs / 8 + 1));
    d.ncc = (int32_t)(Csg / bk);
    d.bk = bk;
    d.x_blk = x_blk; d.y_blk = y_blk;
    d.d_ihw = make_div32((uint32_t)(H * W));
    *out = d;
    return true;
}

// The arrival counters of launches on `st`.
static hipError_t stream_counters(hipStream_t st, uint32_t **out)
{
    uint32_t *base = nullptr;
    hipError_t e = dconv_counters(&base);
    if (e != hipSuccess) return e;
    int slot = 0;
    e = counter_slot(device_state(), st, &slot);
    if (e != hipSuccess) return e;
    *out = base + (size_t)slot * kDconvMaxTiles;
    return hipSuccess;
}

hipError_t dconv_run(const IgemmLaunch &k, DconvParams d, size_t lds, float *partial, hipStream_t st)
{
    if (d.splitk > 1 && k.stream != 3) {
        hipError_t e = stream_counters(st, &d.counters);
        if (e != hipSuccess) return e;
        d.partial = partial;
    }
    return k.launch_direct(d, lds, st);
}

// A problem's sliced tiles in a launch of several have counters of their own.
hipError_t group_run(const GroupFamily &f, GroupParams *g, unsigned workgroups, size_t lds, hipStream_t st)
{
    uint32_t *counters = nullptr;
    for (int i = 0; i < g->n; ++i) {
        if (g->p[i].splitk <= 1) continue;
        if (!counters) {
            const hipError_t e = stream_counters(st, &counters);
            if (e != hipSuccess) return e;
        }
        g->p[i].counters = counters;
        counters += g->p[i].tiles_m * g->p[i].tiles_n;
    }
    return f.launch(*g, workgroups, lds, st);
}

}  // namespace alt
