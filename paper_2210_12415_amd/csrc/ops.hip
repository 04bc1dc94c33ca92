// Host side of alt_conv2d / alt_gemm: descriptor checks, mapping of layouts to
// the implicit-GEMM kernel's addressing, variant table, split-K reduction,
// weight packing.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "dplanar.h"
#include "group.h"
#include "igemm.h"
#include "ops.h"

namespace alt {

// ---- kernel registry -----------------------------------------------------------

static std::vector<IgemmLaunch> &registry()
{
    static std::vector<IgemmLaunch> v;
    return v;
}

void igemm_register(const IgemmLaunch &l) { registry().push_back(l); }

const std::vector<IgemmLaunch> &igemm_table()
{
    static std::once_flag once;
    std::call_once(once, [] {
        auto &v = registry();
        std::sort(v.begin(), v.end(), [](const IgemmLaunch &a, const IgemmLaunch &b) {
            return std::strcmp(a.name, b.name) < 0;
        });
    });
    return registry();
}

const int kSplitFactors[] = {1, 2, 3, 4, 6, 8, 9, 12, 16, 18, 24, 36};
static const int *const kSplits = kSplitFactors;
constexpr int kNumSplits = 12;
int igemm_num_splits() { return kNumSplits; }

int igemm_variant_count() { return (int)igemm_table().size() * kNumSplits; }

// ---- split-K reduction + epilogue ----------------------------------------------

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const IgemmParams p)
{
    const int64_t per_batch = (int64_t)p.M * p.Nc;
    const int64_t total = per_batch * p.batch;
    const int ohow = p.OH * p.OW;
    for (int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int bz = p.batch == 1 ? 0 : (int)(e / per_batch);
        const int64_t r = e - bz * per_batch;
        const int m = (int)fast_div((uint32_t)r, p.fd_nc), n = (int)(r - (int64_t)m * p.Nc);
        float v = 0.f;
        for (int s = 0; s < p.splitk; ++s) v += p.partial[(int64_t)s * total + e];
        if (p.epilogue & ALT_EPI_BIAS) v += p.bias[bz * p.bias_bstride + n];
        if (p.epilogue & ALT_EPI_RELU) v = fmaxf(v, 0.f);
        const int img = (int)fast_div(m, p.fd_ohow), rem = m - img * ohow;
        const int oh = (int)fast_div(rem, p.fd_ow), ow = rem - oh * p.OW;
        const int64_t off = (int64_t)bz * p.y_bstride + dim2_off(p.yn, img) + dim2_off(p.yk, n) +
                            dim2_off(p.yh, oh) + dim2_off(p.yw, ow);
        if (p.out_bf16) ((uint16_t *)p.y)[off] = f32_to_bf16_rne(v);
        else ((float *)p.y)[off] = v;
    }
}

// ---- eligibility of loaders ------------------------------------------------------

static bool mult(int64_t v, int m) { return v % m == 0; }

void igemm_analyse(Problem *pb)
{
    const IgemmParams &p = pb->p;
    const int epv = pb->dtype == ALT_BF16 ? 8 : 4;
    const int es = pb->dtype == ALT_BF16 ? 2 : 4;
    const bool x_spatial_split = (p.xh.f < p.H) || (p.xw.f < p.W);
    pb->spatial_split = x_spatial_split;
    pb->spatial_ok = !x_spatial_split || (p.R == 1 && p.S == 1 && p.pad_h == 0 && p.pad_w == 0);
    // A: 16-byte loads along channels
    pb->a_vec = p.xc.si == 1 && mult(p.xc.f, epv) && (p.xc.f >= p.C || mult(p.xc.so, epv)) &&
                mult(p.xn.si, epv) && mult(p.xn.so, epv) && mult(p.xh.si, epv) && mult(p.xh.so, epv) &&
                mult(p.xw.si, epv) && mult(p.xw.so, epv) && mult(p.x_bstride, epv) &&
                ((uintptr_t)p.x % 16 == 0) && pb->spatial_ok && pb->x_elems * es < 0x7fffffff;
    // A: rows (GMM m) contiguous, no spatial structure
    pb->a_trans = p.H == 1 && p.R == 1 && p.S == 1 && p.pad_h == 0 && p.pad_w == 0 && p.stride_w == 1 &&
                  p.xw.si == 1 && p.xw.f >= p.W && mult(p.M, epv) && p.xc.f >= p.C && mult(p.xc.si, epv) &&
                  mult(p.x_bstride, epv) && ((uintptr_t)p.x % 16 == 0) && p.OW == p.M;
    pb->b_vec = p.wi.si == 1 && mult(p.wi.f, epv) && (p.wi.f >= p.C || mult(p.wi.so, epv)) &&
                mult(p.wo.si, epv) && mult(p.wo.so, epv) && mult(p.wr.si, epv) && mult(p.wr.so, epv) &&
                mult(p.ws.si, epv) && mult(p.ws.so, epv) && mult(p.w_bstride, epv) &&
                ((uintptr_t)p.w % 16 == 0) && pb->w_elems * es < 0x7fffffff;
    pb->b_trans = p.R == 1 && p.S == 1 && p.wo.si == 1 && mult(p.wo.f, epv) &&
                  (p.wo.f >= p.Nc || mult(p.wo.so, epv)) && mult(p.Nc, epv) && mult(p.wi.si, epv) &&
                  mult(p.wi.so, epv) && mult(p.w_bstride, epv) && ((uintptr_t)p.w % 16 == 0);
}

static bool nests(int64_t f, int64_t C, int bk) { return f >= C ? true : (f % bk == 0 || bk % f == 0); }

// Can kernel `k` with split factor `splitk` run this problem?  `p`: a copy of the parameters, or null; its launch-dependent fields but
// the divisors (igemm_divisors) are filled in.  Choosing a kernel asks this a thousand times, so no copy is made here.
static bool applicable(const Problem &pb, const IgemmLaunch &k, int splitk, IgemmParams *p, std::string *why, size_t *lds_bytes)
{
    auto no = [&](const char *m) { if (why) *why = m; return false; };
    const IgemmParams &p0 = pb.p;
    if (k.dtype != pb.dtype) return no("element type");
    if (pb.v.T && !k.taps) return no("depth taps and output phases are built into the kernels over filter taps only");
    if (p0.addend && !k.launch_direct) return no("the fused sum is built into the tile kernels only");
    if (k.launch_direct) {
        if (!dconv_setup(pb, k, splitk, nullptr, lds_bytes, why)) return false;
        if (p) {
            p->splitk = splitk;
            if (k.taps) {
                const int64_t taps = pb.v.T ? (int64_t)pb.v.taps[0] * pb.v.taps[1] * pb.v.taps[2] : (int64_t)p0.R * p0.S;
                p->ksteps_total = (int32_t)((taps * p0.C + k.BK - 1) / k.BK);
                p->ksteps_per_split = (p->ksteps_total + splitk - 1) / splitk;
            }
            p->tiles_m = (p0.M + k.BM - 1) / k.BM;
            p->tiles_n = (p0.Nc + k.BN - 1) / k.BN;
        }
        return true;
    }
    if (!pb.spatial_ok && (k.amode != LOAD_GATHER)) return no("blocked H/W needs R=S=1 without padding");
    const bool uniform = p0.C % k.BK == 0 && nests(p0.xc.f, p0.C, k.BK) && nests(p0.wi.f, p0.C, k.BK);
    if (k.amode == LOAD_VEC && !(pb.a_vec && uniform)) return no("A is not channel-contiguous in 16-byte blocks");
    if (k.bmode == LOAD_VEC && !(pb.b_vec && uniform)) return no("B is not channel-contiguous in 16-byte blocks");
    if (k.amode == LOAD_TRANS && !pb.a_trans) return no("A rows are not contiguous");
    if (k.bmode == LOAD_TRANS && !pb.b_trans) return no("B rows are not contiguous");
    if (pb.spatial_split && k.amode == LOAD_GATHER && !(p0.R == 1 && p0.S == 1 && p0.pad_h == 0 && p0.pad_w == 0))
        return no("blocked H/W with a sliding window");
    const int32_t steps = (p0.Kg + k.BK - 1) / k.BK, per_split = splitk < 1 ? 0 : (steps + splitk - 1) / splitk;
    if (splitk < 1 || splitk > steps) return no("split-K factor exceeds the K steps");
    if (splitk > 1 && (int64_t)p0.M * p0.Nc * 4 >= 0x7fffffff) return no("output too large for the split-K reduction");
    if ((int64_t)(splitk - 1) * per_split >= steps) return no("split-K factor leaves an empty slice");
    if ((int64_t)p0.batch * splitk > 65535) return no("batch x split-K exceeds the grid");
    if (p) {
        p->uniform_rs = uniform ? 1 : 0;
        p->spatial_split = pb.spatial_split ? 1 : 0;
        p->ksteps_total = steps;
        p->splitk = splitk;
        p->ksteps_per_split = per_split;
        p->tiles_m = (p0.M + k.BM - 1) / k.BM;
        p->tiles_n = (p0.Nc + k.BN - 1) / k.BN;
    }
    return true;
}

// What only a launch of a register-staged kernel needs beside that.
static void igemm_divisors(IgemmParams *p)
{
    p->fd_ohow = make_fastdiv((uint32_t)(p->OH * p->OW));
    p->fd_ow = make_fastdiv((uint32_t)p->OW);
    p->fd_c = make_fastdiv((uint32_t)p->C);
    p->fd_s = make_fastdiv((uint32_t)p->S);
    p->fd_nc = make_fastdiv((uint32_t)p->Nc);
}

bool igemm_applicable(const Problem &pb, const IgemmLaunch &k, int splitk, std::string *why)
{
    return applicable(pb, k, splitk, nullptr, why, nullptr);
}

size_t igemm_workspace(const Problem &pb, int splitk)
{
    if (splitk <= 1) return 0;
    return (size_t)splitk * pb.p.batch * pb.p.M * pb.p.Nc * sizeof(float);
}

// What a workgroup of a tile kernel takes of a compute unit: clocks alone, and more for each beside it.
struct TileClocks {
    double alone, beside;
};
template <typename F>
static void tile_clocks(TileClocks *one, F &&round_clk)
{
    if (one) *one = {round_clk(1.0), round_clk(4.0) - round_clk(3.0)};
}

// Microseconds of a bf16 tile kernel (patch-resident, streaming, over filter taps).  A workgroup opens (latency of its first loads,
// and the patch), walks its K steps and stores its tile; as many share a compute unit as LDS and registers allow, and a round of
// them takes what they ask of the unit together (matrix cores, operand bytes into LDS and out of it), but no less than one alone,
// which waits at every step.  Clocks at 2.2 GHz.  Fitted over 43000 launches (740 layers and products of 4 to 500 us under 60 to 100
// variants each): the choice takes 3 % longer than the fastest variant on average.  (The estimate before priced slices and patches
// too low: 30 % on the 3x3 and 1x1 layers among them; 16 x 128 x 28 x 28, 3x3, ran in 19.5 us where 7.7 were to be had, 256 x
// 512 x 7 x 7 in 122 where 69 were.)  What it does not know: how often an L2 line is fetched again, which matters for few output channels
// (86 x 512 x 43 x 43 to 8, 5x5: 468 us on the choice, 249 on the fastest).
static double tile_estimate_us(const Problem &pb, const IgemmLaunch &k, const IgemmParams &p, size_t lds, TileClocks *one)
{
    const bool patch = k.stream == 0;
    const int waves = k.kw * k.wgm * k.wgn;
    const double wtm = (double)k.BM / k.wgm, wtn = (double)k.BN / k.wgn, acc = wtm * wtn / 64;
    const double per_cu = std::max(1.0, std::min(std::floor(160.0 * 1024 / lds), std::floor((acc <= 32 ? 16.0 : 8.0) / waves)));
    const double blocks = (double)p.tiles_m * p.tiles_n * p.splitk * p.batch;
    const double steps = k.taps ? std::ceil((double)p.ksteps_per_split / k.kw) : (double)p.R * p.S * p.C / p.splitk / k.kw / k.BK;
    // (what bounds a step overlaps with the rest of it only in part: the parts' cubes are added, between sum and maximum)
    auto cube = [](double v) { return v * v * v; };
    const double mfma = (double)k.kw * k.BM * k.BN * k.BK / 2048.0;                  // clocks of a step's products on four SIMDs
    const double in = (double)k.kw * ((patch ? 0 : k.BM) + k.BN) * k.BK * 2 / 46.6;   // ... of its operands' way into LDS
    const double out = waves * (wtm + wtn) * k.BK * 2 / 400.0;                        // ... and out of it
    // (the patch-resident kernels' loop over taps and channels is unrolled for up to two steps a tap, and of one tap)
    const bool walks = patch && p.R * p.S > 1 && !(p.R == 3 && p.S == 3 && steps <= 2 * 9);
    const double alone = std::max(mfma * (waves >= 8 ? 1.0 : 1.47) * std::max(1.0, 4.0 / waves), in) + (patch ? 86.0 : 0.0) +
                         (walks ? 417.0 : 0.0) + (k.taps == kTapsRagged ? 97.0 : 0.0);
    const double np = patch ? (double)k.BM * p.stride_h * p.stride_h + 2.0 * (p.pad_h * p.W + p.pad_w) : 0.0;
    const double ends = 4970.0 - (patch ? 180.0 : !k.taps ? 1600.0 : 0.0) - (k.bt ? 1080.0 : 0.0) + (patch ? 0.0 : 9.6 * k.BM) +
                        (waves < 8 && acc >= 64 ? 1420.0 : 0.0) + (k.kw > 1 ? 700.0 + (double)k.kw * k.BM * k.BN / 74.0 : 0.0);
    // (half steps beside whole ones of the same tile: 128 x 128 x 32 takes 10 to 25 % longer than 128 x 128 x 64 where both apply)
    const double begin = !patch && k.BK == 32 ? 15.0 : 0.0;
    auto round_clk = [&](double n) {
        const double rate = acc >= 128 ? 1.0 : waves * n >= 8 ? 1.34 : 1.04;
        const double products = n * mfma * rate * std::max(1.0, 4.0 / (waves * n));
        const double step = std::cbrt(cube(products) + cube(n * in) + cube(n * out) + cube(alone)) + begin;
        return steps * step + ends + n * (k.BM * k.BN / 6.67 + np * p.C / p.splitk * 2 / 83.0);
    };
    tile_clocks(one, round_clk);
    const double whole = std::floor(blocks / (256.0 * per_cu)), rest = std::ceil((blocks - whole * 256.0 * per_cu) / 256.0);
    double us = 1.18 + (whole * round_clk(per_cu) + (rest > 0 ? round_clk(rest) : 0.0)) / 2200.0;
    // (a split's partial sums are written, fetched and added by whoever comes last)
    if (p.splitk > 1) us += 1.11 + 0.47 * p.splitk + 0.67e-6 * p.splitk * p.M * (double)p.Nc * p.batch * 4.0;
    const int entries = pb.v.T ? 1 : p.batch;
    const double mem = 1.18 + 2.0 * ((double)(pb.x_elems + pb.w_elems) * entries + (double)p.M * p.Nc * p.batch) / 4.64e6;   // the tensors' way from and to memory
    return std::sqrt(std::cbrt(cube(us * us) + cube(mem * mem)));
}

// The same for the patch-resident kernels over slabs of channels, fitted over 640 launches (100 3x3 layers of 5 to 400 us): a slab costs
// 400 clocks beside its steps, since no operand read is in flight where two meet, and each slab's patch adds to what its steps load.
// (Volumes and output phases down to a few positions too: over 120 of 9 to 25000 positions the choice with these kernels takes 0.87 of the time
// it takes without them, 0.94 below 64 positions, where a split of a longer sum is sometimes faster: 72 channels on 1x9x1, 3x3x3, 9.1 us against 7.5.)
static double slab_estimate_us(const Problem &pb, const IgemmLaunch &k, const IgemmParams &p, size_t lds, TileClocks *one)
{
    const int nwg = k.wgm * k.wgn, waves = k.kw * nwg;
    const int taps = pb.v.T && p.batch > 1 ? pb.v.taps[1] * pb.v.taps[2] : p.R * p.S;
    const int depth = pb.v.T ? p.batch > 1 ? pb.v.taps[0] : pb.v.T : 1;
    const double wtm = (double)k.BM / k.wgm, wtn = (double)k.BN / k.wgn, acc = wtm * wtn / 64;
    const double per_cu = std::max(1.0, std::min(std::floor(160.0 * 1024 / lds), std::floor((acc <= 32 ? 16.0 : 8.0) / waves)));
    const double blocks = (double)p.tiles_m * p.tiles_n * p.batch;
    const double slabs = std::ceil(std::ceil((double)p.C / k.BK) * depth / k.kw), steps = slabs * taps;
    const double np = k.BM + 2.0 * p.dil_h * (p.W + 1);
    const double mfma = (double)k.kw * k.BM * k.BN * k.BK / 2048.0;
    const double in = (double)k.kw * (k.BN * k.BK * 2 + np * (k.BK * 2 + 16) / taps) / 63.0;
    const double out = waves * (wtm + wtn) * k.BK * 2 / 400.0;
    const double alone = std::max(mfma * (waves >= 8 ? 1.0 : 1.34) * std::max(1.0, 4.0 / waves), in);
    auto cube = [](double v) { return v * v * v; };
    auto round_clk = [&](double n) {
        const double products = n * mfma * (waves * n >= 8 ? 1.3 : 1.0) * std::max(1.0, 4.0 / (waves * n));
        return steps * std::cbrt(cube(products) + cube(n * in) + cube(n * out) + cube(alone)) + slabs * 408.0 + 5340.0 -
               (waves >= 8 ? 1475.0 : 0.0) + n * k.BM * k.BN / 3.36 + (k.kw > 1 ? 2950.0 + (double)k.kw * k.BM * k.BN / 74.0 : 0.0);
    };
    tile_clocks(one, round_clk);
    const double whole = std::floor(blocks / (256.0 * per_cu)), rest = std::ceil((blocks - whole * 256.0 * per_cu) / 256.0);
    const double us = 1.18 + (whole * round_clk(per_cu) + (rest > 0 ? round_clk(rest) : 0.0)) / 2200.0;
    const double mem = 1.18 + 2.0 * ((double)pb.x_elems + pb.w_elems + (double)p.M * p.Nc * p.batch) / 4.64e6;
    return std::sqrt(std::cbrt(cube(us * us) + cube(mem * mem)));
}

// The same for the kernels of a short reduction: what a workgroup's loads (those past the operands' ends cost too), products, bias and stores (rows that
// do not begin at 16 bytes cost nearly twice) take of a compute unit, the chain that it is, rounds of as many as share one, and the tensors' way from and
// to memory.  Fitted over 5600 products and 1x1 layers (K up to 256, with and without bias, batches, 4 to 400 us) under all three tiles, rms 12 %.
// (The fit before was over products without bias and large K alone, 30 % too high for 32 columns and as much too low for 96 with a bias: 238 of
// the 5600 took over 5 % longer than without these kernels, 46 x 248 x 76 x 76 to 296 209 us instead of 144.)
static double short_estimate_us(const IgemmLaunch &k, const IgemmParams &p, size_t lds)
{
    const double rows = (double)p.M / p.tiles_m, cols = (double)p.Nc / p.tiles_n, stages = std::ceil(p.C / 64.0);
    const double rounds = (double)p.tiles_m * p.tiles_n * p.batch / 256.0;
    const double per_cu = std::max(1.0, std::min(std::floor(160.0 * 1024 / lds), k.BN <= 64 ? 4.0 : 3.0));
    const double busy = (rows + cols) * p.C * 2 / 353.0 + stages * (k.BM + k.BN) * 128 / 127.0 + rows * cols * 2 / 35.7 * (p.Nc % 8 ? 1.85 : 1.0) +
                        k.BN / 32 * (stages * 170.0 + (p.epilogue & ALT_EPI_BIAS ? 152.0 : 0.0));
    const double work = busy * std::max(1.0, rounds), chain = (455.0 + 1.195 * busy) * std::max(1.0, rounds / per_cu);
    return 2.49 + (work + chain) / 2200.0 + 2.0 * p.batch * ((double)p.M * p.C + (double)p.Nc * p.C + (double)p.M * p.Nc) / 17.7e6;
}

// Microseconds of a tile kernel.  *family: what the choice between families multiplies them with.
static double direct_estimate_us(const Problem &pb, const IgemmLaunch &k, const IgemmParams &p, size_t lds, double *family, TileClocks *one = nullptr)
{
    *family = 0.05;
    if (k.stream == 4) return slab_estimate_us(pb, k, p, lds, one);
    if (k.stream == 5) {
        // (a little behind the others, whose estimates are 9 % high in the median over the same problems: at this factor the choice takes 2.3 % longer than
        // the fastest, 0.736 of the time without these kernels, and 81 of 5600 problems take more than 5 % longer, at 0.05 1.7 %, 0.732 and 162)
        *family = 0.054;
        return short_estimate_us(k, p, lds);
    }
    if (k.stream <= 1 && k.dtype == ALT_BF16) {
        // (a small factor: wherever one of these kernels applies it has been faster than the register-staged ones, whose estimate below
        // knows little of slices and short sums: at half, 4 x 128 x 5 x 5, 3x3, went there in 36 slices and took 15.6 us, not 7.8.
        // A 1x1 filter leaves a patch nothing to reuse: the streaming kernels run it without staging one first.)
        if (k.stream == 0 && p.R * p.S == 1) *family = 0.075;
        return tile_estimate_us(pb, k, p, lds, one);
    }
    if (k.stream == 1) {
        const int waves = k.kw * k.wgm * k.wgn;
        const double es = 4.0;
        const int per_cu = std::max(1, (int)(160.0 * 1024 / lds));
        const double blocks = (double)p.tiles_m * p.tiles_n * p.splitk * p.batch;
        const double steps = k.taps ? std::ceil((double)p.ksteps_per_split / k.kw) : (double)p.C / p.splitk / k.kw / k.BK;
        // (a split's partial sums are written, fetched and added by whoever comes last: fitted over products of 37 to 10000 rows,
        // 1 us a MB of them; 1536 x 512 x 2048 in eight slices of 256x128 tiles took 38 us, unsplit on 64x64 tiles 10.8)
        const double partial_us = p.splitk > 1 ? 1e-6 * p.splitk * p.M * (double)p.Nc * p.batch * 4.0 : 0.0;
        // fp32: matrix instructions do a sixteenth of the products per clock, so co-resident workgroups share them; a
        // step costs 280 clocks beside its products, a workgroup 7200, a split 0.8 us and 0.9 us a MB (microseconds, within 10 %
        // of 1000 measured launches).  The factor brings them to the estimate of the register-staged kernels, which take two
        // to six times what it says, in steps of 512 tiles.  Of 122 convolutions and products of 5 to 200 us the choice is 2.5 %
        // from the fastest variant on average; the five 3x3 and 1x1 layers stay on these kernels from batch 1 to 40, where the
        // others are at most 5 % faster (64 channels at batch 12, 36.4 us against 38.4) and up to 40 % slower.  At 0.2 batches 16
        // to 23 of two of them go to the others and lose 5 to 16 %.  A step that spans taps (fewer channels than a step is
        // deep) costs more: 28 x 16 x 36 x 36 to 424 channels, 5x5, takes 140 us here and 122 on the others.
        const double need = std::max((double)k.kw * k.BM * k.BN * k.BK / 128.0 * (waves >= 8 ? 1.11 : 1.07) * std::max(1.0, 4.0 / waves),
                                     (double)k.kw * (k.BM + k.BN) * k.BK * es / 33.6);
        auto round_clk = [&](double n) { return steps * std::max(need + 280.0, n * need) + 7200.0; };
        tile_clocks(one, round_clk);
        const double whole = std::floor(blocks / (256.0 * per_cu)), rest = std::ceil((blocks - whole * 256.0 * per_cu) / 256.0);
        const double us = (whole * round_clk(per_cu) + (rest > 0 ? round_clk(rest) : 0.0)) / 2200.0 + (p.splitk > 1 ? 0.8 + 0.9 * partial_us : 0.0);
        // (Batches take no slices here.  A handful of tiles of a long sum leaves the chip idle, and the register-staged kernels in
        // slices take 0.5 to 1.06 times as long: 2 x 4 x 28 x 6360 32 us against 61, 11 x 2 x 8 x 5556 57 and 53; with 22 tiles it
        // is 50 and 39.  The estimate of those that gather is an order too high, hence the factor.)
        const double idle = p.batch > 1 && blocks <= 12.0 && p.C >= 2000 ? 12.0 : 1.0;
        *family = (p.C < 32 && p.R * p.S > 1 ? 0.2 : 0.18) * idle;
        return us;
    }
    if (k.stream == 2) {
        // Channel-planar kernel: a workgroup converts its patch on the way in, 64 pixels x 64 channels of it by a wave at a time (a
        // chain of loads, more where planes do not begin at eight pixels; each plane's run touches 128 bytes more than it has); then
        // per super-step of 64 channels (the last one filled up) it runs all taps out of LDS (matrix-core time of the tile, or the way of the
        // weights into their stages), waits at two barriers, and at a slab's end for the next one's patch; then it stores its tile plane
        // by plane.  A round of workgroups asks of a compute unit what they ask together and waits a little longer than one does.  Clocks
        // at 2.2 GHz, fitted over half of 647 layers and products under all seven tiles, of 4 to 300 us; over the other half the choice takes
        // 1.0 % longer than the fastest tile on average.  (The estimate before left a broken last super-step out, so that 24 channels had no
        // products, and took LDS for all channels at once: 4.3 %; 8 x 320 x 68 x 68 to 80, 1x1, took 29.0 us where 17.9 were to be had.)
        const int taps = p.R * p.S, st = p.stride_h, waves = k.kw * k.wgm * k.wgn;
        const double np = (double)k.BM * st * st + (double)(p.dil_h * (p.R - 1)) * p.W + p.dil_w * (p.S - 1);
        size_t whole_lds = 0;
        const double steps = std::ceil(p.C / 64.0);
        const double slabs = std::ceil(steps * 64.0 / planar_slab(k.BM, k.BN, k.kw, taps, p.C, (size_t)np, k.ragged, &whole_lds));
        const double per_cu = std::max(1.0, std::min(std::floor(160.0 * 1024 / lds), std::floor(16.0 / waves)));
        const double weights = (double)k.BN * 64 * taps * 2 / 18.0;
        const double unaligned = p.H * p.W % 8 ? 1.42 : 1.0;
        const double loads = std::ceil(std::ceil(np / 64.0) * steps / waves) * 950.0 * unaligned;
        const double stored = (double)k.BM * (k.BN + (p.out_bf16 ? 0 : std::min(k.BN, p.Nc)));
        auto round_clk = [&](double n) {
            const double products = taps * (double)k.BM * k.BN / 32.0 * (waves * n >= 8 ? 2.6 : 4.6) * std::max(1.0, 4.0 / (waves * n));
            return n * ((np + 64.0) * p.C * 2 / 30.5 * unaligned + steps * std::max(products, weights) + stored / 3.15) +
                   (1.0 + 0.04 * (n - 1.0)) * (1360.0 + loads + steps * 530.0 + slabs * 270.0) + (k.kw > 1 ? 630.0 * k.kw : 0.0);
        };
        tile_clocks(one, round_clk);
        const double blocks = (double)p.tiles_m * p.tiles_n;
        const double whole = std::floor(blocks / (256.0 * per_cu)), rest = std::ceil((blocks - whole * 256.0 * per_cu) / 256.0);
        // (against the register-staged kernels: they gather a layer's operands, and of 275 layers all but three are fastest here, whatever the
        // factor up to 1.  Products with rows of A contiguous take no slices here.  The kernels that transpose aligned rows promise too much, the
        // ones that gather others too little: at these factors the choice between the families takes 0.6 % and 3.3 % longer than the better
        // one, at 0.5 for all 0.6 % and 7.3 %: 47 x 664 x 3960 takes 60 us here, 36 there; 112 x 1464 x 704 7.9 here, 15.1 there.)
        *family = p.H == 1 && p.R * p.S == 1 && p.W % 8 ? 1.3 : 0.5;
        return 1.67 + (whole * round_clk(per_cu) + (rest > 0 ? round_clk(rest) : 0.0)) / 2200.0;
    }
    // Kernel for images of few channels: a start (the filter into registers), then 16 x 16 pixel tiles at a rate per
    // compute unit.  Measured (7x7 over three channels): 2.2 us per 256 tiles of 32 channels, 2.5 of 64, and starts of 4.5
    // and 6.5 us; the padded part of the reduction counts in full.
    const double tiles = std::ceil((double)p.M / 256.0) * std::ceil((double)p.Nc / k.BN) / 256.0;
    const double us = k.BN == 32 ? 4.5 + std::max(tiles, 0.5) * (1.4 + 0.07 * k.prefetch) : 6.5 + std::max(tiles, 0.5) * (1.4 + 0.1 * k.prefetch);
    *family = 0.5;
    return us;
}

// Rough relative time of one variant, about 45 to the microsecond.  lds: bytes of a workgroup of a tile kernel.
double igemm_estimate(const Problem &pb, const IgemmLaunch &k, const IgemmParams &p, size_t lds)
{
    if (k.launch_direct) {
        double family;
        const double us = direct_estimate_us(pb, k, p, lds, &family);
        return family * 45.0 * us;
    }
    // Register-staged kernels: rounds of workgroups over the chip, their K steps, gathering and transposing loaders penalised.
    double mode_cost = 1.0;
    if (k.amode == LOAD_GATHER) mode_cost *= 6.0;
    if (k.bmode == LOAD_GATHER) mode_cost *= 3.0;
    if (k.amode == LOAD_TRANS) mode_cost *= 1.5;
    if (k.bmode == LOAD_TRANS) mode_cost *= 1.5;
    if (k.prefetch > 1) mode_cost *= 0.8;
    const double blocks = (double)p.tiles_m * p.tiles_n * p.splitk * p.batch;
    const double rounds = std::ceil(blocks / 512.0);
    const double step = (double)k.BM * k.BN * k.BK / 16384.0 + 3.0 * (k.BM + k.BN) * k.BK / 8192.0 + 2.0;
    double est = rounds * (p.ksteps_per_split * step + 60.0) * mode_cost;
    if (p.splitk > 1) est += 30.0 + 0.00002 * p.splitk * (double)p.M * p.Nc * p.batch;
    return est;
}

void igemm_for_each(const Problem &pb, size_t ws_limit, bool counters, const std::function<void(int, double)> &seen)
{
    const auto &tab = igemm_table();
    IgemmParams p = pb.p;
    for (int ki = 0; ki < (int)tab.size(); ++ki) {
        const IgemmLaunch &k = tab[ki];
        if (k.dtype != pb.dtype || (pb.v.T && !k.taps)) continue;
        // (the first factor is 1; the channel-planar, few-channel and slab kernels take no other)
        const int splits = k.launch_direct && (!counters || k.stream >= 2) ? 1 : kNumSplits;
        for (int si = 0; si < splits; ++si) {
            size_t lds = 0;
            if (igemm_workspace(pb, kSplits[si]) > ws_limit) continue;
            if (applicable(pb, k, kSplits[si], &p, nullptr, &lds)) seen(ki * kNumSplits + si, igemm_estimate(pb, k, p, lds));
        }
    }
}

int igemm_default_variant(const Problem &pb, size_t ws_limit, bool counters)
{
    double best = 1e300;
    int best_v = -1;
    igemm_for_each(pb, ws_limit, counters, [&](int v, double est) { if (est < best) { best = est; best_v = v; } });
    return best_v;
}

alt_status_t igemm_run(alt_handle_t h, const Problem &pb, int variant, void *workspace, size_t ws_bytes,
                       hipStream_t st, bool *no_counters, TileLaunch *kept)
{
    if (!h->has_gpu) return fail(h, ALT_HIP_ERROR, "no GPU device available");
    const auto &tab = igemm_table();
    if (variant < 0 || variant >= (int)tab.size() * kNumSplits)
        return fail(h, ALT_INVALID_ARG, "variant %d out of range", variant);
    const IgemmLaunch &k = tab[variant / kNumSplits];
    const int splitk = kSplits[variant % kNumSplits];
    const size_t need = igemm_workspace(pb, splitk);
    std::string why;
    if (k.launch_direct) {
        TileLaunch once;
        TileLaunch &t = kept ? *kept : once;
        if (t.variant != variant) {
            if (!igemm_applicable(pb, k, splitk, &why) || !dconv_setup(pb, k, splitk, &t.d, &t.lds, &why))
                return fail(h, ALT_UNSUPPORTED, "variant %s/splitk%d not applicable: %s", k.name, splitk, why.c_str());
            t.variant = variant;
        }
        if (need > 0 && (!workspace || ws_bytes < need))
            return fail(h, ALT_WORKSPACE_TOO_SMALL, "split-K needs %zu workspace bytes, got %zu", need, ws_bytes);
        t.d.x = pb.p.x; t.d.w = pb.p.w; t.d.bias = pb.p.bias; t.d.y = pb.p.y; t.d.addend = pb.p.addend;
        hipError_t e = dconv_run(k, t.d, t.lds, (float *)workspace, st);
        if (e == hipErrorNotReady && no_counters) *no_counters = true;
        if (e == hipErrorNotReady)
            return fail(h, ALT_UNSUPPORTED, "%s: no split-K counter set is free for this stream (%d streams hold one; sets "
                                            "that captured graphs use are never released)", k.name, kDconvSlots);
        if (e != hipSuccess) return fail(h, ALT_HIP_ERROR, "launch of %s failed: %s", k.name, hipGetErrorString(e));
        return ALT_OK;
    }
    IgemmParams p = pb.p;
    if (!applicable(pb, k, splitk, &p, &why, nullptr))
        return fail(h, ALT_UNSUPPORTED, "variant %s/splitk%d not applicable: %s", k.name, splitk, why.c_str());
    if (need > 0) {
        if (!workspace || ws_bytes < need)
            return fail(h, ALT_WORKSPACE_TOO_SMALL, "split-K needs %zu workspace bytes, got %zu", need, ws_bytes);
        p.partial = (float *)workspace;
    }
    igemm_divisors(&p);
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)(p.batch * p.splitk));
    hipError_t e = k.launch(p, grid, st);
    if (e != hipSuccess) return fail(h, ALT_HIP_ERROR, "launch of %s failed: %s", k.name, hipGetErrorString(e));
    if (splitk > 1) {
        const int64_t total = (int64_t)p.M * p.Nc * p.batch;
        unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 256 * 16);
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3(blocks), dim3(256), 0, st, p);
        ALT_CHECK_HIP(h, hipGetLastError());
    }
    return ALT_OK;
}

std::string igemm_variant_name(int variant)
{
    const auto &tab = igemm_table();
    if (variant < 0 || variant >= (int)tab.size() * kNumSplits) return "";
    char buf[96];
    std::snprintf(buf, sizeof buf, "%s_k%d", tab[variant / kNumSplits].name, kSplits[variant % kNumSplits]);
    return buf;
}

// ---- descriptor -> problem ------------------------------------------------------------

static bool fits32(int64_t v) { return v >= 0 && v <= 0x7fffffff; }

alt_status_t conv_problem(alt_handle_t h, const alt_conv_desc_t *d, const void *x, const void *w,
                          const float *bias, void *y, Problem *pb)
{
    if (!d) return fail(h, ALT_INVALID_ARG, "null descriptor");
    if (d->N < 1 || d->C < 1 || d->H < 1 || d->W < 1 || d->K < 1 || d->R < 1 || d->S < 1)
        return fail(h, ALT_INVALID_ARG, "conv2d: non-positive extent");
    if (d->stride_h < 1 || d->stride_w < 1 || d->pad_h < 0 || d->pad_w < 0 || d->dil_h < 1 || d->dil_w < 1)
        return fail(h, ALT_INVALID_ARG, "conv2d: bad stride/pad/dilation");
    if ((d->in_dtype != ALT_F32 && d->in_dtype != ALT_BF16) || (d->out_dtype != ALT_F32 && d->out_dtype != ALT_BF16))
        return fail(h, ALT_INVALID_ARG, "conv2d: bad dtype");
    if (d->epilogue & ~(ALT_EPI_BIAS | ALT_EPI_RELU)) return fail(h, ALT_INVALID_ARG, "conv2d: unknown epilogue flag");
    const int64_t OH = (d->H + 2 * d->pad_h - d->dil_h * (d->R - 1) - 1) / d->stride_h + 1;
    const int64_t OW = (d->W + 2 * d->pad_w - d->dil_w * (d->S - 1) - 1) / d->stride_w + 1;
    if (d->H + 2 * d->pad_h < d->dil_h * (d->R - 1) + 1 || d->W + 2 * d->pad_w < d->dil_w * (d->S - 1) + 1)
        return fail(h, ALT_INVALID_ARG, "conv2d: kernel larger than padded input");
    const int64_t G = d->groups > 1 ? d->groups : 1;
    if (d->groups < 0 || d->C % G || d->K % G) return fail(h, ALT_INVALID_ARG, "conv2d: groups must divide C and K");
    const int64_t Cg = d->C / G, Kg = d->K / G;
    const int64_t xs[4] = {d->N, d->C, d->H, d->W}, wsh[4] = {d->K, Cg, d->R, d->S}, ys[4] = {d->N, d->K, OH, OW};
    BoundLayout bx, bw, by;
    std::string err;
    alt_status_t s;
    if ((s = bind_layout(&d->x_layout, 4, xs, &bx, &err)) != ALT_OK) return fail(h, s, "x_layout: %s", err.c_str());
    if ((s = bind_layout(&d->w_layout, 4, wsh, &bw, &err)) != ALT_OK) return fail(h, s, "w_layout: %s", err.c_str());
    if ((s = bind_layout(&d->y_layout, 4, ys, &by, &err)) != ALT_OK) return fail(h, s, "y_layout: %s", err.c_str());
    Dim2 dx[4], dw[4], dy[4];
    if (!layout_to_dim2(bx, dx) || !layout_to_dim2(bw, dw) || !layout_to_dim2(by, dy))
        return fail(h, ALT_UNSUPPORTED, "conv2d: layouts must be separable with at most one block level per dimension");
    if (!fits32(d->N * OH * OW) || !fits32(d->C * d->R * d->S) || !fits32(d->K) || !fits32(bx.numel / d->N * 2))
        return fail(h, ALT_UNSUPPORTED, "conv2d: problem too large for 32-bit tile indices");
    std::memset(pb, 0, sizeof(*pb));
    pb->dtype = d->in_dtype;
    pb->groups = G;
    pb->depthwise = G > 1 && Cg == 1 && Kg == 1;
    IgemmParams &p = pb->p;
    p.x = x; p.w = w; p.bias = bias; p.y = y;
    p.M = (int32_t)(d->N * OH * OW); p.Nc = (int32_t)d->K; p.Kg = (int32_t)(d->C * d->R * d->S);
    p.C = (int32_t)d->C; p.H = (int32_t)d->H; p.W = (int32_t)d->W; p.R = (int32_t)d->R; p.S = (int32_t)d->S;
    p.OH = (int32_t)OH; p.OW = (int32_t)OW;
    p.stride_h = d->stride_h; p.stride_w = d->stride_w; p.pad_h = d->pad_h; p.pad_w = d->pad_w;
    p.dil_h = d->dil_h; p.dil_w = d->dil_w;
    p.batch = 1; p.splitk = 1;
    p.epilogue = d->epilogue; p.out_bf16 = d->out_dtype == ALT_BF16;
    p.xn = dx[0]; p.xc = dx[1]; p.xh = dx[2]; p.xw = dx[3];
    p.wo = dw[0]; p.wi = dw[1]; p.wr = dw[2]; p.ws = dw[3];
    p.yn = dy[0]; p.yk = dy[1]; p.yh = dy[2]; p.yw = dy[3];
    pb->x_elems = bx.numel;
    pb->w_elems = bw.numel;
    {
        const int64_t yb = by.numel * (int64_t)dtype_size(d->out_dtype);
        p.y_bytes = yb < 0x7fffffff ? (uint32_t)yb : 0;
    }
    p.x_bytes = (uint32_t)std::min<int64_t>(bx.numel * (int64_t)dtype_size(d->in_dtype), 0x7fffffff);
    p.w_bytes = (uint32_t)std::min<int64_t>(bw.numel * (int64_t)dtype_size(d->in_dtype), 0x7fffffff);
    if (G > 1 && !pb->depthwise) {
        // One group per batch entry of the implicit-GEMM kernels: the group's channels start a fixed
        // number of elements further on in each tensor, which needs whole channel blocks per group.
        auto group_step = [](const Dim2 &c, int64_t extent, int64_t per_group, int64_t *step) {
            if (c.f >= extent) { *step = per_group * c.si; return true; }
            if (per_group % c.f) return false;
            *step = per_group / c.f * c.so;
            return true;
        };
        int64_t sx, sw, sy;
        if (!group_step(p.xc, d->C, Cg, &sx) || !group_step(p.wo, d->K, Kg, &sw) || !group_step(p.yk, d->K, Kg, &sy))
            return fail(h, ALT_UNSUPPORTED, "conv2d: a channel block of a layout straddles two groups");
        p.C = (int32_t)Cg; p.Nc = (int32_t)Kg; p.Kg = (int32_t)(Cg * d->R * d->S);
        p.batch = (int32_t)G;
        p.x_bstride = sx; p.w_bstride = sw; p.y_bstride = sy;
        p.bias_bstride = (int32_t)Kg;
    }
    igemm_analyse(pb);
    return ALT_OK;
}

alt_status_t gemm_problem(alt_handle_t h, const alt_gemm_desc_t *d, const void *A, const void *B, void *C,
                          Problem *pb)
{
    if (!d) return fail(h, ALT_INVALID_ARG, "null descriptor");
    if (d->batch < 1 || d->M < 1 || d->N < 1 || d->K < 1) return fail(h, ALT_INVALID_ARG, "gemm: non-positive extent");
    if ((d->in_dtype != ALT_F32 && d->in_dtype != ALT_BF16) || (d->out_dtype != ALT_F32 && d->out_dtype != ALT_BF16))
        return fail(h, ALT_INVALID_ARG, "gemm: bad dtype");
    const int64_t as[2] = {d->M, d->K}, bs[2] = {d->K, d->N}, cs[2] = {d->M, d->N};
    BoundLayout ba, bb, bc;
    std::string err;
    alt_status_t s;
    if ((s = bind_layout(&d->a_layout, 2, as, &ba, &err)) != ALT_OK) return fail(h, s, "a_layout: %s", err.c_str());
    if ((s = bind_layout(&d->b_layout, 2, bs, &bb, &err)) != ALT_OK) return fail(h, s, "b_layout: %s", err.c_str());
    if ((s = bind_layout(&d->c_layout, 2, cs, &bc, &err)) != ALT_OK) return fail(h, s, "c_layout: %s", err.c_str());
    Dim2 da[2], db[2], dc[2];
    if (!layout_to_dim2(ba, da) || !layout_to_dim2(bb, db) || !layout_to_dim2(bc, dc))
        return fail(h, ALT_UNSUPPORTED, "gemm: layouts must be separable with at most one block level per dimension");
    if (!fits32(d->M) || !fits32(d->N) || !fits32(d->K))
        return fail(h, ALT_UNSUPPORTED, "gemm: problem too large for 32-bit tile indices");
    std::memset(pb, 0, sizeof(*pb));
    pb->dtype = d->in_dtype;
    IgemmParams &p = pb->p;
    const Dim2 one = {1, 0, 0, 0, make_fastdiv(1)};
    p.x = A; p.w = B; p.y = C; p.bias = nullptr;
    p.M = (int32_t)d->M; p.Nc = (int32_t)d->N; p.Kg = (int32_t)d->K;
    p.C = (int32_t)d->K; p.H = 1; p.W = (int32_t)d->M; p.R = 1; p.S = 1; p.OH = 1; p.OW = (int32_t)d->M;
    p.stride_h = p.stride_w = 1; p.dil_h = p.dil_w = 1;
    p.batch = (int32_t)d->batch; p.splitk = 1;
    p.out_bf16 = d->out_dtype == ALT_BF16;
    p.x_bstride = d->M * d->K; p.w_bstride = d->K * d->N; p.y_bstride = d->M * d->N;
    p.xn = one; p.xc = da[1]; p.xh = one; p.xw = da[0];
    p.wo = db[1]; p.wi = db[0]; p.wr = one; p.ws = one;
    p.yn = one; p.yk = dc[1]; p.yh = one; p.yw = dc[0];
    pb->x_elems = ba.numel;
    pb->w_elems = bb.numel;
    {
        const int64_t yb = bc.numel * (int64_t)dtype_size(d->out_dtype);
        p.y_bytes = yb < 0x7fffffff ? (uint32_t)yb : 0;
    }
    p.x_bytes = (uint32_t)std::min<int64_t>(ba.numel * (int64_t)dtype_size(d->in_dtype), 0x7fffffff);
    p.w_bytes = (uint32_t)std::min<int64_t>(bb.numel * (int64_t)dtype_size(d->in_dtype), 0x7fffffff);
    igemm_analyse(pb);
    return ALT_OK;
}

}  // namespace alt

using namespace alt;

extern "C" {

alt_status_t alt_conv2d_output_shape(const alt_conv_desc_t *d, int64_t *out)
{
    if (!d || !out) return ALT_INVALID_ARG;
    if (d->stride_h < 1 || d->stride_w < 1 || d->dil_h < 1 || d->dil_w < 1) return ALT_INVALID_ARG;
    out[0] = d->N;
    out[1] = d->K;
    out[2] = (d->H + 2 * d->pad_h - d->dil_h * (d->R - 1) - 1) / d->stride_h + 1;
    out[3] = (d->W + 2 * d->pad_w - d->dil_w * (d->S - 1) - 1) / d->stride_w + 1;
    return (out[2] < 1 || out[3] < 1) ? ALT_INVALID_ARG : ALT_OK;
}

// ---- launch memo -------------------------------------------------------------------
// Turning a descriptor into launch parameters (three layouts bound, loaders analysed,
// with variant = -1 every kernel estimated) costs far more host time than the launch
// itself, and callers repeat the same few descriptors.  The handle remembers the last
// descriptors byte for byte, with what else the result depends on: 16-byte alignment
// of the buffers, the workspace size, the tune cache's generation.

struct MemoEntry {
    std::vector<unsigned char> desc;
    unsigned sig, gen;
    size_t ws_limit;
    Problem pb;
    int variant;
    TileLaunch tile;      // a tile kernel's launch, made by the first call
};

}  // extern "C"

// The same for the calls of one alt_conv2d_multi that go out as one launch.
struct GroupEntry {
    uint64_t tag;
    std::vector<unsigned char> key;
    const GroupFamily *family;
    GroupParams g;
    int order[kGroupMax];             // the call behind each problem of the launch
    size_t ws_need[kGroupMax], x_bytes[kGroupMax], w_bytes[kGroupMax], y_bytes[kGroupMax];
    unsigned workgroups;
    size_t lds;
};

// Lists kept, the oldest replaced: 64 launches (5 KB each, and 1 KB a call for the key), and 1024 lists of the calls that go out one by one,
// which are remembered by a hash alone: one mistaken for another would run as its calls do by themselves.  (With eight places for both kinds, nine lists
// of three layers in turn were planned on every call: 38 us of host time a list, 3.2 so.)
constexpr size_t kGroupLaunches = 64, kGroupSingles = 1024;

struct alt_launch_memo {
    std::vector<MemoEntry> entries;
    std::vector<GroupEntry> groups;
    std::vector<std::pair<uint64_t, uint64_t>> singles;    // tag, hash of the key
    size_t next = 0, next_group = 0, next_single = 0;
    unsigned group_gen = 0;           // the tune cache's generation that both belong to
};

namespace alt {
void launch_memo_free(alt_handle_t h)
{
    delete h->memo;
    h->memo = nullptr;
}
}  // namespace alt

extern "C" {

static unsigned align_sig(const void *a, const void *b, const void *c, const void *d)
{
    return (unsigned)(((uintptr_t)a & 15) | (((uintptr_t)b & 15) << 4) | (((uintptr_t)c & 15) << 8) |
                      (((uintptr_t)d & 15) << 12) | ((c ? 1u : 0u) << 16));
}

static MemoEntry *memo_find(alt_handle_t h, const void *desc, size_t bytes, unsigned sig, size_t ws_limit)
{
    if (!h->memo) return nullptr;
    for (MemoEntry &e : h->memo->entries)
        if (e.sig == sig && e.gen == h->cache_gen && e.ws_limit == ws_limit && e.desc.size() == bytes &&
            std::memcmp(e.desc.data(), desc, bytes) == 0)
            return &e;
    return nullptr;
}

static void memo_store(alt_handle_t h, const void *desc, size_t bytes, unsigned sig, size_t ws_limit, const Problem &pb,
                       int variant)
{
    constexpr size_t kMemoEntries = 32;
    if (!h->memo) h->memo = new alt_launch_memo();
    MemoEntry e;
    e.desc.assign((const unsigned char *)desc, (const unsigned char *)desc + bytes);
    e.sig = sig; e.gen = h->cache_gen; e.ws_limit = ws_limit; e.pb = pb; e.variant = variant;
    auto &v = h->memo->entries;
    if (v.size() < kMemoEntries) v.push_back(std::move(e));
    else { v[h->memo->next] = std::move(e); h->memo->next = (h->memo->next + 1) % kMemoEntries; }
}

// The tuned variant of a key, -1 if there is none that runs this problem.
static int tuned_variant(alt_handle_t h, const Problem &pb, const std::string &key, size_t ws_limit)
{
    auto it = h->cache.find(key);
    if (it == h->cache.end()) return -1;
    // a cached entry is only trusted if it still applies (pointers may be aligned differently)
    const auto &tab = igemm_table();
    const int v = it->second.variant;
    return v >= 0 && v < (int)tab.size() * kNumSplits &&
                   igemm_applicable(pb, tab[v / kNumSplits], kSplits[v % kNumSplits], nullptr) &&
                   igemm_workspace(pb, kSplits[v % kNumSplits]) <= ws_limit ? v : -1;
}

// variant = -1: the cached tuned variant if it applies and its split-K partial
// sums fit the workspace the caller brought, else the best-estimate variant
// that fits.
static int pick_variant(alt_handle_t h, const Problem &pb, int requested, const std::string &key, size_t ws_limit)
{
    if (requested >= 0) return requested;
    const int v = tuned_variant(h, pb, key, ws_limit);
    return v >= 0 ? v : igemm_default_variant(pb, ws_limit);
}

// Runs variant v.  Where it was the library's own choice and no set of arrival counters is free for its slices (more streams than
// sets, under capture), the best variant that needs none takes its place.
static alt_status_t run_chosen(alt_handle_t h, const Problem &pb, int v, bool own_choice, void *workspace, size_t ws_bytes,
                               hipStream_t st, TileLaunch *kept = nullptr)
{
    bool no_counters = false;
    const alt_status_t s = igemm_run(h, pb, v, workspace, ws_bytes, st, &no_counters, kept);
    if (!no_counters || !own_choice) return s;
    v = igemm_default_variant(pb, workspace ? ws_bytes : 0, false);
    return v < 0 ? s : igemm_run(h, pb, v, workspace, ws_bytes, st);
}

static alt_status_t conv2d_impl(alt_handle_t h, const alt_conv_desc_t *d, const void *x, const void *w, const float *bias,
                                const void *addend, void *y, void *workspace, size_t ws_bytes, void *stream, const char *who)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !x || !w || !y) return fail(h, ALT_INVALID_ARG, "%s: null argument", who);
    if ((d->epilogue & ALT_EPI_BIAS) && !bias) return fail(h, ALT_INVALID_ARG, "%s: bias flag without bias", who);
    const size_t ws_limit = workspace ? ws_bytes : 0;
    const unsigned sig = align_sig(x, w, bias, y) | (addend ? 1u << 17 : 0u) | ((unsigned)((uintptr_t)addend & 15) << 18);
    if (MemoEntry *m = memo_find(h, d, sizeof *d, sig, ws_limit)) {
        m->pb.p.x = x; m->pb.p.w = w; m->pb.p.bias = bias; m->pb.p.y = y; m->pb.p.addend = addend;
        if (m->pb.depthwise) return depthwise_run(h, m->pb, d->N, d->C, (hipStream_t)stream);
        return run_chosen(h, m->pb, m->variant, d->variant < 0, workspace, ws_bytes, (hipStream_t)stream, &m->tile);
    }
    Problem pb;
    alt_status_t s = conv_problem(h, d, x, w, bias, y, &pb);
    if (s != ALT_OK) return s;
    if (addend) {
        if (pb.depthwise || pb.groups > 1) return fail(h, ALT_UNSUPPORTED, "%s: no fused sum for grouped convolutions", who);
        if ((uintptr_t)addend % 16) return fail(h, ALT_INVALID_ARG, "%s: the addend must be 16-byte aligned", who);
        pb.p.addend = addend;
    }
    if (pb.depthwise) {
        memo_store(h, d, sizeof *d, sig, ws_limit, pb, -1);
        return depthwise_run(h, pb, d->N, d->C, (hipStream_t)stream);
    }
    // (a tuned choice for the same problem without the sum is a good one with it, if it applies)
    int v = pick_variant(h, pb, d->variant, d->variant >= 0 ? std::string() : conv_key(h, d), ws_limit);
    if (v < 0) return fail(h, ALT_UNSUPPORTED, "%s: no kernel variant applies", who);
    memo_store(h, d, sizeof *d, sig, ws_limit, pb, v);
    return run_chosen(h, pb, v, d->variant < 0, workspace, ws_bytes, (hipStream_t)stream);
}

}  // extern "C"

namespace alt {
// (a depth-unfolded copy of the input costs T times its traffic, a merged filter all products of the common window, 9/4 of those
// that are not zeros for 4x4 at stride 2 and 27/8 for 4x4x4, and its result one more pass into place: 128 channels, 3x3x3 on
// 8x28x28 at batch 2 took 48 us that way and 16.7 here, T3D 128 -> 64, 4x4x4 at stride 2 on the same volume 128 us and 21; so these
// kernels run whatever they cover, unless the problem's 2-D form has been tuned to a variant of its own)
static bool taps_problem(alt_handle_t h, const TapsCall &c, const void *x, const void *w, const float *bias, void *y, int64_t ws_2d, Problem *out)
{
    BoundLayout bx, by;
    Dim2 dx[4], dy[4];
    std::string err;
    Problem &pb = *out;
    if (!(conv_problem(h, &c.f, x, w, bias, y, &pb) == ALT_OK && pb.groups <= 1 &&
          bind_layout(&c.f.x_layout, 4, c.xs, &bx, &err) == ALT_OK && bind_layout(&c.f.y_layout, 4, c.ys, &by, &err) == ALT_OK &&
          layout_to_dim2(bx, dx) && layout_to_dim2(by, dy)))
        return false;
    // (tuning an operator is tuning its 2-D problem: the winner runs, by the copying path)
    if (ws_2d >= 0 && tuned_variant(h, pb, conv_key(h, &c.f), (size_t)ws_2d) >= 0) return false;
    const int64_t es = (int64_t)dtype_size(c.f.in_dtype), os = (int64_t)dtype_size(c.f.out_dtype);
    IgemmParams &p = pb.p;
    pb.v = c.v;
    p.xn = dx[0]; p.xc = dx[1]; p.xh = dx[2]; p.xw = dx[3];
    p.yn = dy[0]; p.yk = dy[1]; p.yh = dy[2]; p.yw = dy[3];
    p.C = (int32_t)c.C;
    p.Nc = (int32_t)c.K;
    p.batch = c.v.sd * c.v.sh * c.v.sw;
    pb.x_elems = bx.numel;
    pb.w_elems = (int64_t)c.K * c.f.C * c.f.R * c.f.S;
    p.x_bstride = 0; p.w_bstride = pb.w_elems; p.y_bstride = 0;
    p.x_bytes = (uint32_t)std::min<int64_t>(pb.x_elems * es, 0x7fffffff);
    p.w_bytes = (uint32_t)std::min<int64_t>(pb.w_elems * es, 0x7fffffff);
    p.y_bytes = by.numel * 4 < 0x7fffffff ? (uint32_t)(by.numel * os) : 0;
    return true;
}

size_t taps_workspace(alt_handle_t h, const TapsCall &c)
{
    Problem pb;
    if (c.f.variant >= 0 || !taps_problem(h, c, nullptr, nullptr, nullptr, nullptr, INT64_MAX, &pb)) return 0;
    const int v = igemm_default_variant(pb, (size_t)-1);
    return v < 0 ? 0 : igemm_workspace(pb, kSplits[v % kNumSplits]);
}

alt_status_t taps_run(alt_handle_t h, const TapsCall &c, const void *x, const void *w, const float *bias, void *y, void *workspace,
                      size_t ws_bytes, int64_t ws_2d, hipStream_t st, bool *done)
{
    *done = false;
    if (c.f.variant >= 0 || !x || !w || !y || ((c.f.epilogue & ALT_EPI_BIAS) && !bias)) return ALT_OK;
    const size_t ws_limit = workspace ? ws_bytes : 0;
    const unsigned sig = align_sig(x, w, bias, y) | 1u << 31;
    if (MemoEntry *m = memo_find(h, &c, sizeof c, sig, ws_limit)) {
        if (m->variant < 0) return ALT_OK;
        *done = true;
        m->pb.p.x = x; m->pb.p.w = w; m->pb.p.bias = bias; m->pb.p.y = y;
        return run_chosen(h, m->pb, m->variant, true, workspace, ws_bytes, st, &m->tile);
    }
    Problem pb;
    const int v = taps_problem(h, c, x, w, bias, y, ws_2d, &pb) ? igemm_default_variant(pb, ws_limit) : -1;
    memo_store(h, &c, sizeof c, sig, ws_limit, pb, v);
    if (v < 0) return ALT_OK;
    *done = true;
    return run_chosen(h, pb, v, true, workspace, ws_bytes, st);
}
}  // namespace alt

extern "C" {

alt_status_t alt_conv2d(alt_handle_t h, const alt_conv_desc_t *d, const void *x, const void *w, const float *bias,
                        void *y, void *workspace, size_t ws_bytes, void *stream)
{
    return conv2d_impl(h, d, x, w, bias, nullptr, y, workspace, ws_bytes, stream, "alt_conv2d");
}

// ---- alt_conv2d without a caller's workspace ---------------------------------------------
// The split-K partial tiles of alt_conv2d_static live in this array instead of a workspace
// the caller brings.  The name below is a host-side stand-in: the array's device address is
// looked up once per device (static_scratch) and that pointer is what kernels get.
constexpr size_t kStaticScratchBytes = ALT_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static void *g_scratch_ptr[16];
static std::mutex g_scratch_mutex;

}  // extern "C"

namespace alt {
// Device address of `scratch` on the current device; first use on a device asks the runtime.
hipError_t static_scratch(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 16) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
}  // namespace alt

extern "C" {

alt_status_t alt_conv2d_static(alt_handle_t h, const alt_conv_desc_t *d, const void *x, const void *w, const float *bias,
                               void *y, void *stream)
{
    if (!h) return ALT_INVALID_ARG;
    if (!h->has_gpu) return fail(h, ALT_HIP_ERROR, "no GPU device available");
    void *ws = nullptr;
    hipError_t e = static_scratch(&ws);
    if (e != hipSuccess) return fail(h, ALT_HIP_ERROR, "alt_conv2d_static: no address for the static workspace: %s", hipGetErrorString(e));
    // (an explicitly requested variant whose partial tiles exceed the array fails in igemm_run with
    // ALT_WORKSPACE_TOO_SMALL and the two sizes; variant = -1 only picks variants that fit)
    return conv2d_impl(h, d, x, w, bias, nullptr, y, ws, kStaticScratchBytes, stream, "alt_conv2d_static");
}

alt_status_t alt_conv2d_add(alt_handle_t h, const alt_conv_desc_t *d, const void *x, const void *w, const float *bias,
                            const void *addend, void *y, void *workspace, size_t ws_bytes, void *stream)
{
    if (h && !addend) return fail(h, ALT_INVALID_ARG, "alt_conv2d_add: null addend");
    return conv2d_impl(h, d, x, w, bias, addend, y, workspace, ws_bytes, stream, "alt_conv2d_add");
}

// ---- several convolutions in one launch (group.h) ------------------------------------------------

// A tile that runs one of the calls' problems.
struct GroupPick {
    double alone, beside;             // microseconds of a workgroup (TileClocks)
    double workgroups;
    size_t lds;
    int tile, splitk, body;
};

// Microseconds of one launch of them: a workgroup takes of its compute unit what it takes beside others and a share of what it waits
// alone, and the last ones to start run half their length by themselves.  Within 15 % of 51 measured launches of 8 to 420 us; those in fp32 of
// 20 us and less take up to 30 % longer (slices).
static double group_us(const GroupPick *const *pick, int n, int threads)
{
    double workgroups = 0, longest = 0, busy = 0;
    size_t lds = 1;
    for (int i = 0; i < n; ++i) {
        workgroups += pick[i]->workgroups;
        lds = std::max(lds, pick[i]->lds);
        longest = std::max(longest, pick[i]->alone);
    }
    const double per_cu = std::max(1.0, std::min({std::floor(160.0 * 1024 / lds), 2048.0 / threads, std::ceil(workgroups / 256.0)}));
    for (int i = 0; i < n; ++i) busy += pick[i]->workgroups * (pick[i]->beside + (pick[i]->alone - pick[i]->beside) / per_cu);
    return 2.5 + std::max(longest, busy / 256.0 + 0.5 * longest);
}

// The launch of the calls' problems, or false where launches of their own are better or needed.
static bool group_plan(alt_handle_t h, const alt_conv_call_t *calls, int n, GroupEntry *e)
{
    const auto &tab = igemm_table();
    Problem pb[kGroupMax];
    int own[kGroupMax];               // the variant that runs a call by itself, -1: not known
    size_t limit[kGroupMax];
    unsigned sig[kGroupMax];
    for (int i = 0; i < n; ++i) {
        const alt_conv_call_t &c = calls[i];
        limit[i] = c.workspace ? c.ws_bytes : 0;
        sig[i] = align_sig(c.x, c.w, c.bias, c.y);
        own[i] = -1;
        if (const MemoEntry *m = memo_find(h, c.d, sizeof *c.d, sig[i], limit[i])) {
            pb[i] = m->pb;
            pb[i].p.x = c.x; pb[i].p.w = c.w; pb[i].p.bias = c.bias; pb[i].p.y = c.y;
            own[i] = m->variant;
        } else if (conv_problem(h, c.d, c.x, c.w, c.bias, c.y, &pb[i]) != ALT_OK) {
            return false;
        }
        // (a tuned kernel runs)
        if (pb[i].depthwise || pb[i].groups > 1 || pb[i].dtype != pb[0].dtype || tuned_variant(h, pb[i], conv_key(h, c.d), limit[i]) >= 0) return false;
    }
    const GroupFamily &f = pb[0].dtype == ALT_F32 ? group_f32() : pb[0].p.xc.si == 1 ? group_slab() : group_planar();
    std::vector<GroupPick> all[kGroupMax];
    for (int i = 0; i < n; ++i) {
        IgemmParams p = pb[i].p;
        for (int t = 0; t < f.ntiles; ++t) {
            const IgemmLaunch &k = f.tiles[t].k;
            for (int si = 0; si < (k.stream >= 2 ? 1 : kNumSplits); ++si) {
                size_t lds = 0;
                DconvParams d;
                double family;
                TileClocks c;
                if (igemm_workspace(pb[i], kSplits[si]) > limit[i] || !applicable(pb[i], k, kSplits[si], &p, nullptr, &lds) ||
                    !dconv_setup(pb[i], k, kSplits[si], &d, nullptr, nullptr))
                    continue;
                const int body = f.tiles[t].body(d);
                if (body < 0) continue;
                direct_estimate_us(pb[i], k, p, lds, &family, &c);
                all[i].push_back({c.alone / 2200.0, c.beside / 2200.0, (double)d.tiles_m * d.tiles_n * d.splitk, lds, t, kSplits[si], body});
            }
        }
        if (all[i].empty()) return false;
    }
    // What the calls take one by one.  Where that is the answer, the choices made for it are the calls' own.
    auto singly = [&] {
        for (int i = 0; i < n; ++i)
            if (own[i] >= 0 && !memo_find(h, calls[i].d, sizeof *calls[i].d, sig[i], limit[i]))
                memo_store(h, calls[i].d, sizeof *calls[i].d, sig[i], limit[i], pb[i], own[i]);
        return false;
    };
    double one_by_one = 0;
    for (int i = 0; i < n; ++i) {
        if (own[i] < 0) own[i] = igemm_default_variant(pb[i], limit[i]);
        // (the register-staged kernels' estimate is no time)
        if (own[i] < 0 || !tab[own[i] / kNumSplits].launch_direct) return singly();
        IgemmParams p = pb[i].p;
        size_t lds = 0;
        double family;
        if (!applicable(pb[i], tab[own[i] / kNumSplits], kSplits[own[i] % kNumSplits], &p, nullptr, &lds)) return singly();
        one_by_one += direct_estimate_us(pb[i], tab[own[i] / kNumSplits], p, lds, &family);
    }
    // For every bound on a workgroup's length, and on its LDS for one to four on a compute unit: of each problem the tile of least work.
    const GroupPick *best[kGroupMax];
    double best_us = 1e300;
    for (const auto &a : all)
        for (const GroupPick &bound : a)
            for (size_t room : {160 * 1024, 80 * 1024, 53 * 1024, 40 * 1024}) {
                const GroupPick *pick[kGroupMax];
                bool fits = true;
                for (int i = 0; i < n && fits; ++i) {
                    pick[i] = nullptr;
                    for (const GroupPick &c : all[i])
                        if (c.alone <= bound.alone && c.lds <= room &&
                            (!pick[i] || c.workgroups * c.beside < pick[i]->workgroups * pick[i]->beside)) pick[i] = &c;
                    fits = pick[i] != nullptr;
                }
                const double us = fits ? group_us(pick, n, f.threads) : 1e300;
                if (us < best_us) { best_us = us; std::copy(pick, pick + n, best); }
            }
    // (launches of their own have all tiles to choose from and win for large layers)
    if (best_us > f.line * one_by_one) return singly();
    // the longest workgroups first
    for (int i = 0; i < n; ++i) e->order[i] = i;
    std::sort(e->order, e->order + n, [&](int a, int b) { return best[a]->alone > best[b]->alone; });
    std::memset(&e->g, 0, sizeof e->g);
    e->g.n = n;
    e->lds = 0;
    int64_t at = 0, sliced = 0;
    for (int j = 0; j < n; ++j) {
        const int i = e->order[j];
        DconvParams &d = e->g.p[j];
        if (at > 0x3fffffff || !dconv_setup(pb[i], f.tiles[best[i]->tile].k, best[i]->splitk, &d, nullptr, nullptr)) return singly();
        e->g.first[j] = (int32_t)at;
        e->g.body[j] = best[i]->body;
        const int64_t tiles = (int64_t)d.tiles_m * d.tiles_n;
        at += (tiles * d.splitk + 7) / 8 * 8;
        sliced += d.splitk > 1 ? tiles : 0;
        e->lds = std::max(e->lds, best[i]->lds);
        e->ws_need[i] = igemm_workspace(pb[i], d.splitk);
        e->x_bytes[i] = d.x_bytes; e->w_bytes[i] = d.w_bytes; e->y_bytes[i] = d.y_bytes;
    }
    if (at > 0x7fffffff || sliced > kDconvMaxTiles) return singly();
    e->workgroups = (unsigned)at;
    e->family = &f;
    return true;
}

// The list's kept launch, or the one planned for it now; null: its calls go out one by one.  *kept: the answer was there.
static GroupEntry *group_entry(alt_handle_t h, const alt_conv_call_t *calls, int n, bool *kept)
{
    // the descriptors without their layouts' primitives, which no convolution reads
    constexpr size_t kPlain = offsetof(alt_conv_desc_t, x_layout), kLayout = offsetof(alt_layout_t, prims);
    unsigned char key[kGroupMax * (kPlain + 3 * kLayout + sizeof(alt_conv_desc_t::groups) + sizeof(uint64_t) + sizeof(size_t))];
    size_t len = 0;
    auto put = [&](const void *p, size_t bytes) { std::memcpy(key + len, p, bytes); len += bytes; };
    uint64_t tag = (uint64_t)n;       // of what differs most often
    auto mix = [](uint64_t t, uint64_t v) { t = (t ^ v) * 0x9e3779b97f4a7c15ull; return t ^ (t >> 29); };
    *kept = true;
    for (int i = 0; i < n; ++i) {
        const alt_conv_call_t &c = calls[i];
        if (!c.d || !c.x || !c.w || !c.y || ((c.d->epilogue & ALT_EPI_BIAS) && !c.bias)) return nullptr;
        if (c.d->variant >= 0) return nullptr;
        const uint64_t sig = align_sig(c.x, c.w, c.bias, c.y);
        const size_t limit = c.workspace ? c.ws_bytes : 0;
        put(c.d, kPlain);
        for (const alt_layout_t *l : {&c.d->x_layout, &c.d->w_layout, &c.d->y_layout}) put(l, kLayout);
        put(&c.d->groups, sizeof c.d->groups);
        put(&sig, sizeof sig);
        put(&limit, sizeof limit);
        tag = mix(mix(tag, (uint64_t)c.d->N << 32 ^ (uint64_t)c.d->H << 16 ^ (uint64_t)c.d->W), (uint64_t)c.d->C << 32 ^ (uint64_t)c.d->K << 8 ^ (uint64_t)c.d->R);
        tag = mix(mix(tag, sig), limit);
    }
    if (!h->memo) h->memo = new alt_launch_memo();
    alt_launch_memo &memo = *h->memo;
    if (memo.group_gen != h->cache_gen) {
        memo.groups.clear();
        memo.singles.clear();
        memo.next_group = memo.next_single = 0;
        memo.group_gen = h->cache_gen;
    }
    for (GroupEntry &c : memo.groups)
        if (c.tag == tag && c.key.size() == len && std::memcmp(c.key.data(), key, len) == 0) return &c;
    uint64_t hash = 0;                // of the whole key, where it is asked for
    auto whole = [&] {
        if (hash) return hash;
        uint64_t lane[4] = {1, 2, 3, 4}, word[4] = {0, 0, 0, 0};
        for (size_t at = 0; at < len; at += sizeof word) {
            std::memcpy(word, key + at, std::min(sizeof word, len - at));
            for (int l = 0; l < 4; ++l) lane[l] = mix(lane[l], word[l]);
        }
        for (uint64_t l : lane) hash = mix(hash, l);
        return hash;
    };
    for (const auto &c : memo.singles)
        if (c.first == tag && c.second == whole()) return nullptr;
    *kept = false;
    GroupEntry e;
    if (!group_plan(h, calls, n, &e)) {
        const std::pair<uint64_t, uint64_t> single(tag, whole());
        if (memo.singles.size() < kGroupSingles) memo.singles.push_back(single);
        else { memo.singles[memo.next_single] = single; memo.next_single = (memo.next_single + 1) % kGroupSingles; }
        return nullptr;
    }
    e.tag = tag;
    e.key.assign(key, key + len);
    if (memo.groups.size() < kGroupLaunches) { memo.groups.push_back(std::move(e)); return &memo.groups.back(); }
    GroupEntry &place = memo.groups[memo.next_group];
    memo.next_group = (memo.next_group + 1) % kGroupLaunches;
    place = std::move(e);
    return &place;
}

// (a call that writes what another reads or writes has to wait for it, as on the stream)
static bool calls_meet(const GroupEntry &e, const alt_conv_call_t *calls, int n)
{
    struct Range { uintptr_t at; size_t bytes; };
    auto meet = [](Range a, Range b) { return a.at < b.at + b.bytes && b.at < a.at + a.bytes; };
    for (int i = 0; i < n; ++i) {
        const alt_conv_call_t &c = calls[i];
        const Range out[2] = {{(uintptr_t)c.y, e.y_bytes[i]}, {(uintptr_t)c.workspace, e.ws_need[i]}};
        for (int j = 0; j < n; ++j) {
            if (j == i) continue;
            const alt_conv_call_t &o = calls[j];
            const Range other[5] = {{(uintptr_t)o.x, e.x_bytes[j]}, {(uintptr_t)o.w, e.w_bytes[j]},
                                    {(uintptr_t)o.bias, o.bias ? (size_t)o.d->K * 4 : 0}, {(uintptr_t)o.y, e.y_bytes[j]},
                                    {(uintptr_t)o.workspace, e.ws_need[j]}};
            for (const Range &a : out)
                for (const Range &b : other)
                    if (a.bytes && b.bytes && meet(a, b)) return true;
        }
    }
    return false;
}

// The calls from the first on that may go out together: on one stream, as many as a launch takes.
static int calls_together(const alt_conv_call_t *calls, int n)
{
    int m = 1;
    while (m < kGroupMax && m < n && calls[m].stream == calls[0].stream) ++m;
    return m;
}

// Issues the calls, all on one stream, as one launch and says so in *done, or leaves them alone.
static alt_status_t multi_as_one(alt_handle_t h, const alt_conv_call_t *calls, int n, bool *done)
{
    *done = false;
    if (n < 2 || !h->has_gpu) return ALT_OK;
    bool kept;
    GroupEntry *e = group_entry(h, calls, n, &kept);
    if (!e || calls_meet(*e, calls, n)) return ALT_OK;
    for (int j = 0; j < n; ++j) {
        const alt_conv_call_t &c = calls[e->order[j]];
        DconvParams &p = e->g.p[j];
        p.x = c.x; p.w = c.w; p.bias = c.bias; p.y = c.y; p.partial = (float *)c.workspace;
    }
    const hipError_t r = group_run(*e->family, &e->g, e->workgroups, e->lds, (hipStream_t)calls[0].stream);
    if (r == hipErrorNotReady) return ALT_OK;
    *done = true;
    if (r != hipSuccess) return fail(h, ALT_HIP_ERROR, "launch of %d convolutions failed: %s", n, hipGetErrorString(r));
    return ALT_OK;
}

alt_status_t alt_conv2d_multi(alt_handle_t h, const alt_conv_call_t *calls, int32_t n)
{
    if (!h) return ALT_INVALID_ARG;
    if (n < 0 || (n > 0 && !calls)) return fail(h, ALT_INVALID_ARG, "alt_conv2d_multi: bad call list");
    for (int32_t i = 0; i < n;) {
        const int m = calls_together(calls + i, n - i);
        bool done = false;
        alt_status_t s = multi_as_one(h, calls + i, m, &done);
        for (int32_t j = i; j < i + m && !done; ++j) {
            const alt_conv_call_t &c = calls[j];
            s = alt_conv2d(h, c.d, c.x, c.w, c.bias, c.y, c.workspace, c.ws_bytes, c.stream);
            if (s != ALT_OK) return s;
        }
        if (s != ALT_OK) return s;
        i += m;
    }
    return ALT_OK;
}

alt_status_t alt_conv2d_multi_plan(alt_handle_t h, const alt_conv_call_t *calls, int32_t n, alt_multi_plan_t *out)
{
    if (!h) return ALT_INVALID_ARG;
    if (n < 0 || (n > 0 && (!calls || !out))) return fail(h, ALT_INVALID_ARG, "alt_conv2d_multi_plan: bad call list");
    int32_t launch = 0;
    for (int32_t i = 0; i < n;) {
        const int m = calls_together(calls + i, n - i);
        bool kept = false;
        const GroupEntry *e = m > 1 ? group_entry(h, calls + i, m, &kept) : nullptr;
        if (e && calls_meet(*e, calls + i, m)) e = nullptr;
        for (int j = 0; j < m; ++j) out[i + j] = alt_multi_plan_t{e ? launch : launch + j, e ? e->family->code : 0, -1, 0, kept};
        for (int j = 0; j < m && e; ++j) {
            out[i + e->order[j]].body = e->g.body[j];
            out[i + e->order[j]].slices = e->g.p[j].splitk;
        }
        launch += e ? 1 : m;
        i += m;
    }
    return ALT_OK;
}

alt_status_t alt_conv2d_workspace_size(alt_handle_t h, const alt_conv_desc_t *d, size_t *bytes)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !bytes) return fail(h, ALT_INVALID_ARG, "null argument");
    Problem pb;
    // alignment of real pointers is unknown here: assume 16-byte aligned buffers
    alt_status_t s = conv_problem(h, d, (void *)16, (void *)16, nullptr, (void *)16, &pb);
    if (s != ALT_OK) return s;
    if (pb.depthwise) { *bytes = 0; return ALT_OK; }
    int v = pick_variant(h, pb, d->variant, conv_key(h, d), (size_t)-1);
    if (v < 0) return fail(h, ALT_UNSUPPORTED, "no kernel variant applies");
    *bytes = igemm_workspace(pb, kSplits[v % kNumSplits]);
    return ALT_OK;
}

alt_status_t alt_conv2d_variant_count(alt_handle_t h, const alt_conv_desc_t *d, int *count)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !count) return fail(h, ALT_INVALID_ARG, "null argument");
    *count = igemm_variant_count();
    return ALT_OK;
}

alt_status_t alt_conv2d_variant_name(alt_handle_t h, const alt_conv_desc_t *d, int variant, char *buf, size_t buflen)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !buf || buflen == 0) return fail(h, ALT_INVALID_ARG, "null argument");
    Problem pb;
    alt_status_t s = conv_problem(h, d, (void *)16, (void *)16, nullptr, (void *)16, &pb);
    if (s != ALT_OK) return s;
    if (pb.depthwise) return fail(h, ALT_UNSUPPORTED, "depth-wise convolutions have no kernel variants");
    if (variant < 0) {                               // the variant alt_conv2d would run with variant = -1 and any workspace
        variant = pick_variant(h, pb, -1, conv_key(h, d), (size_t)-1);
        if (variant < 0) return fail(h, ALT_UNSUPPORTED, "no kernel variant applies");
    }
    std::string n = igemm_variant_name(variant);
    if (n.empty()) return fail(h, ALT_INVALID_ARG, "variant %d out of range", variant);
    std::snprintf(buf, buflen, "%s", n.c_str());
    std::string why;
    const auto &tab = igemm_table();
    if (!igemm_applicable(pb, tab[variant / kNumSplits], kSplits[variant % kNumSplits], &why))
        return fail(h, ALT_UNSUPPORTED, "%s: %s", n.c_str(), why.c_str());
    return ALT_OK;
}

alt_status_t alt_pack_weights(alt_handle_t h, const alt_conv_desc_t *d, const void *w_oihw, void *w_packed, void *stream)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !w_oihw || !w_packed) return fail(h, ALT_INVALID_ARG, "alt_pack_weights: null argument");
    const int64_t G = d->groups > 1 ? d->groups : 1;
    if (d->C % G) return fail(h, ALT_INVALID_ARG, "alt_pack_weights: groups must divide C");
    const int64_t wsh[4] = {d->K, d->C / G, d->R, d->S};
    alt_layout_t plain;
    alt_layout_parse("OIHW->OIHW", &plain);
    BoundLayout bs, bd;
    std::string err;
    alt_status_t s;
    if ((s = bind_layout(&plain, 4, wsh, &bs, &err)) != ALT_OK) return fail(h, s, "%s", err.c_str());
    if ((s = bind_layout(&d->w_layout, 4, wsh, &bd, &err)) != ALT_OK) return fail(h, s, "w_layout: %s", err.c_str());
    return transform_bound(h, (int)dtype_size(d->in_dtype), bs, w_oihw, bd, w_packed, (hipStream_t)stream);
}

alt_status_t alt_gemm(alt_handle_t h, const alt_gemm_desc_t *d, const void *A, const void *B, void *C,
                      void *workspace, size_t ws_bytes, void *stream)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !A || !B || !C) return fail(h, ALT_INVALID_ARG, "alt_gemm: null argument");
    const size_t ws_limit = workspace ? ws_bytes : 0;
    const unsigned sig = align_sig(A, B, nullptr, C);
    if (MemoEntry *m = memo_find(h, d, sizeof *d, sig, ws_limit)) {
        m->pb.p.x = A; m->pb.p.w = B; m->pb.p.y = C;
        return run_chosen(h, m->pb, m->variant, d->variant < 0, workspace, ws_bytes, (hipStream_t)stream, &m->tile);
    }
    Problem pb;
    alt_status_t s = gemm_problem(h, d, A, B, C, &pb);
    if (s != ALT_OK) return s;
    int v = pick_variant(h, pb, d->variant, d->variant >= 0 ? std::string() : gemm_key(h, d), ws_limit);
    if (v < 0) return fail(h, ALT_UNSUPPORTED, "alt_gemm: no kernel variant applies");
    memo_store(h, d, sizeof *d, sig, ws_limit, pb, v);
    return run_chosen(h, pb, v, d->variant < 0, workspace, ws_bytes, (hipStream_t)stream);
}

alt_status_t alt_splitk_status(alt_handle_t h, alt_splitk_status_t *out)
{
    if (!h) return ALT_INVALID_ARG;
    if (!out) return fail(h, ALT_INVALID_ARG, "alt_splitk_status: null argument");
    std::memset(out, 0, sizeof *out);
    if (!h->has_gpu) return fail(h, ALT_HIP_ERROR, "no GPU device available");
    int bound = 0, nonzero = 0;
    dconv_splitk_state(&bound, &nonzero);
    out->streams_bound = bound; out->counters_nonzero = nonzero;
    out->max_streams = kDconvSlots;
    if (nonzero < 0) return fail(h, ALT_HIP_ERROR, "alt_splitk_status: could not read the counters");
    return ALT_OK;
}

alt_status_t alt_gemm_workspace_size(alt_handle_t h, const alt_gemm_desc_t *d, size_t *bytes)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !bytes) return fail(h, ALT_INVALID_ARG, "null argument");
    Problem pb;
    alt_status_t s = gemm_problem(h, d, (void *)16, (void *)16, (void *)16, &pb);
    if (s != ALT_OK) return s;
    int v = pick_variant(h, pb, d->variant, gemm_key(h, d), (size_t)-1);
    if (v < 0) return fail(h, ALT_UNSUPPORTED, "no kernel variant applies");
    *bytes = igemm_workspace(pb, kSplits[v % kNumSplits]);
    return ALT_OK;
}

alt_status_t alt_gemm_variant_count(alt_handle_t h, const alt_gemm_desc_t *d, int *count)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !count) return fail(h, ALT_INVALID_ARG, "null argument");
    *count = igemm_variant_count();
    return ALT_OK;
}

alt_status_t alt_gemm_variant_name(alt_handle_t h, const alt_gemm_desc_t *d, int variant, char *buf, size_t buflen)
{
    if (!h) return ALT_INVALID_ARG;
    if (!d || !buf || buflen == 0) return fail(h, ALT_INVALID_ARG, "null argument");
    Problem pb;
    alt_status_t s = gemm_problem(h, d, (void *)16, (void *)16, (void *)16, &pb);
    if (s != ALT_OK) return s;
    if (variant < 0) {                               // the variant alt_gemm would run with variant = -1 and any workspace
        variant = pick_variant(h, pb, -1, gemm_key(h, d), (size_t)-1);
        if (variant < 0) return fail(h, ALT_UNSUPPORTED, "no kernel variant applies");
    }
    std::string n = igemm_variant_name(variant);
    if (n.empty()) return fail(h, ALT_INVALID_ARG, "variant %d out of range", variant);
    std::snprintf(buf, buflen, "%s", n.c_str());
    std::string why;
    const auto &tab = igemm_table();
    if (!igemm_applicable(pb, tab[variant / kNumSplits], kSplits[variant % kNumSplits], &why))
        return fail(h, ALT_UNSUPPORTED, "%s: %s", n.c_str(), why.c_str());
    return ALT_OK;
}

}  // extern "C"
