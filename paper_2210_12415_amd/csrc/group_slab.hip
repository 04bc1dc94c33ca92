// Convolutions in one launch: bf16, NHWC, 3x3 and 1x1 filters.
#include "group.h"

namespace alt {
namespace {

// Tiles of 64 and 128 rows by four waves: what small batches have enough of, with room for two and three workgroups on a compute unit.
struct Slab {
    static constexpr int kThreads = 256, kWaves = 2;
    static __device__ __forceinline__ void run(int body, const DconvParams &p, int id)
    {
        const int tiles = p.tiles_m * p.tiles_n;
        switch (body) {
        case 0: dslab_body<64, 64, 2, 2, 1, 32, 3, kSlabLoads[0]>(p, tiles, id, 0); break;
        case 1: dslab_body<64, 64, 2, 2, 1, 32, 3, kSlabLoads[1]>(p, tiles, id, 0); break;
        case 2: dslab_body<64, 64, 2, 2, 1, 32, 3, kSlabLoads[2]>(p, tiles, id, 0); break;
        case 3: dslab_body<64, 32, 1, 1, 4, 32, 3, kSlabLoads[1]>(p, tiles, id, 0); break;
        case 4: dslab_body<64, 32, 1, 1, 4, 32, 3, kSlabLoads[2]>(p, tiles, id, 0); break;
        case 5: dslab_body<128, 64, 2, 2, 1, 32, 3, kSlabLoads[1]>(p, tiles, id, 0); break;
        case 6: dslab_body<128, 64, 2, 2, 1, 32, 3, kSlabLoads[2]>(p, tiles, id, 0); break;
        case 7: dstream_body<64, 64, 2, 2, 1, 3, 64, false, kTapsOne>(p, id, 0); break;
        default: dstream_body<128, 64, 4, 1, 1, 3, 64, false, kTapsOne>(p, id, 0); break;
        }
    }
};

constexpr IgemmLaunch slab(int BM, int BN, int wgm, int wgn, int kw)
{
    return IgemmLaunch{"", ALT_BF16, BM, BN, 32, LOAD_VEC, LOAD_VEC, 2, 1, 0, nullptr, &group_only, wgm, wgn, kw, 4, 0, kTapsRagged};
}
constexpr IgemmLaunch stream(int BM, int BN, int wgm, int wgn)
{
    return IgemmLaunch{"", ALT_BF16, BM, BN, 64, LOAD_VEC, LOAD_VEC, 2, 1, 0, nullptr, &group_only, wgm, wgn, 1, 1, 0, kTapsRagged};
}
// The body by a wave's loads of a patch: bodies B, B + 1, ... issue kSlabLoads[FIRST], ...
template <int B, int FIRST, int WAVES>
int patch_body(const DconvParams &p)
{
    if (p.R != 3 || p.S != 3) return -1;
    const int loads = (int)(((uint32_t)p.patch_bytes - kSlabZero) / 1024 + WAVES - 1) / WAVES;
    for (int i = FIRST; i < 3; ++i)
        if (loads <= kSlabLoads[i]) return B + i - FIRST;
    return -1;
}
template <int B>
int one_tap(const DconvParams &p) { return p.taps == 1 ? B : -1; }
const GroupTile kTiles[] = {
    {slab(64, 64, 2, 2, 1), patch_body<0, 0, 4>}, {slab(64, 32, 1, 1, 4), patch_body<3, 1, 1>}, {slab(128, 64, 2, 2, 1), patch_body<5, 1, 4>},
    {stream(64, 64, 2, 2), one_tap<7>}, {stream(128, 64, 4, 1), one_tap<8>},
};

// 90 sets of five layers and 136 random lists of two to eight, predicted at 0.7 to 1.4 of the time one by one: up to this line together takes 0.56 to 1.07 of it
// (five layers of 172 images of 64 channels at 54 x 54 266 us, 288 one by one), beyond 0.72 to 1.3 (256 images at 56 x 56, predicted 1.03: 408 and 383).  The choice
// takes 3.0 and 1.5 % longer than the better of both, at 0.96 4.1 and 3.0.  (The line goes with the estimate of the kernels for short reductions: it was
// 0.96 while that was up to a third higher.)
constexpr double kLine = 1.0;

}  // namespace

const GroupFamily &group_slab()
{
    static const GroupFamily f = {2, kTiles, (int)(sizeof kTiles / sizeof kTiles[0]), Slab::kThreads, kLine, &group_launch<Slab>};
    return f;
}

}  // namespace alt
