// Convolutions in one launch: fp32, NHWC.
#include "group.h"

namespace alt {
namespace {

// Matrix instructions bound these, so what counts is that every SIMD has some: rings of 48 KB let three workgroups share a compute unit,
// and half tiles even out sums of many steps and channels that are no multiple of 64.  (Five layers of 5 images: 56 us; half tiles alone 59,
// with rings of 73 KB 64, tiles of 64x64 in steps of 16 63, of 128x64 65.)
struct F32 {
    static constexpr int kThreads = 256, kWaves = 2;
    static __device__ __forceinline__ void run(int body, const DconvParams &p, int id)
    {
        if (body == 0) dstream_body<64, 64, 2, 2, 1, 3, 32, false, kTapsDense, float, 4>(p, id, 0);
        else if (body == 1) dstream_body<64, 64, 2, 2, 1, 3, 32, false, kTapsOne, float, 4>(p, id, 0);
        else if (body == 2) dstream_body<64, 32, 2, 1, 2, 4, 16, false, kTapsDense, float, 4>(p, id, 0);
        else dstream_body<64, 32, 2, 1, 2, 4, 16, false, kTapsOne, float, 4>(p, id, 0);
    }
};

constexpr IgemmLaunch tile(int BM, int BN, int wgm, int wgn, int kw, int ns, int bk)
{
    return IgemmLaunch{"", ALT_F32, BM, BN, bk, LOAD_VEC, LOAD_VEC, ns - 1, 1, 0, nullptr, &group_only, wgm, wgn, kw, 1, 0, kTapsRagged};
}
template <int B>
int body(const DconvParams &p) { return p.taps == 1 ? B + 1 : p.w_dense ? B : -1; }
const GroupTile kTiles[] = {{tile(64, 64, 2, 2, 1, 3, 32), body<0>}, {tile(64, 32, 2, 1, 2, 4, 16), body<2>}};

}  // namespace

const GroupFamily &group_f32()
{
    static const GroupFamily f = {kTiles, (int)(sizeof kTiles / sizeof kTiles[0]), F32::kThreads, &group_launch<F32>};
    return f;
}

}  // namespace alt
