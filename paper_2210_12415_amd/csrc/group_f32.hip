// Convolutions in one launch: fp32, NHWC.
#include "group.h"

namespace alt {
namespace {

// Matrix instructions bound these, so what counts is that every SIMD has some: rings of 48 KB let three workgroups share a compute unit,
// and half tiles even out sums of many steps and channels that are no multiple of 64.  Five layers of 5 images: 52 us, matrix cores busy 57 % under
// the profiler's clock; with divisions in every step 55 (53 %, 7.4 vector instructions per matrix instruction instead of 4.0), with tiles of 64x64
// in steps of 16 55.
struct F32 {
    static constexpr int kThreads = 256, kWaves = 2;
    static __device__ __forceinline__ void run(int body, const DconvParams &p, int id)
    {
        switch (body) {
        case 0: dstream_body<64, 64, 2, 2, 1, 3, 32, false, kTapsDense, float, 4>(p, id, 0); break;
        case 1: dstream_body<64, 64, 2, 2, 1, 3, 32, false, kTapsOne, float, 4>(p, id, 0); break;
        case 2: dstream_body<64, 64, 2, 2, 1, 3, 32, false, kTapsUniform, float, 4>(p, id, 0); break;
        case 3: dstream_body<64, 32, 2, 1, 2, 4, 16, false, kTapsDense, float, 4>(p, id, 0); break;
        case 4: dstream_body<64, 32, 2, 1, 2, 4, 16, false, kTapsOne, float, 4>(p, id, 0); break;
        default: dstream_body<64, 32, 2, 1, 2, 4, 16, false, kTapsUniform, float, 4>(p, id, 0); break;
        }
    }
};

constexpr IgemmLaunch tile(int BM, int BN, int wgm, int wgn, int kw, int ns, int bk)
{
    return IgemmLaunch{"", ALT_F32, BM, BN, bk, LOAD_VEC, LOAD_VEC, ns - 1, 1, 0, nullptr, &group_only, wgm, wgn, kw, 1, 0, kTapsRagged};
}
// (where a pixel's channels are whole steps and the slices even, the walk over the taps is scalar, without divisions)
template <int B, int BK, int KW>
int body(const DconvParams &p)
{
    if (p.taps == 1) return B + 1;
    if (p.c16 % (BK / 4) == 0 && p.kq == p.ncc * p.splitk * KW * (BK / 4)) return B + 2;
    return p.w_dense ? B : -1;
}
const GroupTile kTiles[] = {{tile(64, 64, 2, 2, 1, 3, 32), body<0, 32, 1>}, {tile(64, 32, 2, 1, 2, 4, 16), body<3, 16, 2>}};

// (98 lists: together takes 0.56 to 0.88 up to here, and 0.66 to 1.08 above)
constexpr double kLine = 0.96;

}  // namespace

const GroupFamily &group_f32()
{
    static const GroupFamily f = {1, kTiles, (int)(sizeof kTiles / sizeof kTiles[0]), F32::kThreads, kLine, &group_launch<F32>};
    return f;
}

}  // namespace alt
