// Convolutions in one launch: bf16, NCHW, 3x3 and 1x1 filters.
#include "group.h"

namespace alt {
namespace {

// The tiles of eight waves of dplanar.h, one workgroup on a compute unit: a launch of their own leaves a quarter of the units idle where a layer has
// 196 tiles.
struct Planar {
    static constexpr int kThreads = 512, kWaves = 2;
    static __device__ __forceinline__ void run(int body, const DconvParams &p, int id)
    {
        switch (body) {
        case 0: dplanar_body<256, 64, 4, 2, 1, 1>(p, id); break;
        case 1: dplanar_body<256, 64, 4, 2, 1, 3>(p, id); break;
        case 2: dplanar_body<128, 64, 4, 2, 1, 1>(p, id); break;
        case 3: dplanar_body<128, 64, 4, 2, 1, 3>(p, id); break;
        case 4: dplanar_body<128, 32, 4, 1, 2, 1>(p, id); break;
        case 5: dplanar_body<128, 32, 4, 1, 2, 3>(p, id); break;
        case 6: dplanar_body<64, 32, 2, 1, 4, 1>(p, id); break;
        default: dplanar_body<64, 32, 2, 1, 4, 3>(p, id); break;
        }
    }
};

constexpr IgemmLaunch tile(int BM, int BN, int wgm, int wgn, int kw, int ragged)
{
    return IgemmLaunch{"", ALT_BF16, BM, BN, 64, LOAD_VEC, LOAD_VEC, 0, 0, 0, nullptr, &group_only, wgm, wgn, kw, 2, 0, 0, ragged};
}
template <int B>
int body(const DconvParams &p) { return p.R == 3 ? B + 1 : B; }
// (a problem's channels fit a tile of one of the two kinds)
const GroupTile kTiles[] = {
    {tile(256, 64, 4, 2, 1, 0), body<0>}, {tile(256, 64, 4, 2, 1, 1), body<0>}, {tile(128, 64, 4, 2, 1, 0), body<2>},
    {tile(128, 64, 4, 2, 1, 1), body<2>}, {tile(128, 32, 4, 1, 2, 0), body<4>}, {tile(128, 32, 4, 1, 2, 1), body<4>},
    {tile(64, 32, 2, 1, 4, 0), body<6>},  {tile(64, 32, 2, 1, 4, 1), body<6>},
};

// (64 random lists of two to eight: the few predicted above take 0.79 to 1.6 of the time one by one)
constexpr double kLine = 0.96;

}  // namespace

const GroupFamily &group_planar()
{
    static const GroupFamily f = {3, kTiles, (int)(sizeof kTiles / sizeof kTiles[0]), Planar::kThreads, kLine, &group_launch<Planar>};
    return f;
}

}  // namespace alt
