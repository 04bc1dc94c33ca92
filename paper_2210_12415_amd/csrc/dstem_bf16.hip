// Instantiations of the direct convolution for images of few channels: chunk pairs of the reduction x 32-channel tiles.
#include "dstem.h"

namespace alt {
namespace {

#define ALT_DSTEM(NKC, TN, BN, BK)                                                                                \
    const bool reg_dstem_##NKC##_##TN =                                                                          \
        (igemm_register(IgemmLaunch{"bf16_256x" #BN "x" #BK "_few", ALT_BF16, 256, BN, BK, LOAD_GATHER, LOAD_GATHER, \
                                    NKC, 0, 0, nullptr, &dstem_launch<NKC, TN>, 4, 1, 1, 3}),                    \
         true)

ALT_DSTEM(5, 1, 32, 80);                          // 3x3 over three channels
ALT_DSTEM(5, 2, 64, 80);
ALT_DSTEM(8, 1, 32, 128);                          // 5x5
ALT_DSTEM(8, 2, 64, 128);
ALT_DSTEM(11, 1, 32, 176);                         // 7x7
ALT_DSTEM(11, 2, 64, 176);

}  // namespace
}  // namespace alt
