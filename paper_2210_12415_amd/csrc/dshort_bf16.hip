// Instantiations of the kernel for short reductions.  (Wider tiles, up to 192 columns, were best for 7 % of 9400 products, by 3 %: fewer of their
// workgroups share a compute unit.)
#include "dshort.h"

namespace alt {
namespace {

#define ALT_DSHORT(TN, BN)                                                                                       \
    const bool reg_dshort_##TN = (igemm_register(IgemmLaunch{"bf16_128x" #BN "x64_short_w4x1", ALT_BF16, kShortRows, BN, 64, LOAD_VEC, LOAD_VEC, 0, 1, 0, \
                                                             nullptr, &dshort_launch<TN>, 4, 1, 1, 5}),            \
                                  true)
ALT_DSHORT(1, 32);
ALT_DSHORT(2, 64);
ALT_DSHORT(3, 96);

}  // namespace
}  // namespace alt
