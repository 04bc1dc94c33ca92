// Instantiations of the streaming GEMM kernel: small tiles and K groups.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DSTREAM(128, 64, 2, 1, 1, 4, 64);
ALT_DSTREAM(128, 64, 4, 1, 1, 4, 64);
ALT_DSTREAM(128, 64, 4, 1, 1, 8, 32);
ALT_DSTREAM(128, 64, 2, 1, 2, 3, 64);
ALT_DSTREAM(128, 64, 2, 1, 2, 6, 32);
ALT_DSTREAM(64, 128, 1, 2, 2, 3, 64);
ALT_DSTREAM(64, 64, 2, 2, 1, 4, 64);
ALT_DSTREAM(64, 64, 2, 2, 1, 8, 32);
ALT_DSTREAM(256, 64, 8, 1, 1, 3, 64);
ALT_DSTREAM(256, 64, 8, 1, 1, 4, 64);
// few rows or columns: twice the workgroups of 64x64, two K groups each (380 x 832 x 3328 10.7 us in 64x64, 8.5 here; 210 x 896 x 3584 9.5 and
// 8.4; four groups and three stages 10.0 and 9.9)
ALT_DSTREAM(64, 32, 2, 1, 2, 4, 64);

}  // namespace
}  // namespace alt
