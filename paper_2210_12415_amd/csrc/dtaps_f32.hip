// Instantiations of the streaming kernel over filter taps: fp32, large tiles.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DRTAPS_F32(128, 128, 4, 2, 1, 4, 32);
ALT_DRTAPS_F32(128, 64, 4, 2, 1, 4, 32);
ALT_DRTAPS_F32(64, 64, 2, 2, 1, 4, 32);

}  // namespace
}  // namespace alt
