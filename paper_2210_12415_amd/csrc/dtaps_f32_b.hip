// Instantiations of the streaming kernel over filter taps: fp32, small tiles.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DRTAPS_F32(64, 64, 2, 2, 2, 3, 32);
ALT_DRTAPS_F32(64, 32, 2, 1, 4, 4, 16);
ALT_DRTAPS_F32(64, 32, 2, 1, 2, 4, 32);

}  // namespace
}  // namespace alt
