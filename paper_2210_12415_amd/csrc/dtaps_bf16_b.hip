// Instantiations of the streaming kernel over filter taps: bf16, any channel count (and any K of a product) that is
// a multiple of eight; large tiles.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DRTAPS(256, 256, 2, 4, 1, 4, 32);
ALT_DRTAPS(256, 128, 4, 2, 1, 3, 64);
ALT_DRTAPS(128, 128, 4, 2, 1, 4, 64);
ALT_DRTAPS(256, 64, 8, 1, 1, 3, 64);

}  // namespace
}  // namespace alt
