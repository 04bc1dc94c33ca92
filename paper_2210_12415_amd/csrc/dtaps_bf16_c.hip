// Instantiations of the streaming kernel over filter taps: bf16, any channel count (and any K of a product) that is
// a multiple of eight; small tiles.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DRTAPS(128, 64, 4, 1, 1, 4, 64);
ALT_DRTAPS(256, 32, 4, 1, 1, 4, 64);
ALT_DRTAPS(64, 64, 2, 2, 1, 4, 64);
ALT_DRTAPS(64, 64, 2, 1, 4, 4, 32);

}  // namespace
}  // namespace alt
