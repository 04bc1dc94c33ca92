// Instantiations of the streaming kernel over filter taps: bf16 products with B stored [K][N] and any K that is a
// multiple of eight.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DRSTREAM_KN(256, 256, 2, 4, 1, 4, 32);
ALT_DRSTREAM_KN(256, 128, 4, 2, 1, 3, 64);
ALT_DRSTREAM_KN(128, 128, 4, 2, 1, 4, 64);
ALT_DRSTREAM_KN(64, 64, 2, 2, 1, 4, 64);

}  // namespace
}  // namespace alt
