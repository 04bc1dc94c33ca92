// Instantiations of the streaming kernel over filter taps: bf16, channels a multiple of the K step.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DTAPS(256, 256, 2, 4, 1, 4, 32);
ALT_DTAPS(256, 128, 4, 2, 1, 3, 64);
ALT_DTAPS(128, 128, 4, 2, 1, 4, 64);
ALT_DTAPS(256, 64, 8, 1, 1, 3, 64);
ALT_DTAPS(128, 64, 4, 1, 1, 4, 64);
ALT_DTAPS(64, 64, 2, 2, 1, 4, 64);
ALT_DTAPS(64, 64, 2, 1, 4, 4, 32);

}  // namespace
}  // namespace alt
