// Instantiations of the patch-resident convolution over slabs of channels: tiles of 256 pixels, steps of 32 channels.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DSLAB(256, 128, 4, 2, 1, 32);
ALT_DSLAB(256, 64, 4, 1, 1, 32);

}  // namespace
}  // namespace alt
