// Instantiations of the patch-resident convolution over slabs of channels: steps of 64 channels, K groups of 128 x 64 tiles.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DSLAB(256, 64, 8, 1, 1, 64);
ALT_DSLAB(128, 64, 2, 2, 2, 32);

}  // namespace
}  // namespace alt
