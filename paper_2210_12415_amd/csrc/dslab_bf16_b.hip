// Instantiations of the patch-resident convolution over slabs of channels: smaller tiles.
#include "dconv_reg.h"

namespace alt {
namespace {

ALT_DSLAB(128, 64, 2, 2, 1, 32);
ALT_DSLAB(64, 64, 2, 2, 1, 32);
ALT_DSLAB(64, 32, 1, 1, 4, 32);

}  // namespace
}  // namespace alt
