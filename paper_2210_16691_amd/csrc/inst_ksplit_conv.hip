// Kernels whose waves split the reduction axis (schedule variant 3): convolution gather, both
// weight layouts, channel counts that 64 divides and any multiple of 8.
#include "alcop_instantiate_ksplit.hip.h"
namespace alcop {
void register_ksplit_conv(std::vector<KernelEntry>& t)
{
  ALCOP_KSPLIT_TILES(t, 0, 0, 1, 0)
  ALCOP_KSPLIT_TILES(t, 0, 1, 1, 0)
  ALCOP_KSPLIT_TILES(t, 1, 0, 1, 0)
  ALCOP_KSPLIT_TILES(t, 1, 1, 1, 0)
  ALCOP_KSPLIT_TILES(t, 0, 0, 2, 0)
  ALCOP_KSPLIT_TILES(t, 0, 1, 2, 0)
  ALCOP_KSPLIT_TILES(t, 1, 0, 2, 0)
  ALCOP_KSPLIT_TILES(t, 1, 1, 2, 0)
}
}  // namespace alcop
