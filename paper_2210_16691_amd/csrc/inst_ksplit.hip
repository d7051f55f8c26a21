// Kernels whose waves split the reduction axis (schedule variant 3): matrix operands, every layout.
#include "alcop_instantiate_ksplit.hip.h"
namespace alcop {
void register_ksplit(std::vector<KernelEntry>& t)
{
  ALCOP_KSPLIT_TILES(t, 0, 0, 0, 0)
  ALCOP_KSPLIT_TILES(t, 0, 1, 0, 0)
  ALCOP_KSPLIT_TILES(t, 1, 0, 0, 0)
  ALCOP_KSPLIT_TILES(t, 1, 1, 0, 0)
  ALCOP_KSPLIT_TILES(t, 0, 0, 0, 1)
  ALCOP_KSPLIT_TILES(t, 0, 1, 0, 1)
  ALCOP_KSPLIT_TILES(t, 1, 0, 0, 1)
  ALCOP_KSPLIT_TILES(t, 1, 1, 0, 1)
}
}  // namespace alcop
