// Convolution kernels with a resident patch for any geometry (schedule variant 4), RSCK weights.
#include "alcop_instantiate_convres.hip.h"
namespace alcop {
void register_convres_rsck(std::vector<KernelEntry>& t)
{
  ALCOP_CONVRES_TILES(t, 0, 0)
  ALCOP_CONVRES_TILES(t, 1, 0)
}
}  // namespace alcop
