// Convolution kernels with a resident patch for any geometry (schedule variant 4), KRSC weights.
#include "alcop_instantiate_convres.hip.h"
namespace alcop {
void register_convres_krsc(std::vector<KernelEntry>& t)
{
  ALCOP_CONVRES_TILES(t, 0, 1)
  ALCOP_CONVRES_TILES(t, 1, 1)
}
}  // namespace alcop
