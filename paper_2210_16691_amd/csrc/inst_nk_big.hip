// B stored N x K and A stored K x M: the wide tiles that the K x N layout has had.
#include "alcop_instantiate.hip.h"
namespace alcop {
// the fused pipelines, which are the faster ones of every wide tile
#define ALCOP_WIDE_PIPES(T, DT, BM, BN, BK, WM, WN, BL, AL)  \
  add_instance<DT, BM, BN, BK, WM, WN, 3, 2, 1, BL, 0, AL>(T); \
  add_instance<DT, BM, BN, BK, WM, WN, 4, 2, 1, BL, 0, AL>(T);
void register_nk_big(std::vector<KernelEntry>& t)
{
  ALCOP_WIDE_PIPES(t, 0, 256, 256, 32, 128, 64, 1, 0)
  ALCOP_WIDE_PIPES(t, 1, 256, 256, 32, 128, 64, 1, 0)
  ALCOP_WIDE_PIPES(t, 1, 256, 128, 64, 128, 64, 1, 0)
  ALCOP_WIDE_PIPES(t, 0, 256, 192, 32, 128, 96, 0, 1)
  ALCOP_WIDE_PIPES(t, 1, 256, 192, 32, 128, 96, 0, 1)
  ALCOP_WIDE_PIPES(t, 0, 256, 128, 64, 128, 64, 0, 1)
  ALCOP_WIDE_PIPES(t, 1, 256, 128, 64, 128, 64, 0, 1)
}
}  // namespace alcop
