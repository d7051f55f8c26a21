// Launcher of the pack kernel behind the entry points for unaligned operands.
#include "alcop_gfx950.hip.h"
#include "alcop_registry.h"
namespace alcop {

hipError_t launch_pack(const PackParams& p, unsigned blocks, hipStream_t st)
{
  alcop_pack<Gfx950><<<dim3(blocks), dim3(PACK_THREADS), 0, st>>>(p);
  return hipGetLastError();
}

}  // namespace alcop
