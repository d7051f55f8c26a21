// Launchers of the copy kernels behind the entry points for unaligned operands.
#include "alcop_gfx950.hip.h"
#include "alcop_registry.h"
namespace alcop {

hipError_t launch_pack(const PackParams& p, unsigned blocks, hipStream_t st)
{
  alcop_pack<Gfx950><<<dim3(blocks), dim3(PACK_THREADS), 0, st>>>(p);
  return hipGetLastError();
}

hipError_t launch_copy_out(const CopyOutParams& p, hipStream_t st)
{
  alcop_copy_out<Gfx950><<<dim3(copy_out_blocks(p)), dim3(PACK_THREADS), 0, st>>>(p);
  return hipGetLastError();
}

hipError_t prepare_copies()
{
  hipFuncAttributes at;
  const hipError_t rc = hipFuncGetAttributes(&at, (const void*)alcop_pack<Gfx950>);
  return rc != hipSuccess ? rc : hipFuncGetAttributes(&at, (const void*)alcop_copy_out<Gfx950>);
}

}  // namespace alcop
