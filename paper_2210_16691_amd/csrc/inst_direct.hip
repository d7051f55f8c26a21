// Products of operands at any element address: both types, every operand layout, one, two, four or eight partial
// sums.
#include "alcop_gfx950.hip.h"
#include "alcop_registry.h"
namespace alcop {
namespace {
template <class C>
struct Launch {
  static hipError_t go(const DirectArgs& a, unsigned blocks, hipStream_t st)
  {
    alcop_direct<C, Gfx950><<<dim3(blocks), dim3(C::NT), C::LDS_BYTES, st>>>(a);
    return hipGetLastError();
  }
};
template <class C>
struct Load {
  static hipError_t go(const DirectArgs&, unsigned, hipStream_t)
  {
    hipFuncAttributes at;
    return hipFuncGetAttributes(&at, (const void*)alcop_direct<C, Gfx950>);
  }
};
}  // namespace

hipError_t launch_direct(const DirectArgs& a, int dt, bool transA, bool transB, bool split, hipStream_t st)
{
  return dispatch_direct<Launch>(a, dt, transA, transB, split, st);
}

hipError_t prepare_direct() { return every_direct<Load>(); }

}  // namespace alcop
