// Products of operands at any element address: both types, every operand layout, two pipeline depths, one or eight
// partial sums.
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
}  // namespace

hipError_t launch_direct(const DirectArgs& a, int dt, bool transA, bool transB, bool split, hipStream_t st)
{
  return dispatch_direct<Launch>(a, dt, transA, transB, split, st);
}

}  // namespace alcop
