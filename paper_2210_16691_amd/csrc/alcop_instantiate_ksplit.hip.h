// Launcher and table helpers of the kernels whose waves split the reduction axis.
#pragma once
#include "alcop_instantiate.hip.h"
#include "alcop_ksplit.hip.h"

namespace alcop {

template <class C>
hipError_t prepare_ksplit()
{
  static std::once_flag once;
  static hipError_t attr_rc = hipSuccess;
  std::call_once(once, [] {
    attr_rc = hipFuncSetAttribute((const void*)alcop_ksplit<C, Gfx950>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    if constexpr (C::AM == 0) {
      if (attr_rc == hipSuccess)
        attr_rc = hipFuncSetAttribute((const void*)alcop_ksplit_small<C, Gfx950>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_BYTES);
    }
  });
  return attr_rc;
}

template <class C>
hipError_t launch_ksplit(const Params& p, dim3 grid, hipStream_t st)
{
  const hipError_t rc = prepare_ksplit<C>();
  if (rc != hipSuccess) return rc;
  if constexpr (C::AM == 0) {
    SmallArgs s;
    if (small_args(p, grid.y, &s)) {
      alcop_ksplit_small<C, Gfx950><<<grid, dim3(C::NT), C::LDS_BYTES, st>>>(s);
      return hipGetLastError();
    }
  }
  alcop_ksplit<C, Gfx950><<<grid, dim3(C::NT), C::LDS_BYTES, st>>>(p);
  return hipGetLastError();
}

// schedules name these by their tile, k-tile 64 and ring stages (wave tile = block tile)
template <int DT, int BM, int BN, int NW, int S, int BL, int AM, int AL = 0>
void add_ksplit(std::vector<KernelEntry>& t)
{
  using C = WCfg<DT, BM, BN, NW, S, BL, AM, AL>;
  t.push_back(KernelEntry{DT, BM, BN, 64, BM, BN, S, 1, 0, BL, AM, AL, 0, 0, 2, C::LDS_BYTES, C::NT, C::L, 0,
                          &launch_ksplit<C>, &prepare_ksplit<C>});
}

}  // namespace alcop

#define ALCOP_KSPLIT_TILES(T, DT, BL, AM, AL)      \
  add_ksplit<DT, 16, 16, 8, 2, BL, AM, AL>(T);     \
  add_ksplit<DT, 16, 32, 8, 2, BL, AM, AL>(T);     \
  add_ksplit<DT, 32, 32, 8, 2, BL, AM, AL>(T);     \
  add_ksplit<DT, 32, 64, 4, 2, BL, AM, AL>(T);
