// Launcher and table helpers of the convolution kernels with a resident patch for any geometry.
#pragma once
#include "alcop_instantiate.hip.h"
#include "alcop_convres.hip.h"

namespace alcop {

// C and the same kernel for ragged windows, D (C itself where no call has such windows)
template <class C, class D>
hipError_t prepare_convres()
{
  static std::once_flag once;
  static hipError_t attr_rc = hipSuccess;
  std::call_once(once, [] {
    for (const void* f : {(const void*)alcop_convres<C, Gfx950>, (const void*)alcop_convres<D, Gfx950>})
      if (attr_rc == hipSuccess)
        attr_rc = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  });
  return attr_rc;
}

template <class C, class D>
hipError_t launch_convres(const Params& p, dim3 grid, hipStream_t st)
{
  const hipError_t rc = prepare_convres<C, D>();
  if (rc != hipSuccess) return rc;
  const unsigned lds = (unsigned)convres_lds(C::RING_BYTES, C::MIN_LDS, p.rloads, p.rtab, p.ragged);
  if (p.ragged)
    alcop_convres<D, Gfx950><<<grid, dim3(D::NT), lds, st>>>(p);
  else
    alcop_convres<C, Gfx950><<<grid, dim3(C::NT), lds, st>>>(p);
  return hipGetLastError();
}

// schedules name these by their tile, k-tile 64, wave tile 64 x 64 and ring stages
template <int DT, int BM, int BN, int S, int BL>
void add_convres(std::vector<KernelEntry>& t)
{
  using C = RCfg<DT, BM, BN, S, BL>;
  using D = RCfg<DT, BM, BN, S, BL, BL == 0>;   // ragged windows come with RSCK weights only
  t.push_back(KernelEntry{DT, BM, BN, 64, 64, 64, S, 2, 1, BL, 4, 0, 0, 0, 3, C::MIN_LDS, C::NT, C::L, C::RING_BYTES,
                          &launch_convres<C, D>, &prepare_convres<C, D>});
}

}  // namespace alcop

#define ALCOP_CONVRES_TILES(T, DT, BL)  \
  add_convres<DT, 256, 64, 2, BL>(T);   \
  add_convres<DT, 256, 64, 3, BL>(T);   \
  add_convres<DT, 128, 128, 2, BL>(T);  \
  add_convres<DT, 128, 128, 3, BL>(T);  \
  add_convres<DT, 128, 64, 2, BL>(T);   \
  add_convres<DT, 128, 64, 3, BL>(T);   \
  add_convres<DT, 64, 128, 2, BL>(T);   \
  add_convres<DT, 64, 64, 2, BL>(T);
