// Table of the kernels built into the library: one entry per template instance.
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>
#include <vector>

#include "alcop_direct.hip.h"
#include "alcop_kernel.hip.h"
#include "alcop_pack.hip.h"
#include "alcop_splitk.hip.h"

namespace alcop {

struct KernelEntry {
  int dt, bm, bn, bk, wm, wn, stages, reg_stages, fuse, bl, am, al;
  int sk;   // 1: split-K variant (grid.z slices of the reduction axis, fp32 partial tiles)
  int pf;   // 1: the kernel has the HBM -> L2 touch level (schedules with l2_prefetch > 0)
  int st;   // 1: persistent producer / consumer kernel (schedule variant 2); 2: the waves of a block
            // split the reduction axis (schedule variant 3); 3: convolution with a resident patch for
            // any geometry (schedule variant 4)
  int lds_bytes, threads, loads_per_stage;
  int patch_off;   // am == 3, 4: LDS offset of the input patch (its size is per call)
  hipError_t (*launch)(const Params&, dim3, hipStream_t);
  // what the first launch would do besides launching (the opt-in to the kernel's LDS size), so
  // that alcop_init can do it ahead of time; may be null
  hipError_t (*prepare)() = nullptr;
};

// Sub-tables, one per source shard (compiled in parallel).
void register_f16_kn_big(std::vector<KernelEntry>&);
void register_f16_kn_mid(std::vector<KernelEntry>&);
void register_f16_kn_small(std::vector<KernelEntry>&);
void register_bf16_kn(std::vector<KernelEntry>&);
void register_nk(std::vector<KernelEntry>&);
void register_conv(std::vector<KernelEntry>&);
void register_ta(std::vector<KernelEntry>&);
void register_conv_krsc(std::vector<KernelEntry>&);
void register_conv_anyc(std::vector<KernelEntry>&);
void register_conv_patch(std::vector<KernelEntry>&);
void register_bk128(std::vector<KernelEntry>&);
void register_deep(std::vector<KernelEntry>&);
void register_wide(std::vector<KernelEntry>&);
void register_pf(std::vector<KernelEntry>&);
void register_stream(std::vector<KernelEntry>&);
void register_ksplit(std::vector<KernelEntry>&);
void register_ksplit_conv(std::vector<KernelEntry>&);
void register_convres_rsck(std::vector<KernelEntry>&);
void register_convres_krsc(std::vector<KernelEntry>&);
void register_splitk_gemm(std::vector<KernelEntry>&);
void register_splitk_conv(std::vector<KernelEntry>&);

// Second step of a split-K product (alcop_splitk.hip.h).
hipError_t launch_splitk_reduce(const ReduceParams& p, dim3 grid, hipStream_t st);

// Copies into the padded workspace images, all segments of a call (alcop_pack.hip.h).
hipError_t launch_pack(const PackParams& p, unsigned blocks, hipStream_t st);
// C from a dense image of it in the workspace.
hipError_t launch_copy_out(const CopyOutParams& p, hipStream_t st);
// Loads both kernels, so that alcop_init can do it ahead of time.
hipError_t prepare_copies();

// Product of operands at any element address (alcop_direct.hip.h); split: in place of a kernel whose waves
// split K.
hipError_t launch_direct(const DirectArgs& a, int dt, bool transA, bool transB, bool split, hipStream_t st);
// Loads all of them.
hipError_t prepare_direct();
// ... with a launcher of one configuration, LAUNCH<DCfg>::go(args, blocks, stream).  Two k-tiles ahead
// where there are no more (K <= 128: 235 x 3780 x 59 4.2 us, 4.5 with four, which load the last again), else
// four (26 x 41 x 2500 22.7 us with two, 15.8 with four).
template <template <class> class LAUNCH>
hipError_t dispatch_direct(const DirectArgs& a, int dt, bool transA, bool transB, bool split, hipStream_t st)
{
  const unsigned blocks = (unsigned)((a.M + 63) / 64) * (unsigned)((a.N + 63) / 64);
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  auto depth = [&](auto cdt, auto cbl, auto cal) {
    constexpr int DT = decltype(cdt)::value, BL = decltype(cbl)::value, AL = decltype(cal)::value;
    if (!split)
      return a.K <= 128 ? LAUNCH<DCfg<DT, 2, BL, AL, 1>>::go(a, blocks, st) : LAUNCH<DCfg<DT, 4, BL, AL, 1>>::go(a, blocks, st);
    if (a.K > 256) return LAUNCH<DCfg<DT, 4, BL, AL, 8>>::go(a, blocks, st);
    return a.K <= 128 ? LAUNCH<DCfg<DT, 2, BL, AL, 2>>::go(a, blocks, st) : LAUNCH<DCfg<DT, 4, BL, AL, 4>>::go(a, blocks, st);
  };
  auto layouts = [&](auto cdt) {
    if (transA) return transB ? depth(cdt, I1{}, I1{}) : depth(cdt, I0{}, I1{});
    return transB ? depth(cdt, I1{}, I0{}) : depth(cdt, I0{}, I0{});
  };
  return dt ? layouts(I1{}) : layouts(I0{});
}
// LAUNCH<DCfg>::go for every configuration; the arguments are none of a call's.
template <template <class> class LAUNCH>
hipError_t every_direct()
{
  for (int i = 0; i < 16; i++)
    for (int K : {128, 256, 512}) {
      DirectArgs a = {};
      a.M = a.N = 1;
      a.K = K;
      const hipError_t rc = dispatch_direct<LAUNCH>(a, i & 1, i & 2, i & 4, i & 8, nullptr);
      if (rc != hipSuccess) return rc;
    }
  return hipSuccess;
}

// Device address and size of the library's own scratch array on the current device (set up on
// the first call per device; allocates nothing afterwards).  Its size is part of the interface
// (ALCOP_SPLITK_STATIC_BYTES in alcop.h; alcop_api.cpp checks that the two agree).
constexpr size_t kSplitkStaticBytes = 32u << 20;
hipError_t splitk_scratch(void** ptr, size_t* bytes);

const std::vector<KernelEntry>& registry();

}  // namespace alcop
