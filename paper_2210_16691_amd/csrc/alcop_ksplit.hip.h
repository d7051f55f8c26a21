// Products with few output tiles (schedule variant 3): the waves of a block split the reduction axis.
//
// What bounds these.  A 1024 x 64 output with K = 2048, sixteen rows against a weight matrix, or a
// 256^3 product have fewer 64 x 64 tiles than the machine has compute units, and each tile walks
// its whole K through one barrier-paced ring: the time is the length of that chain (8.6 us for
// 1024 x 64 x 2048 with 16 blocks) while most compute units idle.  Two things shorten it: smaller
// tiles (16 to 64 wide, so that there are hundreds of blocks), and many loads in flight per tile.
// Here every wave of a block owns the whole BM x BN tile and one contiguous slice of K, which it
// streams through a ring of its own: no barrier in the loop, only the wave's own load counter, and
// NW * S k-tiles in flight per block.  At the end the waves' fp32 tiles are added in LDS in wave
// order (deterministic), with the fused epilogue and the conversion in the same pass.
//
// Small tiles fetch more bytes per flop than large ones, so this pays only while the machine is
// short of tiles; measured_applies and measured_conv_applies in alcop_dispatch.h draw that line.
//
// The matrix instruction is v_mfma_f32_16x16x32: X lane l = row l%16, k = 8*(l/16)..+7, Y likewise
// by column, D lane l = column l%16, rows 4*(l/16)..+3 (X from B, Y from A, as in alcop_kernel.hip.h:
// a lane owns 4 consecutive n of one output row).
#pragma once
#include "alcop_kernel.hip.h"

namespace alcop {

// One operand's 16- to 64-wide slice of a k-tile of 64, moved by one wave: 64 lanes of 16 bytes per
// load, the LDS image linear in (load, lane), swizzled on the source side.
//   k-contiguous: rows of 128 bytes, two rows per 256-byte bank line; physical chunk = chunk XOR
//     ((row/2) mod 8): a read of 16 rows hits 16 different 16-byte bank groups.
//   m/n-contiguous: one row per k; the transposing read of lanes 16g..16g+15 takes 16 columns of
//     rows 8g..8g+3 (then +4): odd g use the other 32-byte half (or, 16 wide, the other four rows) of
//     the lines even g use, and, 64 wide, rows 2,3 of every four the other 64-byte half.
template <int LAY_, int BX_>
struct WaveOpnd {
  static constexpr int LAY = LAY_, BX = BX_, BK = 64;
  static constexpr int BYTES = BX * BK * 2;
  static constexpr int NL = BYTES / 1024;                        // loads per k-tile
  static constexpr int CPR = LAY == LAY_K ? BK / 8 : BX / 8;     // 16-byte chunks per LDS row
  static constexpr int RSTEP = 64 / CPR;                         // LDS rows per load
  static constexpr int T = BX / 16;                              // 16-wide sub-tiles
  static constexpr int NV = LAY == LAY_K || BX == 64 ? 2 : 1;    // loads in one period of the swizzle
  static_assert(BX == 16 || BX == 32 || BX == 64, "tile width");

  // logical row and chunk held by slot q of the image
  __device__ static __forceinline__ void slot(int q, int& row, int& c)
  {
    const int pr = q / CPR, pc = q % CPR;
    row = pr;
    c = pc;
    if constexpr (LAY == LAY_K) {
      c = pc ^ ((pr >> 1) & 7);
    } else if constexpr (BX == 16) {
      row = pr ^ (((pr >> 3) & 1) << 2);
    } else {
      c = pc ^ (((pr >> 3) & 1) << 1);
      if constexpr (BX == 64) c ^= ((pr >> 1) & 1) << 2;
    }
  }
  // byte address of fragment data inside the image.  LAY_K: chunk 4*ki + lane/16 of row
  // 16 t + lane%16.  LAY_MN: the 8 bytes lane l supplies to half h of the transposing read of
  // fragment ki, sub-tile t.
  __device__ static __forceinline__ uint32_t addr(int lane, int t, int ki, int h)
  {
    if constexpr (LAY == LAY_K) {
      const int row = 16 * t + (lane & 15);
      return (uint32_t)(row * 128 + (((4 * ki + (lane >> 4)) ^ ((row >> 1) & 7)) * 16));
    } else {
      const int s = lane & 15;
      const int k = 32 * ki + 8 * (lane >> 4) + 4 * h + (s >> 2);
      const int col = 16 * t + 4 * (s & 3);
      int pr = k, pc = col >> 3;
      if constexpr (BX == 16) {
        pr = k ^ (((k >> 3) & 1) << 2);
      } else {
        pc ^= ((k >> 3) & 1) << 1;
        if constexpr (BX == 64) pc ^= ((k >> 1) & 1) << 2;
      }
      return (uint32_t)(pr * (BX * 2) + pc * 16 + (col & 7) * 2);
    }
  }
};

// DT, tile, NW waves, S ring stages per wave; layouts and A producer as in KCfg (AM 0, 1, 2).
template <int DT_, int BM_, int BN_, int NW_, int S_, int BL_, int AM_, int AL_ = 0>
struct WCfg {
  static constexpr int DT = DT_, BM = BM_, BN = BN_, BK = 64, NW = NW_, S = S_, BL = BL_, AM = AM_, AL = AL_;
  static constexpr int NT = NW * 64;
  using OA = WaveOpnd<AL ? LAY_MN : LAY_K, BM>;
  using OB = WaveOpnd<BL ? LAY_K : LAY_MN, BN>;
  static constexpr int TM = OA::T, TN = OB::T;
  static constexpr int L = OA::NL + OB::NL;
  static constexpr int STAGE_BYTES = OA::BYTES + OB::BYTES;
  static constexpr int RING_BYTES = S * STAGE_BYTES;
  static constexpr int RS = BN * 4 + 16;                        // row stride of a wave's fp32 tile
  static constexpr int RED_BYTES = NW * BM * RS;
  static constexpr int LDS_BYTES = NW * RING_BYTES > RED_BYTES ? NW * RING_BYTES : RED_BYTES;
  static_assert(S >= 2 && (S - 1) * L <= 63, "vmcnt is a 6-bit counter");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
  static_assert(AM >= 0 && AM <= 2 && !(AM != 0 && AL == 1), "A producer");
};

template <class C, class HW>
__device__ __forceinline__ void ksplit_body(const Params& p)
{
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, S = C::S, TM = C::TM, TN = C::TN;
  using OA = typename C::OA;
  using OB = typename C::OB;
  const uint32_t lds0 = HW::lds_base();
  const int lane = HW::lane_id();
  const int wave = HW::wave_id();
  const int batch = HW::block_y();
  int tm, tn;
  tile_of_block(p, HW::block_x(), tm, tn);

  // this wave's k-tiles: [kt0, kt1)
  const int nko = (p.K + BK - 1) / BK;
  const int per = (nko + C::NW - 1) / C::NW;
  const int kt0 = wave * per;
  const int kt1 = (kt0 + per) < nko ? (kt0 + per) : nko;

  const char* Ab = (const char*)p.A + (long)batch * p.strideA * 2;
  const char* Bb = (const char*)p.B + (long)batch * p.strideB * 2;

  // ---- producer state -------------------------------------------------------------------------
  // lane offset of load i = vo[i % NV] + (i / NV) * step; k of the lane's chunk (k-contiguous), so
  // that chunks past K can be pushed out of range in the last k-tile
  typename HW::Rsrc rsA, rsB;
  uint32_t voA[2] = {0, 0}, voB[2] = {0, 0}, stA = 0, stB = 0, ksA = 0, ksB = 0;
  int k8A[2] = {0, 0}, k8B[2] = {0, 0};
  auto setup = [&](auto op, const char* base, int t, int extent, int ld, typename HW::Rsrc& rs, uint32_t (&vo)[2],
                   int (&k8)[2], uint32_t& st, uint32_t& ks) __attribute__((always_inline)) {
    using O = decltype(op);
    const int valid = (extent - t * O::BX) < O::BX ? (extent - t * O::BX) : O::BX;
#pragma unroll
    for (int v = 0; v < O::NV; v++) {
      int row, c;
      O::slot(v * 64 + lane, row, c);
      vo[v] = (uint32_t)(row * ld * 2 + c * 16);
      k8[v] = c * 8;
    }
    if constexpr (O::LAY == LAY_K) {
      rs = HW::make_rsrc(base + (long)t * O::BX * ld * 2, ((valid - 1) * ld + p.K) * 2);
      ks = BK * 2;
    } else {
      rs = HW::make_rsrc(base + (long)t * O::BX * 2, ((p.K - 1) * ld + valid) * 2);
      ks = (uint32_t)(BK * ld * 2);
    }
    st = (uint32_t)(O::NV * O::RSTEP * ld * 2);
  };
  // convolution: geometry of the row each load gathers, tap of the next k-tile (AM 1: uniform; AM 2:
  // per lane and chunk parity)
  constexpr int NVA = OA::NV;
  int ih0[OA::NL], iw0[OA::NL];
  uint32_t coff[OA::NL];
  int cc0[2] = {0, 0}, cs[2] = {0, 0}, crd[2] = {0, 0}, csd[2] = {0, 0};
  if constexpr (C::AM == 0) {
    setup(OA{}, Ab, tm, p.M, p.lda, rsA, voA, k8A, stA, ksA);
  } else {
    rsA = HW::make_rsrc(p.A, (int)p.a_span);
#pragma unroll
    for (int i = 0; i < OA::NL; i++) {
      int row, c;
      OA::slot(i * 64 + lane, row, c);
      const int m = tm * BM + row;
      const int img = (int)p.rPQ.div((uint32_t)m);
      const int pq = m - img * (p.cP * p.cQ);
      const int pp = (int)p.rQ.div((uint32_t)pq), qq = pq - pp * p.cQ;
      ih0[i] = (m < p.M) ? pp * p.csh - p.cph : -0x40000000;
      iw0[i] = qq * p.csw - p.cpw;
      coff[i] = (uint32_t)((((img * p.cH + (pp * p.csh - p.cph)) * p.cW) + iw0[i]) * p.cPix * 2 +
                           (C::AM == 1 ? c * 16 : 0));
      if (i < NVA) {
        k8A[i] = c * 8;
        const int kc = kt0 * BK + (C::AM == 2 ? c * 8 : 0);
        const int tap = (int)p.rC8.div((uint32_t)kc / 8u);
        const int r = (int)p.rS.div((uint32_t)tap);
        cc0[i] = kc - tap * p.cC;
        cs[i] = tap - r * p.cS;
        crd[i] = r * p.cdh;
        csd[i] = cs[i] * p.cdw;
      }
    }
  }
  setup(OB{}, Bb, tn, p.N, p.ldb, rsB, voB, k8B, stB, ksB);

  const uint32_t ring = lds0 + (uint32_t)wave * C::RING_BYTES;
  // the L loads of k-tile kt (past the slice: as many loads that fetch nothing) into ring slot `slot`
  auto issue = [&](int kt, int slot) __attribute__((always_inline)) {
    const uint32_t dst = ring + (uint32_t)slot * C::STAGE_BYTES;
    const bool live = kt < kt1;
    const uint32_t kb = live ? (uint32_t)kt * ksB : 0x80000000u;
    const uint32_t ka = live ? (uint32_t)kt * ksA : 0x80000000u;
    const int k0 = kt * BK;
    const int kend = live ? p.K : 0;
#pragma unroll
    for (int i = 0; i < OA::NL; i++) {
      constexpr int V = NVA;
      const int v = i % V;
      uint32_t off;
      if constexpr (C::AM == 0) {
        off = voA[v] + (uint32_t)(i / V) * stA + ka;
        if (OA::LAY == LAY_K && k0 + k8A[v] >= p.K) off |= 0x80000000u;
      } else {
        const bool ok = (k0 + k8A[v] < kend) & ((unsigned)(ih0[i] + crd[v]) < (unsigned)p.cH) &
                        ((unsigned)(iw0[i] + csd[v]) < (unsigned)p.cW);
        off = ok ? coff[i] + (uint32_t)(((crd[v] * p.cW + csd[v]) * p.cPix + cc0[v]) * 2) : 0x80000000u;
      }
      HW::dma16(rsA, off, dst + i * 1024);
    }
#pragma unroll
    for (int i = 0; i < OB::NL; i++) {
      const int v = i % OB::NV;
      uint32_t off = voB[v] + (uint32_t)(i / OB::NV) * stB + kb;
      if (OB::LAY == LAY_K && k0 + k8B[v] >= p.K) off |= 0x80000000u;
      HW::dma16(rsB, off, dst + OA::BYTES + i * 1024);
    }
    if constexpr (C::AM != 0) {
#pragma unroll
      for (int v = 0; v < NVA; v++) {
        cc0[v] += BK;
        while (cc0[v] >= p.cC) {
          cc0[v] -= p.cC;
          cs[v]++;
          csd[v] += p.cdw;
          if (cs[v] == p.cS) {
            cs[v] = 0;
            csd[v] = 0;
            crd[v] += p.cdh;
          }
        }
      }
    }
  };

  // ---- consumer ---------------------------------------------------------------------------------
  auto read = [&](auto op, uint32_t base, int t, int ki) __attribute__((always_inline)) {
    using O = decltype(op);
    u32x4 f;
    if constexpr (O::LAY == LAY_K) {
      f = HW::lds_read16(base + O::addr(lane, t, ki, 0));
    } else {
      const u32x2 lo = HW::lds_read_tr8(base + O::addr(lane, t, ki, 0));
      const u32x2 hi = HW::lds_read_tr8(base + O::addr(lane, t, ki, 1));
      f = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
    return f;
  };
  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TM; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < S; s++) issue(kt0 + s, s);
  int slot = 0;
  for (int kt = kt0; kt < kt1; kt++) {
    HW::template wait_vm<(S - 1) * C::L>();      // k-tile kt has landed; no other wave is involved
    const uint32_t base = ring + (uint32_t)slot * C::STAGE_BYTES;
    u32x4 fa[2][TM], fb[2][TN];
#pragma unroll
    for (int ki = 0; ki < 2; ki++) {
#pragma unroll
      for (int j = 0; j < TM; j++) fa[ki][j] = read(OA{}, base, j, ki);
#pragma unroll
      for (int i = 0; i < TN; i++) fb[ki][i] = read(OB{}, base + OA::BYTES, i, ki);
    }
    HW::wait_lds();                              // the slot is read: refill it
    issue(kt + S, slot);
    slot = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
    for (int ki = 0; ki < 2; ki++)
#pragma unroll
      for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++) acc[i][j] = HW::template mma16<C::DT>(fb[ki][i], fa[ki][j], acc[i][j]);
  }

  // ---- sum over the waves, epilogue -----------------------------------------------------------------
  const bool fused = p.alpha != 1.0f || p.bias != nullptr || p.act != 0;
  constexpr int GPR = BN / 4;                    // groups of 4 columns per row
  constexpr int GROUPS = BM * GPR;
  HW::template wait_vm<0>();                     // the loads that fetch nothing still write LDS
  HW::block_barrier();
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TM; j++)
      HW::lds_write(lds0 + (uint32_t)((wave * BM + j * 16 + (lane & 15)) * C::RS + (i * 16 + 4 * (lane >> 4)) * 4), acc[i][j]);
  HW::wait_lds();
  HW::block_barrier();
  const float floor = p.act == 1 ? 0.f : -__builtin_inff();
#pragma unroll
  for (int g0 = 0; g0 < GROUPS; g0 += C::NT) {
    const int g = g0 + wave * 64 + lane;
    if (GROUPS % C::NT != 0 && g0 + wave * 64 >= GROUPS) break;
    const int row = g / GPR, col = (g % GPR) * 4;
    const int m = tm * BM + row, n = tn * BN + col;
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (p.bias != nullptr) b = HW::global_load_f32x4(p.bias + (n < p.N ? n : 0));
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < C::NW; w++) {
      const u32x4 t = HW::lds_read16(lds0 + (uint32_t)((w * BM + row) * C::RS + col * 4));
      const f32x4 f = __builtin_bit_cast(f32x4, t);
#pragma unroll
      for (int e = 0; e < 4; e++) v[e] += f[e];
    }
    if (fused) {
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const float t = v[e] * p.alpha + b[e];
        v[e] = t < floor ? 0.f : t;
      }
    }
    auto store = [&](auto zero) __attribute__((always_inline)) {
      using OT = decltype(zero);
      typedef OT ot4 __attribute__((ext_vector_type(4)));
      char* dst = (char*)p.C + ((long)batch * p.strideC + (long)m * p.ldc + n) * (long)sizeof(OT);
      const ot4 h = {HW::template cvt<OT>(v[0]), HW::template cvt<OT>(v[1]), HW::template cvt<OT>(v[2]),
                     HW::template cvt<OT>(v[3])};
      if (m >= p.Mv) return;
      if (!p.c_any) {
        if (n < p.N) HW::template global_store<ot4>(dst, h);
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (n + e < p.Nv) HW::template global_store<OT>(dst + e * (long)sizeof(OT), h[e]);
      }
    };
    if (p.out_dtype == 2)
      store(0.0f);
    else if (p.out_dtype == 0)
      store((_Float16)0);
    else
      store((__bf16)0);
  }
}

template <class C, class HW>
__global__ void __launch_bounds__(C::NT) alcop_ksplit(const Params p)
{
  ksplit_body<C, HW>(p);
}

template <class C, class HW>
__global__ void __launch_bounds__(C::NT) alcop_ksplit_small(const SmallArgs s)
{
  ksplit_body<C, HW>(expand_args<C>(s));
}

}  // namespace alcop
