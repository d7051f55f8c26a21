// Products of operands that are not made of aligned 16-byte chunks, in one launch.
//
// The pipelined loops take such operands from padded copies in a workspace (alcop_pack.hip.h): two
// launches, and a product that reads what another kernel has just written to another L2.  Here the
// tile loads go through registers instead: a global load of 16 bytes may start at any element, a
// direct-to-LDS load may not.  The LDS image of a tile is the one of the pipelined loops (Opnd), two
// stages of it; two or four k-tiles are in registers or on their way there.
//
// Edges.  A chunk that would reach past the end of its row starts earlier, where the row's last eight
// elements are, and is shifted down by what it starts early; zeros come in at the top.  A row past the
// last k is the last one, shifted out whole.  So the terms past K are zero times zero, and the shifts are behind a
// branch that only blocks at an edge and the last k-tile take (rows hold eight elements at least).
//   Operands that run along m or n do so in the last k-tile only.  Before it, a chunk at the edge reads up to
// seven elements past its row's end, what lies between two rows or the next row, which the operand has since the
// row is not the last; whatever they hold goes into accumulators of rows >= M or columns >= N, and those are not
// stored.  Nothing is read behind an operand's last row.
//
// What bounds it: misaligned loads, 24 bytes per clock and compute unit however many are in flight (aligned
// direct-to-LDS loads 40 to 50): 0.3 us per k-tile of 16 KB, which is also what a block alone on its unit takes.
// Tiles of 128 x 64 took 24 KB in 0.42 us and were slower for all but one of 60 products; reading the next
// k-tile's fragments beside the matrix instructions cost a block per unit and gained nothing.  Against copies and
// a pipelined kernel (bf16): 507 x 1611 x 23 4.2 us and 7.0, 142 x 1816 x 229 4.9 and 7.8, 435 x 386 x 385 6.1 and
// 8.5; long reductions lose (direct_pays).
//
// Sums.  In place of a pipelined kernel (P = 1) the k order of an element is that kernel's: the same bits.  In place
// of one whose waves split K it has P partial sums, one per k-tile up to four, else eight.  One sum over all of K had
// 1.2 (K = 170) to 2.1 times (K = 1056) the error of the copies' route (fp32 results, against 64 bits); these have
// 0.96 times in the mean over 165 products, 1.01 at most where there are more than a few hundred elements.  They
// cost 3 % (median; 0.2 us of 6): as vector registers, which two waves per SIMD make the compiler take, since reading
// 128 accumulation registers cost another 0.4 us, and cleared while the first loads are on their way.
#pragma once
#include "alcop_kernel.hip.h"

namespace alcop {

// The arguments in one 64-byte line, for the same reason as SmallArgs.
struct DirectArgs {
  const void* A;
  const void* B;
  void* C;
  const float* bias;
  int M, N, K;
  int lda, ldb, ldc;
  float alpha;
  int flags;                   // out_dtype, + 4 ReLU, + 8 raster order, + 16 c_any
};
static_assert(sizeof(DirectArgs) == 64, "one line");

// D: k-tiles in registers or on their way there.  P: partial sums per element of C.
template <int DT_, int D_, int BL_, int AL_, int P_>
struct DCfg {
  static constexpr int DT = DT_, BM = 64, BN = 64, BK = 64, WM = BM / 2, WN = BN / 2, BL = BL_, AL = AL_;
  static constexpr int NT = 256, D = D_, P = P_;
  using OA = Opnd<AL ? LAY_MN : LAY_K, BM, WM, BK, NT>;
  using OB = Opnd<BL ? LAY_K : LAY_MN, BN, WN, BK, NT>;
  static constexpr int TM = WM / 32, TN = WN / 32;
  static constexpr int STAGE_BYTES = OA::BYTES + OB::BYTES;
  static constexpr int EPI_WAVE_BYTES = 32 * (WN * 4 + 16);
  static constexpr int LDS_BYTES = 2 * STAGE_BYTES > 4 * EPI_WAVE_BYTES ? 2 * STAGE_BYTES : 4 * EPI_WAVE_BYTES;
  static_assert(D % 2 == 0 && LDS_BYTES <= 64 * 1024, "stages");
  static_assert(P == 1 || P == D || P == 2 * D, "partial sums");
};

// The upper elements of v moved down by n elements, zeros above; nothing is left from 8 on.
__device__ __forceinline__ u32x4 shift_elements(u32x4 v, int n)
{
  const bool s4 = n & 4, s2 = n & 2, s1 = n & 1, s8 = n >= 8;
  v = s4 ? u32x4{v[2], v[3], 0u, 0u} : v;
  v = s2 ? u32x4{v[1], v[2], v[3], 0u} : v;
  v = s1 ? u32x4{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16), v[3] >> 16} : v;
  return s8 ? u32x4{0u, 0u, 0u, 0u} : v;
}

// One operand's chunks of a thread: load i of k-tile kt is the chunk `col` of LDS row r + i * RSTEP.
template <class O, class HW>
struct DirectOperand {
  const char* base;            // the tile's first row or column
  uint32_t off[O::NL];         // bytes from there to load i of k-tile 0
  int r, col;                  // first LDS row; first element of the chunk within its row
  int K, ld;
  int back;                    // M/N-contiguous: elements that the chunk starts early in the last row
  bool edge;                   // ... in a tile whose chunks may reach past a row's end

  __device__ __forceinline__ void setup(const void* ptr, int t, int extent, int ld_, int K_, int q0)
  {
    K = K_;
    ld = ld_;
    r = q0 / O::CPR;
    col = ((q0 % O::CPR) ^ O::template swz<HW>(r)) * 8;
    const int left = extent - t * O::BX;
    back = 0;
    edge = false;
    if constexpr (O::LAY == LAY_K) {
      base = (const char*)ptr + (long)t * O::BX * ld * 2;
#pragma unroll
      for (int i = 0; i < O::NL; i++) {
        const int row = r + i * O::RSTEP;                   // rows past the last read it
        off[i] = (uint32_t)((row < left ? row : left - 1) * ld) * 2u;
      }
    } else {
      base = (const char*)ptr + (long)t * O::BX * 2;
      edge = left < O::BX;
      const int c = col < left ? col : 0;                   // chunks wholly past a row's end read its first
      back = c > left - 8 ? c - (left - 8) : 0;
#pragma unroll
      for (int i = 0; i < O::NL; i++) off[i] = (uint32_t)((r + i * O::RSTEP) * ld + c) * 2u;
    }
  }
  __device__ __forceinline__ void load(int kt, bool last, u32x4 (&v)[O::NL]) const
  {
    const int k0 = kt * O::BK;
    if constexpr (O::LAY == LAY_K) {
      const int at = k0 + col < K - 8 ? k0 + col : K - 8;
#pragma unroll
      for (int i = 0; i < O::NL; i++) v[i] = HW::global_load16_any(base + (off[i] + (uint32_t)at * 2u));
    } else {
      const char* b = base + (long)k0 * ld * 2;
      const int rows = K - k0 < O::BK ? K - k0 : O::BK;     // rows past the last read it
#pragma unroll
      for (int i = 0; i < O::NL; i++) {
        const int row = r + i * O::RSTEP, over = row < rows ? 0 : row - (rows - 1);
        v[i] = HW::global_load16_any(b + (long)(int)(off[i] - (uint32_t)((over * ld + (last ? back : 0)) * 2)));
      }
    }
  }
  // zeros for what the chunks of the last k-tile hold past K (and past the last row's end)
  __device__ __forceinline__ void trim(int kt, u32x4 (&v)[O::NL]) const
  {
    const int k0 = kt * O::BK;
#pragma unroll
    for (int i = 0; i < O::NL; i++) {
      int n;
      if constexpr (O::LAY == LAY_K)
        n = k0 + col < K - 8 ? 0 : k0 + col - (K - 8);
      else
        n = k0 + r + i * O::RSTEP < K ? back : 8;
      v[i] = shift_elements(v[i], n);
    }
  }
  __device__ __forceinline__ void store(uint32_t dst, int q0, const u32x4 (&v)[O::NL]) const
  {
#pragma unroll
    for (int i = 0; i < O::NL; i++) HW::lds_write(dst + (uint32_t)(q0 + i * O::NT) * 16u, v[i]);
  }
};

template <class C, class HW>
__global__ void __launch_bounds__(C::NT, C::P > 1 ? 2 : 1) alcop_direct(const DirectArgs s)
{
  constexpr int BM = C::BM, BN = C::BN, WM = C::WM, WN = C::WN, TM = C::TM, TN = C::TN;
  using OA = typename C::OA;
  using OB = typename C::OB;
  Params p = {};
  p.C = s.C;
  p.M = p.Mv = s.M;
  p.N = p.Nv = s.N;
  p.ldc = s.ldc;
  p.alpha = s.alpha;
  p.bias = s.bias;
  p.out_dtype = s.flags & 3;
  p.act = (s.flags >> 2) & 1;
  p.raster = (s.flags >> 3) & 1;
  p.c_any = (s.flags >> 4) & 1;
  p.ntm = (s.M + BM - 1) / BM;
  p.ntn = (s.N + BN - 1) / BN;
  p.group_m = p.ntm < 8 ? p.ntm : 8;
  const uint32_t lds0 = HW::lds_base();
  const int lane = HW::lane_id();
  const int wave = HW::wave_id();
  const int wm = wave & 1, wn = wave >> 1;
  const int q0 = wave * 64 + lane;
  int tm, tn;
  tile_of_block(p, HW::block_x(), tm, tn);

  const int nko = (s.K + 63) / 64;
  DirectOperand<OA, HW> la;
  DirectOperand<OB, HW> lb;
  la.setup(s.A, tm, s.M, s.lda, s.K, q0);
  lb.setup(s.B, tn, s.N, s.ldb, s.K, q0);

  uint32_t rdA[OA::NRD], rdB[OB::NRD];
  setup_reader<OA, HW>(lane, wm, lds0, rdA);
  setup_reader<OB, HW>(lane, wn, lds0 + OA::BYTES, rdB);
  constexpr int D = C::D;
  u32x4 ra[D][OA::NL], rb[D][OB::NL];
  const bool trim = (s.K & 63) != 0 || la.edge || lb.edge;
  // k-tiles past the last one load the last again (their waits are those of every other)
  auto load = [&](int kt, int set) __attribute__((always_inline)) {
    const bool last = kt >= nko - 1;
    la.load(last ? nko - 1 : kt, last, ra[set]);
    lb.load(last ? nko - 1 : kt, last, rb[set]);
  };
  auto store = [&](int kt, int set, bool maybe_last) __attribute__((always_inline)) {
    if (maybe_last && trim && kt == nko - 1) {
      la.trim(kt, ra[set]);
      lb.trim(kt, rb[set]);
    }
    const uint32_t dst = lds0 + (uint32_t)((set & 1) * C::STAGE_BYTES);
    la.store(dst, q0, ra[set]);
    lb.store(dst + OA::BYTES, q0, rb[set]);
  };
#pragma unroll
  for (int d = 0; d < D; d++) load(d, d);
  HW::sched_fence();               // clearing the sums costs nothing while the loads are on their way
  constexpr int P = C::P;
  f32x16 sum[P][TN][TM];
#pragma unroll
  for (int q = 0; q < P; q++)
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int j = 0; j < TM; j++)
#pragma unroll
        for (int v = 0; v < 16; v++) sum[q][i][j][v] = 0.f;
  store(0, 0, true);
  HW::wait_lds();
  HW::block_barrier();
  auto multiply = [&](int set) __attribute__((always_inline)) {
    uint32_t curA[OA::NRD], curB[OB::NRD];
#pragma unroll
    for (int i = 0; i < OA::NRD; i++) curA[i] = rdA[i] + (uint32_t)((set & 1) * C::STAGE_BYTES);
#pragma unroll
    for (int i = 0; i < OB::NRD; i++) curB[i] = rdB[i] + (uint32_t)((set & 1) * C::STAGE_BYTES);
#pragma unroll
    for (int ki = 0; ki < 4; ki++) {
      const int q = P == 1 ? 0 : P == D ? set : 2 * set + ki / 2;
      u32x4 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < OA::NRI; i++) read_instr<OA, HW>(curA, ki, i, fa);
#pragma unroll
      for (int i = 0; i < OB::NRI; i++) read_instr<OB, HW>(curB, ki, i, fb);
#pragma unroll
      for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++) {
          f32x16& acc = sum[q][i][j];
          acc = HW::template mma<C::DT>(fb[i], fa[j], acc);
        }
    }
  };
  // No way out of this loop but its end: the compiler would wait for all loads at the loop's head.  The
  // k-tile stored last in a turn is the only one there that can be the last of all.
  int kt = 0;
  for (; kt + D < nko; kt += D) {
#pragma unroll
    for (int h = 0; h < D; h++) {
      load(kt + h + D, h);
      HW::sched_fence();
      multiply(h);
      store(kt + h + 1, (h + 1) % D, h == D - 1);   // its last readers passed the barrier before this k-tile
      HW::wait_lds();
      HW::block_barrier();
    }
  }
#pragma unroll
  for (int h = 0; h < D; h++) {
    multiply(h);
    if (kt + h + 1 >= nko) break;
    store(kt + h + 1, (h + 1) % D, true);
    HW::wait_lds();
    HW::block_barrier();
  }

#pragma unroll
  for (int d = P / 2; d > 0; d /= 2)
#pragma unroll
    for (int q = 0; q < d; q++)
#pragma unroll
      for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++)
#pragma unroll
          for (int v = 0; v < 16; v++) sum[q][i][j][v] += sum[q + d][i][j][v];

  // ---- epilogue: as in the pipelined loops; the bias one value at a time, from any address ----------
  const int m0 = tm * BM + wm * WM, n0 = tn * BN + wn * WN;
  const bool fused = p.alpha != 1.0f || p.bias != nullptr || p.act != 0;
  f32x4 bv[TN * 4];
#pragma unroll
  for (int g = 0; g < TN * 4; g++) bv[g] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (p.bias != nullptr) {
#pragma unroll
    for (int g = 0; g < TN * 4; g++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int n = n0 + 8 * g + 4 * (lane >> 5) + e;
        bv[g][e] = __builtin_bit_cast(float, HW::global_load_u32(p.bias + (n < p.N ? n : p.N - 1)));
      }
  }
  HW::wait_lds();
  HW::block_barrier();             // every wave has left the stages
  const uint32_t mine = lds0 + (uint32_t)(wave * C::EPI_WAVE_BYTES);
  auto epilogue = [&](auto zero) __attribute__((always_inline)) {
    using OT = decltype(zero);
    constexpr int OBY = sizeof(OT), RS = WN * OBY + 16, LPR = WN * OBY / 16, RPI = 64 / LPR;
#pragma unroll
    for (int j = 0; j < TM; j++) {
      park_band<OT, RS, HW>(p, sum[0], j, mine, lane, fused, n0, bv);
#pragma unroll
      for (int t = 0; t < 32 / RPI; t++) {
        const int r = t * RPI + lane / LPR, c16 = lane % LPR;
        const u32x4 v = HW::lds_read16(mine + r * RS + c16 * 16);
        const int m = m0 + j * 32 + r, n = n0 + c16 * (16 / OBY);
        if (m < p.Mv) store_chunk<OT, HW>(p, (char*)p.C + ((long)m * p.ldc + n) * OBY, n, v);
      }
    }
  };
  if (p.out_dtype == 2)
    epilogue(0.0f);
  else if (p.out_dtype == 0)
    epilogue((_Float16)0);
  else
    epilogue((__bf16)0);
}

}  // namespace alcop
