// Convolution with the input patch of a tile resident in LDS, any geometry (schedule variant 4).
//
// What bounds the gathering kernels.  They bring every k-tile of A from L2 into the LDS ring: an
// R x S filter fetches each input pixel R * S times, at the 40 to 58 bytes per clock and compute
// unit that path delivers.  Here the pixels a tile's windows cover are loaded once, filter taps are
// formed by the address of the LDS read, and only the weights stream through the ring: per tile of
// 128 x 64 with a 3 x 3 filter over 256 channels 100 + 295 KB instead of 590 + 295.
//
// Positions.  The images lie one after the other as rows of Ws = W + pad_w positions, Hs = H + pad_h
// rows each: the right padding of a row is the left padding of the next, the bottom padding of an
// image the top padding of the next.  Output pixel (n, p, q) reads position
// (n Hs + p stride_h) Ws + q stride_w, filter tap (r, s) the one r dil_h Ws + s dil_w further.  A tile
// is BM consecutive output pixels, as in the gathering kernels, so no position is computed that is
// not stored; its patch runs from the first pixel's position to the last one's plus the halo.
//
// LDS image.  A position takes an odd number of 16-byte chunks (C / 8, or one more that stays zero),
// so the 16 lanes of a read clock, which want the same chunk of 16 consecutive positions, hit 16
// different bank groups without a swizzle, and the address of a read is a sum: position of the
// lane's row + offset of (tap, channels).  The second term is the same for all rows; a table in LDS
// holds it for every 8 elements of K, which covers any channel count, dilation, and windows that
// overlap (cPix < cC).  A chunk past K points at a slot of zeros.
//
// Ragged windows (RG).  Where several pixels share a chunk, the last chunk of a filter row may hold
// pixels past the window.  They are data of other windows and meet weights of zero, which is not
// enough: 0 * inf.  The second half of those chunks is cleared in the fragments before their first use,
// with a mask that the table holds beside the offset: per 16 elements of K four vector instructions
// beside four matrix instructions, 0.5 us of the 33 that the call on the stem below takes.
//
// Waves.  Every wave owns a 64 x 64 tile (4 waves of 64 x 64 read 96 clocks of LDS per 128 of
// matrix instructions; 32-wide wave tiles are bound by those reads).  Tiles smaller than 256 x 64 or
// 128 x 128 split each ring stage, WK k-tiles of 64 deep, among WK waves; the fp32 tiles are added
// in wave order at the end.
//
// What it measured, against the best gathering kernel: 7 x 7 RGB stem of 32 x 224 x 224 27.7 us against
// 35 (per block 1070 vector instructions a wave, half of them prologue and epilogue, bound it; the
// stores of C alone take 9.3), 2368 x 256 x 7200 (5 x 5, 288 channels) 24.3 against 41.6, 12005 x 64 x
// 1728 10.6 against 12.1.  A stage of 16 matrix instructions per wave takes 0.34 us (256 x 64), 0.15 of it
// waiting for LDS; a block-wide load of the patch (4 KB) 0.13 us, which nothing of the same block
// overlaps: with 256 channels and few tiles the gather stays ahead (14 x 14 x 256: 13.5 against 14.7).
//
// Pipeline: the fused two-level loop of alcop_kernel.hip.h (paper Sec. 4.2, Fig. 3(d)) with the patch
// as one more load in front of the prologue.
#pragma once
#include "alcop_kernel.hip.h"

namespace alcop {

template <int DT_, int BM_, int BN_, int S_, int BL_, int RG_ = 0>
struct RCfg {
  static constexpr int DT = DT_, BM = BM_, BN = BN_, BK = 64, S = S_, BL = BL_, RG = RG_;
  static constexpr int WAVES_M = BM / 64, WAVES_N = BN / 64, WK = 4 / (WAVES_M * WAVES_N);
  static constexpr int NT = 256;
  using OB = Opnd<BL ? LAY_K : LAY_MN, BN, 64, 64, NT>;
  static constexpr int SUB_BYTES = OB::BYTES;                    // one k-tile of B
  static constexpr int STAGE_BYTES = WK * SUB_BYTES;
  static constexpr int RING_BYTES = S * STAGE_BYTES;             // the patch follows, then the table
  static constexpr int L = WK * OB::NL;                          // loads per thread and stage
  static constexpr int WAIT = (S - 2) * L;
  static constexpr int RS = 64 * 4 + 16;                         // row stride of a parked fp32 wave tile
  static constexpr int EPI_WAVE_BYTES = (WK > 1 ? 64 : 32) * RS;
  static constexpr int MIN_LDS = RING_BYTES > 4 * EPI_WAVE_BYTES ? RING_BYTES : 4 * EPI_WAVE_BYTES;
  static_assert(WAVES_M * WAVES_N * WK == 4, "four waves of 64 x 64");
  static_assert(S >= 2 && S <= 4 && WAIT <= 63, "ring");
};

// Entries of the chunk table: 8 elements of K each, for every k-tile of the ring's stages and one
// stage more (the fused pipeline reads ahead), whole block-wide writes.
inline int convres_table(int K, int wk)
{
  const int stages = ((K + 63) / 64 + wk - 1) / wk;
  return ((stages + 1) * wk * 8 + 255) / 256 * 256;
}
inline long convres_lds(long ring, long min_lds, long loads, long table, bool ragged)
{
  const long need = ring + loads * 4096 + table * (ragged ? 8 : 4);
  return need > min_lds ? need : min_lds;
}

// Ragged windows are few-channel stems: their patches are small (50 KB of LDS per block of the one below), and
// three blocks share a compute unit where the registers allow it, 131 of them instead of 188: 32 x 224 x 224 x 3
// 7 x 7 32.6 -> 32.1 us.  Elsewhere the patch leaves room for one or two blocks.
template <class C, class HW>
__global__ void __launch_bounds__(C::NT, C::RG ? 3 : 1) alcop_convres(const Params p)
{
  constexpr int BM = C::BM, BN = C::BN, S = C::S, WK = C::WK;
  using OB = typename C::OB;
  const uint32_t lds0 = HW::lds_base();
  const int lane = HW::lane_id();
  const int wave = HW::wave_id();
  const int wm = wave % C::WAVES_M, wn = (wave / C::WAVES_M) % C::WAVES_N, wk = wave / (C::WAVES_M * C::WAVES_N);
  const int q0 = wave * 64 + lane;
  int tm, tn;
  tile_of_block(p, HW::block_x(), tm, tn);

  const int nko = (p.K + 63) / 64;             // k-tiles
  const int nst = (nko + WK - 1) / WK;         // ring stages
  const bool ktail = (p.K % 64) != 0;

  auto position = [&](int m) __attribute__((always_inline)) {
    const int img = (int)p.rPQ.div((uint32_t)m);
    const int pq = m - img * (p.cP * p.cQ);
    const int pp = (int)p.rQ.div((uint32_t)pq);
    return (img * p.rHs + pp * p.csh) * p.rWs + (pq - pp * p.cQ) * p.csw;
  };
  const int pos0 = position(tm * BM);

  // ---- patch: slot q holds chunk q % CP of position pos0 + q / CP ------------------------------
  const uint32_t patch = lds0 + C::RING_BYTES;
  const auto rsA = HW::make_rsrc(p.A, (int)p.a_span);
  {
    // A lane's slots are 256 apart: chunk, column, row and the row's byte offset in x step along with
    // them (three divisions per slot cost 2.4 us of a 100 KB patch).
    int d = (int)p.rCP.div((uint32_t)q0), c = q0 - d * (int)p.rCP.d;
    const int j = pos0 + d;
    const int img = (int)p.rImg.div((uint32_t)j);
    const int rem = j - img * (p.rHs * p.rWs);
    int row = (int)p.rWsDiv.div((uint32_t)rem), col = rem - row * p.rWs;
    const uint32_t rowb = (uint32_t)(p.cW * p.cPix) * 2u;        // bytes of a row of x
    uint32_t base = (uint32_t)(img * p.cH + row - p.cph) * rowb;
    const uint32_t step_b = (uint32_t)p.rstep_row * rowb, img_b = (uint32_t)p.cph * rowb;
    int q = q0;
    uint32_t dst = patch + (uint32_t)wave * 1024u;
    for (int i = 0; i < p.rloads; i++) {
      const int ih = row - p.cph, iw = col - p.cpw;
      const bool ok = q < p.rslots && c < p.rc8 && (unsigned)ih < (unsigned)p.cH && (unsigned)iw < (unsigned)p.cW;
      const uint32_t off = base + (uint32_t)(iw & 0xffffff) * (uint32_t)(p.cPix & 0xffff) * 2u + (uint32_t)c * 16u;
      HW::dma16(rsA, ok ? off : 0x80000000u, dst);
      q += C::NT;
      dst += C::NT * 16u;
      c += p.rstep_c;
      col += p.rstep_col;
      row += p.rstep_row;
      base += step_b;
      if (c >= (int)p.rCP.d) {
        c -= (int)p.rCP.d;
        col++;
      }
      if (col >= p.rWs) {
        col -= p.rWs;
        row++;
        base += rowb;
      }
      while (row >= p.rHs) {
        row -= p.rHs;
        base -= img_b;                         // the next image's first row follows ph rows earlier
      }
    }
  }

  // ---- ring of weights ---------------------------------------------------------------------------
  const LoadState<HW> lb = setup_loader<OB, HW>(p.B, tn, p.N, p.ldb, p.K, nko, q0);
  int st_kt = 0;
  uint32_t st_dst = 0;
  auto stage_begin = [&](int kt, int slot) __attribute__((always_inline)) {
    st_kt = kt;
    st_dst = lds0 + (uint32_t)slot * C::STAGE_BYTES + (uint32_t)wave * 1024u;
  };
  auto issue_one = [&](int idx) __attribute__((always_inline)) {
    const int w = idx / OB::NL, i = idx % OB::NL;
    const int k = st_kt * WK + w;
    const uint32_t vo = (ktail && k == nko - 1) ? lb.voff_t : lb.voff;
    const uint32_t kb = k < nko ? (uint32_t)k * lb.kstep : 0x80000000u;
    HW::dma16(lb.rsrc, vo + kb + (uint32_t)i * lb.step, st_dst + w * C::SUB_BYTES + i * 4096);
  };
#pragma unroll
  for (int s = 0; s < S - 1; s++) {
    stage_begin(s, s);
#pragma unroll
    for (int i = 0; i < C::L; i++) issue_one(i);
  }

  // ---- chunk table ---------------------------------------------------------------------------------
  const uint32_t tab = patch + (uint32_t)p.rloads * 4096u;
  for (int e = 0; e < p.rtab; e += C::NT) {
    const int kc = e + q0;
    const int tap = (int)p.rC8.div((uint32_t)kc);
    const int r = (int)p.rS.div((uint32_t)tap);
    const int cc = kc - tap * (int)p.rC8.d;
    const uint32_t off = kc * 8 < p.K ? (uint32_t)(cc * 16 + (tap - r * p.cS) * p.rdS + r * p.rdR) : 0x80000000u;
    if constexpr (C::RG)
      HW::lds_write(tab + (uint32_t)kc * 8u, u32x2{off, cc == (int)p.rC8.d - 1 ? 0u : ~0u});
    else
      HW::lds_write(tab + (uint32_t)kc * 4u, off);
  }

  // ---- readers ---------------------------------------------------------------------------------------
  uint32_t rdB[OB::NRD], curB[OB::NRD], rdA[2];
  setup_reader<OB, HW>(lane, wn, (uint32_t)wk * C::SUB_BYTES, rdB);
#pragma unroll
  for (int t = 0; t < 2; t++) {
    const int m = tm * BM + wm * 64 + t * 32 + (lane & 31);      // rows past M read the tile's first
    rdA[t] = patch + (uint32_t)((position(m < p.M ? m : tm * BM) - pos0) * p.rpitch);
  }
  const uint32_t zeros = patch + (uint32_t)p.rslots * 16u;       // the patch has rslots + 1 slots at least
  constexpr uint32_t TE = C::RG ? 8u : 4u;     // bytes per table entry
  const uint32_t tabw = tab + (uint32_t)(wk * 8 + (lane >> 5)) * TE;
  uint32_t oc[4], on[4], mc[4], mn[4];         // offsets; RG: masks of the chunks' second halves
  auto read_offsets = [&](int kt, uint32_t (&o)[4], uint32_t (&mask)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int ki = 0; ki < 4; ki++) {
      const uint32_t at = tabw + (uint32_t)(kt * (WK * 8) + ki * 2) * TE;
      if constexpr (C::RG) {
        const u32x2 v = HW::lds_read8(at);
        o[ki] = v[0];
        mask[ki] = v[1];
      } else {
        o[ki] = HW::lds_read4(at);
      }
    }
  };
  constexpr int NRI = 2 + OB::NRI;
  u32x4 fa[2][2], fb[2][2];
  auto read_one = [&](int ki, int r, uint32_t o, u32x4 (&a)[2], u32x4 (&b)[2]) __attribute__((always_inline)) {
    if (r < 2)
      a[r] = HW::lds_read16((int)o < 0 ? zeros : rdA[r] + o);
    else
      read_instr<OB, HW>(curB, ki, r - 2, b);
  };
  auto open_slot = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < OB::NRD; i++) curB[i] = lds0 + (uint32_t)slot * C::STAGE_BYTES + rdB[i];
  };

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  HW::template wait_vm<C::WAIT>();             // the patch and stage 0 have landed (this wave's part)
  HW::wait_lds();
  HW::block_barrier();
  read_offsets(0, oc, mc);
  open_slot(0);
#pragma unroll
  for (int r = 0; r < NRI; r++) read_one(0, r, oc[0], fa[0], fb[0]);
  HW::sched_fence();
  int rslot = 0, wslot = S - 1;
  for (int kt = 0; kt < nst; kt++) {
    stage_begin(kt + S - 1, wslot);
    wslot = (wslot + 1 == S) ? 0 : wslot + 1;
#pragma unroll
    for (int ki = 0; ki < 4; ki++) {
      if (ki == 0) read_offsets(kt + 1, on, mn);
      const uint32_t mask = C::RG ? mc[ki] : 0u;   // step 3 moves on to the next stage's masks
#pragma unroll
      for (int m = 0; m < 4; m++) {
        const int i = m >> 1, j = m & 1;
        if constexpr (C::RG) {
          if (m < 2) {                         // the first use of fragment m
            fa[ki & 1][m][2] &= mask;
            fa[ki & 1][m][3] &= mask;
          }
        }
        acc[i][j] = HW::template mma<C::DT>(fb[ki & 1][i], fa[ki & 1][j], acc[i][j]);
        if (ki < 3) {
#pragma unroll
          for (int r = 2 * m; r < 2 * m + 2 && r < NRI; r++)
            read_one(ki + 1, r, oc[(ki + 1) & 3], fa[(ki + 1) & 1], fb[(ki + 1) & 1]);
          // the stage's loads, spread over the first three steps
          const int t = ki * 4 + m;
#pragma unroll
          for (int d = t * C::L / 12; d < (t + 1) * C::L / 12; d++) issue_one(d);
        } else {
          if (m == 0) {
            HW::template wait_vm<C::WAIT>();   // consumer_wait: stage kt+1 has landed (this wave)
            HW::wait_lds();                    // consumer_release: my reads of stage kt are done
            HW::block_barrier();
            rslot = (rslot + 1 == S) ? 0 : rslot + 1;
            open_slot(rslot);
#pragma unroll
            for (int e = 0; e < 4; e++) {
              oc[e] = on[e];
              if (C::RG) mc[e] = mn[e];
            }
          }
#pragma unroll
          for (int r = 2 * m; r < 2 * m + 2 && r < NRI; r++) read_one(0, r, oc[0], fa[0], fb[0]);
        }
        HW::sched_fence();
      }
    }
  }

  // ---- epilogue ------------------------------------------------------------------------------------
  const bool fused = p.alpha != 1.0f || p.bias != nullptr || p.act != 0;
  const int n0 = tn * BN, m0 = tm * BM;
  f32x4 bv[8];
  if (WK == 1 && fused) load_bias<8, HW>(p, n0 + wn * 64, lane, bv);
  HW::template wait_vm<0>();                   // the loads that fetch nothing still write LDS
  HW::wait_lds();
  HW::block_barrier();                         // every wave has left the ring and the patch
  const uint32_t mine = lds0 + (uint32_t)wave * C::EPI_WAVE_BYTES;
  if constexpr (WK > 1) {
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int vq = 0; vq < 4; vq++)
          HW::lds_write(mine + (uint32_t)((j * 32 + (lane & 31)) * C::RS + (i * 32 + 8 * vq + 4 * (lane >> 5)) * 4),
                        f32x4{acc[i][j][4 * vq + 0], acc[i][j][4 * vq + 1], acc[i][j][4 * vq + 2], acc[i][j][4 * vq + 3]});
    HW::wait_lds();
    HW::block_barrier();
  }
  auto epilogue = [&](auto zero) __attribute__((always_inline)) {
    using OT = decltype(zero);
    constexpr int OBY = sizeof(OT), PER = 16 / OBY;
    typedef OT otv __attribute__((ext_vector_type(PER)));
    if constexpr (WK > 1) {
      constexpr int GPR = BN / PER;            // 16-byte chunks of C per row
      const float floor = p.act == 1 ? 0.f : -__builtin_inff();
#pragma unroll
      for (int g0 = 0; g0 < BM * GPR; g0 += C::NT) {
        const int g = g0 + q0;
        const int row = g / GPR, col = (g % GPR) * PER;
        const int w = row / 64 + C::WAVES_M * (col / 64);
        const uint32_t src = lds0 + (uint32_t)(w * C::EPI_WAVE_BYTES + (row % 64) * C::RS + (col % 64) * 4);
        const int n = n0 + col;
        otv h;
#pragma unroll
        for (int e4 = 0; e4 < PER / 4; e4++) {
          f32x4 b = {0.f, 0.f, 0.f, 0.f};
          if (p.bias != nullptr) b = HW::global_load_f32x4(p.bias + (n + 4 * e4 < p.N ? n + 4 * e4 : 0));
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < WK; k++) {
            const f32x4 f = __builtin_bit_cast(
                f32x4, HW::lds_read16(src + (uint32_t)(k * (4 / WK) * C::EPI_WAVE_BYTES + e4 * 16)));
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] += f[e];
          }
#pragma unroll
          for (int e = 0; e < 4; e++) {
            float t = v[e];
            if (fused) {
              t = t * p.alpha + b[e];
              t = t < floor ? 0.f : t;
            }
            h[e4 * 4 + e] = HW::template cvt<OT>(t);
          }
        }
        if (m0 + row < p.Mv)
          store_chunk<OT, HW>(p, (char*)p.C + ((long)(m0 + row) * p.ldc + n) * OBY, n, __builtin_bit_cast(u32x4, h));
      }
    } else {
      constexpr int RSB = 64 * OBY + 16, LPR = 64 * OBY / 16, RPI = 64 / LPR;
#pragma unroll
      for (int j = 0; j < 2; j++) {
        park_band<OT, RSB, HW>(p, acc, j, mine, lane, fused, n0 + wn * 64, bv);
#pragma unroll
        for (int t = 0; t < 32 / RPI; t++) {
          const int r = t * RPI + lane / LPR, c16 = lane % LPR;
          const u32x4 v = HW::lds_read16(mine + r * RSB + c16 * 16);
          const int m = m0 + wm * 64 + j * 32 + r, n = n0 + wn * 64 + c16 * PER;
          if (m < p.Mv) store_chunk<OT, HW>(p, (char*)p.C + ((long)m * p.ldc + n) * OBY, n, v);
        }
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
