// Operands whose shape or placement the pipelined loops cannot take as they are: N or K not a
// multiple of 8, row pitches or base addresses that are not 16-byte aligned, a channel count such
// as 3.  The loops move 16-byte chunks (paper Sec. 4.2: the asynchronous copies of a pipeline
// stage; here one buffer_load_dwordx4 ... lds per lane), so such operands are first copied into a
// workspace with every extent rounded up to 8 elements and the tail zero-filled, and the ordinary
// kernels compute the product there; their epilogue stores the valid part of the result straight
// to C (Params::c_any).  Zero padding leaves every valid output element unchanged: the extra k
// terms are exact zeros.
//
// ONE launch copies all operands of a call (A and B, or x and w, and the bias): a call on odd
// sizes costs two launches.  With a launch per operand and a copy of C behind the product it was
// five, which is what a small product of that kind took its time for (1021 x 1531 x 767 bf16:
// 24.9 us, of which the product 6.9).
//
// Like the main loops, the kernel takes the hardware operations from a policy class.
#pragma once
#include <stdint.h>

#include "alcop_kernel.hip.h"

namespace alcop {

// What a segment's 16-byte chunks hold.
enum {
  PACK_MAT = 0,   // a matrix: rows of `cols` elements, zero beyond; rows may come in groups of rg
                  // of which the first nm (and the first nq groups) exist in the source
  PACK_PIX = 1,   // an image row as pixels of cg elements, 8 / cg to a chunk: cg = 1 or 2 channels, or 4 with 3
                  // or 4 channels (`chans`) and zeros; `pad` zero pixels before the first
  PACK_WIN = 2,   // an image row as one window of cu elements per output column: the `win` elements
                  // its filter row covers (all taps and channels, contiguous in the source)
};

struct PackSeg {
  const void* src;
  void* dst;
  int kind, esize;        // bytes per element: 2, or 4 (PACK_MAT only)
  uint32_t first;         // first block of this segment
  uint32_t chunks;        // 16-byte chunks in all: batch * rows_d * cpr
  FastDiv cpr, rows_d;    // chunks per destination row; destination rows per batch entry
  FastDiv rg;             // PACK_MAT: rows per group; PACK_WIN: chunks per window
  long s_batch, s_grp, s_row;   // source strides in elements: batch entry, row group, row
  long total;             // elements from the source's first to its last, and what lies between: what may be read; where
                          // gaps part the entries of a batch, minus those of one entry
  int nq, nm, cols;       // PACK_MAT: valid groups, rows of a group, columns
  int width, chans;       // PACK_PIX / PACK_WIN: pixels of a source row, channels
  int pad, cg, stride;    // ... zero pixels on the left; elements per pixel; columns per output
  int win;
};

constexpr int PACK_THREADS = 256;
constexpr int PACK_SEGS = 3;

struct PackParams {
  PackSeg seg[PACK_SEGS];
  int nseg;
};

// Elements [lo, hi) of the eight (four) at s that exist; the others are zero.
template <class HW>
__device__ __forceinline__ u32x4 load_chunk(const char* s, int esize, int lo, int hi)
{
  const int per = 16 / esize;
  if (lo <= 0 && hi >= per) return HW::global_load16_any(s);
  u32x4 v = {0u, 0u, 0u, 0u};
  if (esize == 2) {
#pragma unroll
    for (int e = 0; e < 8; e++)
      if (e >= lo && e < hi) v[e >> 1] |= (uint32_t)HW::global_load_u16(s + 2 * e) << (16 * (e & 1));
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (e >= lo && e < hi) v[e] = HW::global_load_u32(s + 4 * e);
  }
  return v;
}

// The eight 2-byte elements from element f of a source of `total` (0 <= f + 7 and f < total where any of them
// is kept): one load but for the chunks at the source's very ends.  What belongs to no row or window of the
// chunk is cleared afterwards (keep_elements): element by element, with a load each, a chunk of the 7 x 7
// stem's images cost eight loads (32 x 224 x 224 x 3 8.7 us and now 6.9; windows of 21 elements of
// 33 x 137 x 142 x 3 14.2 and 10.5).
template <class HW>
__device__ __forceinline__ u32x4 load_elements(const void* src, long f, long total)
{
  const char* s = (const char*)src + f * 2;
  if (f >= 0 && f + 8 <= total) return HW::global_load16_any(s);
  return load_chunk<HW>(s, 2, f < 0 ? (f < -8 ? 8 : (int)-f) : 0, total - f < 8 ? (total > f ? (int)(total - f) : 0) : 8);
}

// Elements [lo, hi) of v, zeros in place of the others.
__device__ __forceinline__ u32x4 keep_elements(u32x4 v, int lo, int hi)
{
#pragma unroll
  for (int d = 0; d < 4; d++)
    v[d] &= (2 * d >= lo && 2 * d < hi ? 0xffffu : 0u) | (2 * d + 1 >= lo && 2 * d + 1 < hi ? 0xffff0000u : 0u);
  return v;
}

// One thread writes one 16-byte chunk of one segment; the destinations are dense images.  Sources
// need element alignment only.
template <class HW>
__global__ void __launch_bounds__(PACK_THREADS) alcop_pack(const PackParams p)
{
  const uint32_t bx = HW::block_x();
  int k = 0;
  if (p.nseg > 1 && bx >= p.seg[1].first) k = 1;
  if (p.nseg > 2 && bx >= p.seg[2].first) k = 2;
  const PackSeg& g = p.seg[k];
  const uint32_t idx = (bx - g.first) * PACK_THREADS + (uint32_t)(HW::wave_id() * 64 + HW::lane_id());
  if (idx >= g.chunks) return;
  const uint32_t rr = g.cpr.div(idx);
  const uint32_t c = idx - rr * g.cpr.d;
  const uint32_t b = g.rows_d.div(rr);
  const uint32_t r = rr - b * g.rows_d.d;
  u32x4 v = {0u, 0u, 0u, 0u};
  if (g.kind == PACK_MAT) {
    const uint32_t q = g.rg.div(r);
    const uint32_t m = r - q * g.rg.d;
    if ((int)q < g.nq && (int)m < g.nm) {
      const int c0 = (int)c * (16 / g.esize);
      const long first = (long)b * g.s_batch;
      const long off = first + (long)q * g.s_grp + (long)m * g.s_row + c0;
      if (g.esize == 2)
        v = keep_elements(load_elements<HW>(g.src, off, g.total < 0 ? first - g.total : g.total), 0, g.cols - c0);
      else
        v = load_chunk<HW>((const char*)g.src + off * 4, 4, 0, g.cols - c0);
    }
  } else if (g.kind == PACK_WIN) {
    const uint32_t q = g.rg.div(c);
    const int e0 = (int)(c - q * g.rg.d) * 8;
    const int f = ((int)q * g.stride - g.pad) * g.chans + e0;         // element of the image row
    const int end = g.width * g.chans - f;                            // elements left in the row
    const int hi = (g.win - e0) < end ? (g.win - e0) : end;
    if (f > -8 && hi > 0) v = keep_elements(load_elements<HW>(g.src, (long)r * g.s_row + f, g.total), -f, hi);
  } else {
    const int px = 8 / g.cg;
    const int iw = (int)c * px - g.pad;                               // the chunk's first pixel
    if (iw > -px && iw < g.width) {
      v = load_elements<HW>(g.src, (long)r * g.s_row + (long)iw * g.chans, g.total);
      if (g.cg == 4 && g.chans == 3)
        v = u32x4{v[0], v[1] & 0xffffu, (v[1] >> 16) | (v[2] << 16), v[2] >> 16};
      v = keep_elements(v, -iw * g.cg, (g.width - iw) * g.cg);
    }
  }
  HW::global_store16_keep((char*)g.dst + (size_t)idx * 16, v);
}

// C from a dense image of it, for rows of C further apart than the products can address: one element
// per thread.  For completeness, not for speed.
struct CopyOutParams {
  const void* src;
  void* dst;
  int batch, rows, cols, esize;      // bytes per element: 2 or 4
  long s_row, s_batch, d_row, d_batch;   // in elements
};

template <class HW>
__global__ void __launch_bounds__(PACK_THREADS) alcop_copy_out(const CopyOutParams p)
{
  const long i = (long)HW::block_x() * PACK_THREADS + HW::wave_id() * 64 + HW::lane_id();
  const long r = i / p.cols, c = i - r * p.cols;
  const long b = r / p.rows, m = r - b * p.rows;
  if (b >= p.batch) return;
  const char* s = (const char*)p.src + (b * p.s_batch + m * p.s_row + c) * p.esize;
  char* d = (char*)p.dst + (b * p.d_batch + m * p.d_row + c) * p.esize;
  if (p.esize == 2)
    HW::global_store_u16(d, HW::global_load_u16(s));
  else
    HW::global_store_u32(d, HW::global_load_u32(s));
}

inline unsigned copy_out_blocks(const CopyOutParams& p)
{
  return (unsigned)(((long)p.batch * p.rows * p.cols + PACK_THREADS - 1) / PACK_THREADS);
}

}  // namespace alcop
