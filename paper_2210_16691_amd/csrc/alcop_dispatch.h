// Which kernel a product without an explicit schedule gets: measured costs of a few kernels.
//
// The static model of Table 1 ranks hundreds of schedules for a tuner that times the best of them.
// Taken at its word, its first choice was 28 % slower than the best schedule in the mean over 243
// products of the kinds this library serves (linear layers and their gradients, attention; 1 to
// 8192 rows, K from 32 to 8192, fp16 and bf16, every layout; a tenth of them more than 60 %): it
// does not know the per-tile cost of a block, that persistent kernels whose consumers restart
// their register pipeline per k-tile are the faster ones, or the kernels whose waves split K.
//
// So the library measured every kernel on those products and fits, per kernel,
//     us = a + b * turns * k-tiles + c * turns + d * (bytes of A, B and C at 5.1 TB/s)
// with turns = ceil(tiles / 256), the tiles one compute unit works through in a row (least squares
// of the relative error, no negative coefficient); k-tiles are those of one wave where the waves
// split K.  a is the launch and the first loads, b the pace of the main loop (a 128 x 128 x 64
// step 0.30 us, 64 x 64 x 64 0.17 us), c the epilogue and restart of a tile.  The estimates are within
// 15 % for nine products in ten.  The kernels below are the ones that a greedy selection by the regret of
// the estimated best keeps; with them it is 4 % in the mean, 15 % at the 90th percentile.
#pragma once
#include <algorithm>

#include "../../include/alcop.h"

namespace alcop {

struct MeasuredCost {
  alcop_sched s;
  int waves_k;         // waves a tile's k-tiles are divided among
  double a, b, c, d;
};

inline const MeasuredCost kMeasured[] = {
    // waves split K: while there are fewer 64 x 64 tiles than compute units
    {{16, 16, 64, 16, 16, 2, 1, 0, 1, 0, 3}, 8, 2.10, 0.329, 0.72, 0.45},
    {{16, 32, 64, 16, 32, 2, 1, 0, 1, 0, 3}, 8, 1.23, 0.417, 1.69, 0.59},
    {{32, 32, 64, 32, 32, 2, 1, 0, 1, 0, 3}, 8, 1.23, 0.508, 2.05, 0.56},
    {{32, 64, 64, 32, 64, 2, 1, 0, 1, 0, 3}, 4, 1.47, 0.367, 2.09, 0.52},
    // persistent
    {{64, 64, 64, 32, 32, 3, 2, 0, 1, 0, 2}, 1, 2.51, 0.177, 0.45, 0.25},
    {{128, 128, 64, 64, 64, 3, 2, 0, 1, 0, 2}, 1, 2.46, 0.302, 1.01, 0.46},
    {{128, 128, 64, 64, 64, 2, 2, 0, 1, 0, 2}, 1, 2.28, 0.383, 0.82, 0.50},
    {{128, 64, 64, 64, 32, 3, 2, 0, 1, 0, 2}, 1, 2.38, 0.239, 0.82, 0.39},
    {{128, 64, 64, 64, 32, 2, 2, 0, 1, 0, 2}, 1, 2.47, 0.293, 0.60, 0.36},
    {{128, 128, 32, 64, 64, 3, 2, 0, 1, 0, 2}, 1, 2.20, 0.192, 1.01, 0.40},
    {{128, 192, 32, 64, 96, 3, 2, 0, 1, 0, 2}, 1, 1.28, 0.251, 2.52, 0.37},
    // tile at a time
    {{64, 64, 64, 32, 32, 3, 2, 1, 1, 0, 0}, 1, 2.60, 0.167, 0.37, 0.47},
    {{64, 64, 64, 32, 32, 4, 2, 1, 1, 0, 0}, 1, 2.39, 0.164, 0.62, 0.45},
    {{64, 64, 32, 32, 32, 4, 2, 1, 1, 0, 0}, 1, 2.60, 0.104, 0.30, 0.42},
    {{128, 128, 64, 64, 64, 4, 2, 1, 1, 0, 0}, 1, 1.60, 0.300, 2.29, 0.51},
    {{256, 128, 64, 128, 64, 3, 2, 1, 1, 0, 0}, 1, 0.93, 0.511, 4.02, 0.40},
    {{256, 256, 32, 128, 64, 3, 2, 1, 1, 0, 0}, 1, 0.00, 0.474, 4.60, 0.50},
    {{64, 128, 64, 32, 64, 4, 2, 1, 1, 0, 0}, 1, 1.63, 0.214, 1.75, 0.47},
    {{128, 64, 64, 64, 32, 4, 2, 1, 1, 0, 0}, 1, 1.62, 0.226, 1.70, 0.53},
};

inline double measured_us(const alcop_problem& p, const MeasuredCost& m)
{
  auto up = [](double x, double y) { return (double)(long)((x + y - 1) / y); };
  const double tiles = up(p.M, m.s.bm) * up(p.N, m.s.bn) * p.batch;
  const double turns = up(tiles, 256), kt = up(up(p.K, m.s.bk), m.waves_k);
  const double out = p.out == ALCOP_F32 ? 4.0 : 2.0;
  const double bytes = p.batch * (2.0 * p.M * p.K + 2.0 * p.K * p.N + out * p.M * p.N);
  return m.a + m.b * turns * kt + m.c * turns + m.d * bytes / 5.1e6;
}

// The measured kernels worth considering for a product: small tiles cost more bytes per flop, so the
// kernels whose waves split K are compared only while 64 x 64 tiles leave compute units idle (with 384
// such tiles, 1021 x 1536 x 768, they take 11.9 us at best against 6.2).
inline bool measured_applies(const alcop_problem& p, const MeasuredCost& m)
{
  if (p.op == ALCOP_OP_CONV2D) return false;
  return m.s.variant != 3 || (double)((p.M + 63) / 64) * ((p.N + 63) / 64) * p.batch <= 256;
}

// Convolutions.  The same fit over 200 convolutions (1 x 1, 3 x 3, 5 x 5; 7 to 112 wide images; 16 to
// 512 channels; strides 1 and 2; fp16 and bf16, both weight layouts), with the loader of A as part of the
// kernel: the gather that tracks the tap of every chunk (channel counts the k-tile does not divide)
// costs more per k-tile.  Bytes are those of M * C input elements, the weights and C.  The kernels with
// a resident patch of any geometry instead have
//     us = a + b * turns * stages + c * turns + d * turns * (block-wide loads of the patch).
// The model's first choice was 30 % above the best kernel in the mean (most where few tiles leave
// compute units idle: 20 x 32 x 2400 20.4 us against 6.0, and where a patch saves eight of nine reads
// of A: 100352 x 64 x 576 19.1 against 12.2); the cheapest of these is 2 %.
struct MeasuredConv {
  alcop_sched s;
  int am;              // loader of A: 1 tap per k-tile, 2 tap per chunk, 3 patch, 4 patch of any geometry
  int waves_k;         // waves a tile's k-tiles are divided among
  double a, b, c, d;
};

inline const MeasuredConv kMeasuredConv[] = {
    // the waves of a block split the reduction axis: few output tiles
    {{32, 32, 64, 32, 32, 2, 1, 0, 1, 0, 3}, 1, 8, 1.51, 0.676, 2.53, 0.19},
    {{32, 32, 64, 32, 32, 2, 1, 0, 1, 0, 3}, 2, 8, 1.66, 0.661, 3.12, 0.00},
    {{16, 32, 64, 16, 32, 2, 1, 0, 1, 0, 3}, 1, 8, 1.56, 0.516, 2.03, 0.10},
    {{16, 32, 64, 16, 32, 2, 1, 0, 1, 0, 3}, 2, 8, 1.63, 0.491, 2.58, 0.00},
    {{32, 64, 64, 32, 64, 2, 1, 0, 1, 0, 3}, 1, 4, 1.57, 0.548, 3.07, 0.04},
    {{32, 64, 64, 32, 64, 2, 1, 0, 1, 0, 3}, 2, 4, 1.53, 0.584, 3.51, 0.00},
    {{16, 16, 64, 16, 16, 2, 1, 0, 1, 0, 3}, 1, 8, 3.21, 0.342, 0.92, 0.00},
    {{16, 16, 64, 16, 16, 2, 1, 0, 1, 0, 3}, 2, 8, 3.25, 0.313, 1.30, 0.00},
    // tile at a time, gathering A
    {{128, 64, 32, 64, 32, 4, 2, 1, 1, 0, 0}, 1, 1, 3.42, 0.188, 0.51, 0.06},
    {{128, 64, 32, 64, 32, 4, 2, 1, 1, 0, 0}, 2, 1, 3.75, 0.196, 0.71, 0.00},
    {{128, 64, 64, 64, 32, 3, 2, 1, 1, 0, 0}, 1, 1, 3.08, 0.293, 1.07, 0.03},
    {{128, 64, 64, 64, 32, 3, 2, 1, 1, 0, 0}, 2, 1, 3.55, 0.352, 1.12, 0.02},
    {{64, 64, 32, 32, 32, 3, 2, 1, 1, 0, 0}, 1, 1, 3.34, 0.119, 0.29, 0.00},
    {{64, 64, 32, 32, 32, 3, 2, 1, 1, 0, 0}, 2, 1, 3.99, 0.142, 0.00, 0.00},
    {{128, 128, 32, 64, 64, 3, 2, 1, 1, 0, 0}, 1, 1, 3.70, 0.239, 0.60, 0.35},
    {{128, 128, 32, 64, 64, 3, 2, 1, 1, 0, 0}, 2, 1, 4.26, 0.267, 0.77, 0.00},
    {{64, 64, 64, 32, 32, 3, 2, 1, 1, 0, 0}, 1, 1, 3.41, 0.184, 0.53, 0.06},
    {{64, 64, 64, 32, 32, 3, 2, 1, 1, 0, 0}, 2, 1, 3.66, 0.217, 0.37, 0.00},
    {{256, 128, 64, 128, 64, 3, 2, 1, 1, 0, 0}, 1, 1, 0.00, 0.660, 6.17, 0.09},
    {{64, 128, 32, 32, 64, 2, 1, 0, 1, 0, 0}, 1, 1, 3.88, 0.196, 0.00, 0.00},
    {{128, 128, 64, 64, 64, 3, 2, 1, 1, 0, 0}, 1, 1, 1.11, 0.394, 3.26, 0.10},
    {{128, 128, 64, 64, 64, 3, 2, 1, 1, 0, 0}, 2, 1, 1.18, 0.500, 3.64, 0.18},
    {{64, 64, 64, 32, 32, 2, 1, 0, 1, 0, 0}, 1, 1, 3.88, 0.221, 0.22, 0.07},
    {{64, 64, 64, 32, 32, 2, 1, 0, 1, 0, 0}, 2, 1, 3.92, 0.248, 0.01, 0.00},
    {{128, 128, 64, 64, 64, 1, 1, 0, 1, 0, 0}, 1, 1, 4.64, 0.638, 0.05, 0.12},
    {{128, 128, 64, 64, 64, 1, 1, 0, 1, 0, 0}, 2, 1, 4.20, 0.679, 0.12, 0.05},
    {{128, 64, 32, 64, 32, 3, 2, 1, 1, 0, 0}, 1, 1, 3.40, 0.194, 0.44, 0.03},
    {{128, 64, 32, 64, 32, 3, 2, 1, 1, 0, 0}, 2, 1, 3.65, 0.191, 0.63, 0.07},
    // persistent, gathering A
    {{64, 128, 64, 32, 64, 4, 2, 1, 1, 0, 2}, 1, 1, 2.66, 0.258, 1.39, 0.00},
    // input patch resident, one k-tile per tap
    {{256, 64, 64, 64, 64, 3, 2, 1, 1, 0, 1}, 3, 1, 2.65, 0.390, 2.51, 0.00},
    {{128, 64, 32, 64, 32, 3, 2, 1, 1, 0, 1}, 3, 1, 3.61, 0.145, 0.43, 0.14},
    {{64, 64, 32, 32, 32, 3, 2, 1, 1, 0, 1}, 3, 1, 3.15, 0.113, 0.40, 0.00},
    {{256, 64, 32, 64, 64, 4, 2, 1, 1, 0, 1}, 3, 1, 3.95, 0.210, 0.92, 0.27},
    // input patch resident, any geometry
    {{128, 128, 64, 64, 64, 3, 2, 1, 1, 0, 4}, 4, 1, 2.79, 0.350, 1.17, 0.15},
    {{64, 64, 64, 64, 64, 2, 2, 1, 1, 0, 4}, 4, 4, 2.75, 0.508, 1.27, 0.17},
    {{256, 64, 64, 64, 64, 3, 2, 1, 1, 0, 4}, 4, 1, 2.84, 0.339, 1.15, 0.13},
    {{128, 64, 64, 64, 64, 3, 2, 1, 1, 0, 4}, 4, 2, 3.09, 0.361, 1.47, 0.17},
};

// row_tiles: tiles along M (the patch kernels count padded positions); patch_loads: am == 4 only
inline double measured_conv_us(const alcop_problem& p, const MeasuredConv& m, double row_tiles, int patch_loads)
{
  auto up = [](double x, double y) { return (double)(long)((x + y - 1) / y); };
  const double turns = up(row_tiles * up(p.N, m.s.bn), 256), kt = up(up(p.K, m.s.bk), m.waves_k);
  const double out = p.out == ALCOP_F32 ? 4.0 : 2.0;
  const double bytes = 2.0 * p.M * p.conv_C + 2.0 * p.K * p.N + out * p.M * p.N;
  return m.a + m.b * turns * kt + m.c * turns + m.d * (m.am == 4 ? turns * patch_loads : bytes / 5.1e6);
}

// as for the products: the kernels whose waves split K only while 64 x 64 tiles are few
inline bool measured_conv_applies(const alcop_problem& p, const MeasuredConv& m)
{
  return m.s.variant != 3 || (double)((p.M + 63) / 64) * ((p.N + 63) / 64) <= 512;
}

}  // namespace alcop
