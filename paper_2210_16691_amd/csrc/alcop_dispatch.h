// Which kernel a product without an explicit schedule gets: measured costs of a few kernels.
//
// The static model of Table 1 ranks hundreds of schedules for a tuner that times the best of them.
// Taken at its word, its first choice was 28 % slower than the best schedule in the mean over 243
// products of the kinds this library serves (linear layers and their gradients, attention; 1 to
// 8192 rows, K from 32 to 8192, fp16 and bf16, every layout; a tenth of them more than 60 %): it
// does not know the per-tile cost of a block, that persistent kernels whose consumers restart
// their register pipeline per k-tile are the faster ones, or the kernels whose waves split K.
//
// So the library measured every kernel on 330 products and fits, per kernel and operand layout,
//     us = a + b * turns * k-tiles + c * turns + d * (bytes of A, B and C at 5.1 TB/s)
//            + e * (flops at 1.4 PFLOP/s) + f * turns2 * k-tiles
// (least squares of the relative error, no negative coefficient) with turns = ceil(tiles / 256), the
// tiles one compute unit works through in a row, and, for kernels of which two blocks share a compute
// unit, turns2 = 2 ceil(tiles / 512); k-tiles are those of one wave where the waves split K.  a is the
// launch and the first loads, b and f the pace of the main loop (a 128 x 128 x 64 step 0.3 us), c the
// epilogue and restart of a tile, e the matrix rate that the card's power allows, which bounds the
// largest.  The layout matters: rows along k whose pitch is not a multiple of 128 bytes touch a second
// cache line per row and k-tile, and wide tiles fetch fewer rows (3873 x 2872 with B stored N x K, bf16:
// K = 7232 187 us with persistent 128 x 128 tiles and 167 with 256 x 192, K = 7192 235 and 181).  The
// kernels below are the ones that a greedy selection by the regret of the estimated best keeps; the
// pick is 3 % above the best in the mean and 7 % at the 90th percentile (1.53 times it at worst), on
// products above 12 GFLOP too, where a fit without e, f and the layouts left 8 % and 30 % (operands
// cycled through three buffers).  These figures are of the products that the kernels and coefficients
// were chosen on; none were held out.
#pragma once
#include <algorithm>
#include <cstring>

#include "../../include/alcop.h"

namespace alcop {

struct MeasuredCost {
  alcop_sched s;
  int transA, transB;  // operand layout the costs were measured with
  int waves_k;         // waves a tile's k-tiles are divided among
  int blocks;          // blocks that share a compute unit
  double a, b, c, d, e, f;
};

inline const MeasuredCost kMeasured[] = {
    // waves split K: while there are fewer 64 x 64 tiles than compute units
    {{32, 32, 64, 32, 32, 2, 1, 0, 1, 0, 3}, 0, 0, 8, 1, 1.655, 0.683, 1.495, 0.600, 1.303, 0.000},
    {{32, 32, 64, 32, 32, 2, 1, 0, 1, 0, 3}, 0, 1, 8, 1, 1.746, 0.391, 1.719, 0.300, 2.078, 0.000},
    {{32, 32, 64, 32, 32, 2, 1, 0, 1, 0, 3}, 1, 0, 8, 1, 2.093, 0.387, 1.430, 0.259, 5.506, 0.000},
    {{16, 16, 64, 16, 16, 2, 1, 0, 1, 0, 3}, 0, 0, 8, 1, 2.688, 0.320, 0.444, 0.846, 6.123, 0.000},
    {{16, 16, 64, 16, 16, 2, 1, 0, 1, 0, 3}, 0, 1, 8, 1, 2.475, 0.188, 0.671, 0.456, 2.358, 0.000},
    {{16, 16, 64, 16, 16, 2, 1, 0, 1, 0, 3}, 1, 0, 8, 1, 2.915, 0.178, 0.471, 0.000, 17.408, 0.000},
    {{32, 64, 64, 32, 64, 2, 1, 0, 1, 0, 3}, 0, 0, 4, 1, 1.919, 0.396, 1.701, 0.612, 0.592, 0.000},
    {{32, 64, 64, 32, 64, 2, 1, 0, 1, 0, 3}, 0, 1, 4, 1, 1.769, 0.328, 1.759, 0.633, 1.025, 0.000},
    {{32, 64, 64, 32, 64, 2, 1, 0, 1, 0, 3}, 1, 0, 4, 1, 2.628, 0.389, 1.066, 0.222, 2.619, 0.000},
    {{16, 32, 64, 16, 32, 2, 1, 0, 1, 0, 3}, 0, 0, 8, 1, 1.912, 0.438, 1.246, 0.643, 3.452, 0.000},
    {{16, 32, 64, 16, 32, 2, 1, 0, 1, 0, 3}, 0, 1, 8, 1, 1.741, 0.279, 1.500, 0.494, 2.654, 0.000},
    {{16, 32, 64, 16, 32, 2, 1, 0, 1, 0, 3}, 1, 0, 8, 1, 2.509, 0.211, 1.156, 0.000, 10.781, 0.000},
    // persistent
    {{128, 128, 64, 64, 64, 3, 2, 0, 1, 0, 2}, 0, 0, 1, 1, 2.508, 0.319, 1.120, 0.207, 0.445, 0.000},
    {{128, 128, 64, 64, 64, 3, 2, 0, 1, 0, 2}, 0, 1, 1, 1, 2.795, 0.294, 0.982, 0.188, 0.570, 0.000},
    {{128, 128, 64, 64, 64, 3, 2, 0, 1, 0, 2}, 1, 0, 1, 1, 2.699, 0.313, 1.019, 0.000, 0.582, 0.000},
    {{128, 64, 64, 64, 32, 3, 2, 0, 1, 0, 2}, 0, 0, 1, 1, 2.588, 0.258, 0.628, 0.272, 0.381, 0.000},
    {{128, 64, 64, 64, 32, 3, 2, 0, 1, 0, 2}, 0, 1, 1, 1, 2.852, 0.217, 0.671, 0.278, 0.675, 0.000},
    {{128, 192, 32, 64, 96, 3, 2, 0, 1, 0, 2}, 0, 0, 1, 1, 2.149, 0.246, 1.921, 0.209, 0.372, 0.000},
    // tile at a time
    {{64, 64, 64, 32, 32, 3, 2, 1, 1, 0, 0}, 0, 0, 1, 2, 2.415, 0.086, 0.330, 0.541, 0.092, 0.058},
    {{64, 64, 64, 32, 32, 3, 2, 1, 1, 0, 0}, 0, 1, 1, 2, 2.585, 0.023, 0.381, 0.458, 0.700, 0.080},
    {{64, 64, 64, 32, 32, 3, 2, 1, 1, 0, 0}, 1, 0, 1, 2, 2.769, 0.061, 0.165, 0.376, 0.793, 0.067},
    {{256, 128, 64, 128, 64, 3, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 0.000, 0.519, 4.954, 0.277, 0.327, 0.000},
    {{256, 128, 64, 128, 64, 3, 2, 1, 1, 0, 0}, 0, 1, 1, 1, 1.807, 0.490, 3.249, 0.294, 0.407, 0.000},
    {{256, 128, 64, 128, 64, 3, 2, 1, 1, 0, 0}, 1, 0, 1, 1, 0.814, 0.504, 4.371, 0.000, 0.442, 0.000},
    {{128, 128, 64, 64, 64, 4, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 1.384, 0.318, 2.552, 0.249, 0.317, 0.000},
    {{128, 128, 64, 64, 64, 4, 2, 1, 1, 0, 0}, 0, 1, 1, 1, 1.858, 0.304, 2.121, 0.305, 0.392, 0.000},
    {{128, 128, 64, 64, 64, 4, 2, 1, 1, 0, 0}, 1, 0, 1, 1, 1.654, 0.320, 2.428, 0.034, 0.412, 0.000},
    {{256, 192, 32, 128, 96, 3, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 0.141, 0.433, 5.835, 0.257, 0.262, 0.000},
    {{256, 192, 32, 128, 96, 3, 2, 1, 1, 0, 0}, 0, 1, 1, 1, 1.366, 0.437, 4.559, 0.235, 0.357, 0.000},
    {{256, 192, 32, 128, 96, 3, 2, 1, 1, 0, 0}, 1, 0, 1, 1, 1.366, 0.399, 5.047, 0.144, 0.291, 0.000},
    {{128, 128, 64, 64, 64, 2, 1, 0, 1, 0, 0}, 0, 0, 1, 2, 2.167, 0.043, 0.873, 0.347, 0.461, 0.263},
    {{128, 128, 64, 64, 64, 2, 1, 0, 1, 0, 0}, 0, 1, 1, 2, 2.181, 0.005, 1.051, 0.284, 0.548, 0.272},
    {{128, 128, 64, 64, 64, 2, 1, 0, 1, 0, 0}, 1, 0, 1, 2, 1.680, 0.016, 1.318, 0.000, 0.583, 0.285},
    {{128, 256, 64, 64, 128, 3, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 0.930, 0.503, 4.130, 0.341, 0.274, 0.000},
    {{256, 256, 32, 128, 64, 3, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 0.092, 0.464, 4.571, 0.406, 0.317, 0.000},
    {{256, 256, 32, 128, 64, 3, 2, 1, 1, 0, 0}, 0, 1, 1, 1, 0.460, 0.502, 4.408, 0.240, 0.424, 0.000},
    {{256, 256, 32, 128, 64, 3, 2, 1, 1, 0, 0}, 1, 0, 1, 1, 0.000, 0.459, 4.782, 0.402, 0.231, 0.000},
    {{64, 128, 64, 32, 64, 4, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 1.700, 0.228, 1.750, 0.224, 0.385, 0.000},
    {{64, 64, 64, 32, 32, 4, 2, 1, 1, 0, 0}, 0, 0, 1, 2, 2.339, 0.108, 0.546, 0.452, 0.134, 0.038},
    {{64, 64, 64, 32, 32, 4, 2, 1, 1, 0, 0}, 0, 1, 1, 2, 2.396, 0.064, 0.649, 0.355, 0.557, 0.056},
    {{64, 64, 64, 32, 32, 4, 2, 1, 1, 0, 0}, 1, 0, 1, 2, 2.679, 0.091, 0.395, 0.256, 0.690, 0.049},
    {{64, 64, 32, 32, 32, 3, 1, 0, 1, 0, 0}, 0, 0, 1, 2, 2.425, 0.037, 0.176, 0.489, 0.000, 0.061},
    {{64, 64, 32, 32, 32, 3, 1, 0, 1, 0, 0}, 0, 1, 1, 2, 2.604, 0.000, 0.188, 0.464, 1.035, 0.069},
    {{64, 64, 32, 32, 32, 3, 1, 0, 1, 0, 0}, 1, 0, 1, 2, 2.766, 0.038, 0.000, 0.449, 0.000, 0.061},
    {{128, 64, 64, 64, 32, 4, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 1.427, 0.261, 1.774, 0.334, 0.205, 0.000},
    {{128, 64, 64, 64, 32, 4, 2, 1, 1, 0, 0}, 0, 1, 1, 1, 1.775, 0.219, 1.798, 0.264, 0.459, 0.000},
    {{64, 64, 128, 32, 32, 4, 2, 1, 1, 0, 0}, 0, 0, 1, 1, 1.743, 0.337, 1.560, 0.428, 0.187, 0.000},
    {{64, 64, 128, 32, 32, 4, 2, 1, 1, 0, 0}, 0, 1, 1, 1, 2.016, 0.332, 1.690, 0.200, 0.312, 0.000},
};

inline double measured_us(const alcop_problem& p, const MeasuredCost& m)
{
  auto up = [](double x, double y) { return (double)(long)((x + y - 1) / y); };
  const double tiles = up(p.M, m.s.bm) * up(p.N, m.s.bn) * p.batch;
  const double turns = up(tiles, 256), kt = up(up(p.K, m.s.bk), m.waves_k);
  const double turns2 = m.blocks == 2 ? 2.0 * up(tiles, 512) : 0.0;
  const double out = p.out == ALCOP_F32 ? 4.0 : 2.0;
  const double bytes = p.batch * (2.0 * p.M * p.K + 2.0 * p.K * p.N + out * p.M * p.N);
  const double flops = 2.0 * p.batch * p.M * p.N * (double)p.K;
  return m.a + m.b * turns * kt + m.c * turns + m.d * bytes / 5.1e6 + m.e * flops / 1.4e9 + m.f * turns2 * kt;
}

// The measured kernels worth considering for a product: small tiles cost more bytes per flop, so the
// kernels whose waves split K are compared only while 64 x 64 tiles leave compute units idle (with 384
// such tiles, 1021 x 1536 x 768, they take 11.9 us at best against 6.2).  Mean time of the pick over the
// best kernel, with and without them: up to 64 such tiles 1.02 and 1.35, 64 to 128 1.02 and 1.08, 128 to
// 256 1.02 and 1.01; above 256 their costs never come out lowest (45 products up to 512), the line only
// keeps the fit from being used where nothing speaks for it.  Both operands transposed use the costs of
// A stored K x M.
inline bool measured_applies(const alcop_problem& p, const MeasuredCost& m)
{
  if (p.op == ALCOP_OP_CONV2D) return false;
  if (m.transA != (p.transA ? 1 : 0) || (!p.transA && m.transB != (p.transB ? 1 : 0))) return false;
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
// of A: 100352 x 64 x 576 19.1 against 12.2); the cheapest of these is 2 %, on the convolutions that the
// fit has seen.
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

// The kernels whose waves split K only while 64 x 64 tiles are few.  A gather pays longer for few tiles
// than a matrix does: with and without them the pick of a gathering kernel is 1.01 and 1.40 times the best
// up to 128 tiles, 1.02 and 1.04 from 128 to 256.  From 256 to 512 (22 convolutions) they are never
// the cheapest by cost, so that there the line may lie anywhere.
inline bool measured_conv_applies(const alcop_problem& p, const MeasuredConv& m)
{
  return m.s.variant != 3 || (double)((p.M + 63) / 64) * ((p.N + 63) / 64) <= 512;
}

// The estimated time of a product with a schedule, or of the cheapest measured kernel where that one
// was not measured.
inline double measured_sched_us(const alcop_problem& p, const alcop_sched& s)
{
  double best = 1e30;
  for (const MeasuredCost& m : kMeasured) {
    if (!measured_applies(p, m)) continue;
    if (std::memcmp(&m.s, &s, sizeof(s)) == 0) return measured_us(p, m);
    best = std::min(best, measured_us(p, m));
  }
  return best;
}

// Products of operands that are not made of aligned chunks: padded copies and a pipelined kernel
// (`product_us` by its estimate, `copied` bytes written by the copy), or 64 x 64 tiles that load them as
// they are (alcop_direct.hip.h).  Fitted on one half of 296 products (16 to 4096 rows, columns and K, every
// layout, bf16); on the other half the estimates are within 17 and 12 % at the 90th percentile.  A k-tile of
// the direct kernel costs 0.3 us per turn (misaligned loads: 24 bytes per clock and compute unit, the aligned
// ones of the pipelined loops 40 to 50), so it loses on long K and where tiles are many; short of that it
// saves the copy's launch (216 x 89 x 1766: 10.2 us with copies, 12.3 without; 142 x 1816 x 229: 7.8 and 4.9).
// With the line at 0.85 the direct kernel is taken for 73 % of the products, 1.38 times faster in the mean over
// all of them; one is slower by more than 1 % (26 x 30 x 567, one operand copied: 6.5 and 7.3), at 1.0 there
// are eleven.  In place of a kernel whose waves split K (`split`), eight partial sums cost 0.17 us in the median;
// 0.3 are counted.  Of 1796 products drawn afterwards (8 to 4096, and 120 up to 40000; both types, results of 16 and 32
// bits) the line without them takes 1297, of which 22 are slower by more than 1 %, up to 1.17 times (25 x 1195 x 801
// 8.5 us and 7.3); with them 1271, 13 slower, up to 1.06 times, and 16 that gain, up to 1.28 times, go back to the copies.
// What is taken is 1.52 times faster in the mean, 1.27 in place of kernels that split K.
inline bool direct_pays(int M, int N, int K, bool split, double product_us, double copied)
{
  const double tiles = (double)((M + 63) / 64) * ((N + 63) / 64), turns = (double)(((long)tiles + 255) / 256);
  const double kt = (K + 63) / 64, bytes = 2.0 * ((double)M * K + (double)K * N + (double)M * N);
  const double with_copies = 2.38 + 1.41 * product_us + 1.64 * copied / 5.1e6;
  const double direct = (split && K > 256 ? 3.42 : 3.12) + (0.033 + 0.282 * turns) * kt + 0.267 * turns + 0.68 * bytes / 5.1e6;
  return direct < 0.85 * with_copies;
}

}  // namespace alcop
