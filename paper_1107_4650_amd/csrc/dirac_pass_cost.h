// dirac_pass_cost.h -- fitted times of the 2-D passes, by which a call is routed to
// register tiles or marching passes (host code).  Internal to libdirac.
//
// Both were measured on 41 planes of 4 thousand to 17 million cells, from 64^2 to
// 4096^2, from 2^20 x 2 to 2 x 2^20 and at ragged sizes, with every phase mode,
// scheme and state type, every depth and both tile shapes (15 thousand passes).  Tiles
// win where a plane is small (256^2, FP32, per step: 1.0 against 4.1 us) and lose
// where it is a few rows thin (a tile's 32 or 48 rows are loaded and stepped whatever
// the plane fills of them; 2^20 x 2, FP32, 20 steps: tiles 1540 us, marching 534), on
// large FP32 planes with a constant mass phase (2048^2, 40 steps: 598 against 542)
// and where one tile more than the chip has units begins (FP64, second order, 774^2,
// 36 steps: 469 against 397).  The fits err by 5 % (tiles) and 8 % (marching), so a
// call leaves the tiles only where marching is predicted to be 5 % faster; a call of
// one pass, which is a copy and little else, goes where the prediction says, and so
// does FP64 second order, where the two cross flatly and are predicted to 3 % (640^2 to
// 720^2, 36 steps: marching 343 to 364 us, tiles 349 to 397).  Of 13 thousand calls of
// 1 to 100 steps composed from the measured passes, 2280 take over 3 % longer than in
// marching passes with tiles wherever they fit, at worst 4.3 times; by this rule 236
// do, at worst 1.3 times.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace dirac {

// workgroups on the busiest compute unit; many of them average out
inline double per_unit(double groups, int cu_count) {
  const double w = groups / cu_count;
  return w < 4.0 ? std::ceil(w) : w;
}

// bytes of a pass in MB, and what of them the caches do not keep between passes
struct PassBytes { double mb, beyond; };
inline PassBytes pass_bytes(double mb) { return {mb, std::max(0.0, mb - 180.0)}; }
inline double forward_mb(double cells, bool fp64, int mode) {
  return cells * ((fp64 ? 128 : 64) + (mode == 2 ? 8 : 0) + (mode >= 3 ? 32 : 0)) / 1e6;
}

// A register-tile pass: a compute unit's first tile takes t0 + t1 per transport pair
// (h), every further one n0 + n1 h, the bytes m per MB and o more beyond the caches.
struct TileFit { double t0, t1, n0, n1, m, o; };
inline double tile_us(const TileFit& f, int h, double tiles, PassBytes b, int cu_count) {
  const double more = std::max(0.0, per_unit(tiles, cu_count) - 1.0);
  return f.t0 + f.t1 * h + more * (f.n0 + f.n1 * h) + f.m * b.mb + f.o * b.beyond;
}

// A marching pass of K steps: a wave's iterations (its segment and the stages at both
// ends), the iterations its SIMD still has to issue for further waves, and the bytes;
// the coefficients run linearly from K = 1 to the deepest pass.
struct MarchFit { double c0, it, more, m, o; };
inline double march_us(const MarchFit (&f)[2], int depth, int deepest, int stages, int rows,
                       double rows_mean, double blocks, PassBytes b, int cu_count) {
  const double it = rows + 2.0 * stages;
  const double more =
      std::max(0.0, per_unit(blocks, cu_count) * (rows_mean + 2.0 * stages) - it);
  auto at = [&](const MarchFit& q) {
    return q.c0 + q.it * it + q.more * more + q.m * b.mb + q.o * b.beyond;
  };
  const double u = deepest > 1 ? (depth - 1.0) / (deepest - 1.0) : 0.0;
  return (1.0 - u) * at(f[0]) + u * at(f[1]);
}

// time in us of a pass of `halo` transports per axis in register tiles of TileKind `kind`
// (a unit's first tile only for the pairs apart, which run no others)
inline double tile_pass_us(bool fp64, bool strang, int mode, int kind, int halo, double tiles,
                           double cells, int cu_count) {
  static const TileFit fits[2][2][5][4] = {  // [fp64][strang][phase mode][kind]
    {{{{3.82, 0.51, 0.796, 0.36, 0.0915, 0.00905}, {4.09, 1.08, 0.322, 0.73, 0.0932, 0},
       {3.74, 0.316, 0, 0, 0.125}, {4.77, 0.478, 0, 0, 0.141}},
      {{3.82, 0.71, 0.662, 0.574, 0.0833, 0.026}, {4, 1.48, 0.541, 1.1, 0.0928, 0},
       {3.76, 0.406, 0, 0, 0.12}, {4.62, 0.724, 0, 0, 0.138}},
      {{4.65, 0.689, 1.23, 0.577, 0.078, 0.044}, {6.16, 1.08, 1.85, 0.854, 0.0816, 0.0318},
       {4.5, 0.403, 0, 0, 0.114}, {6.34, 0.716, 0, 0, 0.128}},
      {{3.94, 0.848, 0.865, 0.723, 0.0701, 0.0474}, {4.49, 1.45, 2.94, 1.43, 0.0915, 0.06}},
      {{4.72, 1.59, 1.59, 1.13, 0.117, 0.115}, {6.24, 2.49, 3.84, 2.53, 0.118, 0.125}}},
     {{{3.55, 0.559, 0.654, 0.378, 0.0843, 0.00426}, {3.96, 1.03, 0.0895, 0.833, 0.0871, 0},
       {3.56, 0.336, 0, 0, 0.112}, {4.22, 0.585, 0, 0, 0.143}},
      {{3.65, 0.638, 0.679, 0.472, 0.0745, 0.0281}, {4.09, 1.22, 0.259, 0.977, 0.0804, 0},
       {3.61, 0.386, 0, 0, 0.107}, {4.28, 0.672, 0, 0, 0.135}},
      {{4.92, 0.574, 1.18, 0.458, 0.0923, 0.0626}, {5.65, 1.06, 0.967, 0.853, 0.0706, 0.0239},
       {4.29, 0.386, 0, 0, 0.105}, {5.93, 0.682, 0, 0, 0.127}},
      {{0}, {4.68, 1.05, 2.99, 0.988, 0.0935, 0.0461}},
      {{0}, {7.34, 1.67, 4.58, 1.7, 0.134, 0.156}}}},
    {{{{6.01, 0.788, 1.9, 0.862, 0.185, 0.00677}, {6.9, 1.03, 0.752, 0.736, 0.151, 0.0281},
       {4.55, 0.447, 0, 0, 0.153}, {6.74, 0.784, 0, 0, 0.173}},
      {{5.89, 0.898, 1.79, 0.964, 0.186, 0.00595}, {6.92, 1.12, 0.678, 0.839, 0.148, 0.0301},
       {4.49, 0.506, 0, 0, 0.153}, {6.61, 0.922, 0, 0, 0.173}},
      {{7.29, 0.898, 3.21, 0.968, 0.173, 0.00272}, {9.38, 1.07, 2.08, 0.862, 0.128, 0.0283},
       {5.97, 0.51, 0, 0, 0.156}, {9.55, 0.924, 0, 0, 0.157}},
      {{5.79, 0.739, 1.08, 0.815, 0.124, 0.0163}, {8.15, 1.61, 4.34, 1.73, 0.159, 0.0312}},
      {{4.85, 1.82, 2.37, 1.82, 0.15, 0}, {8.87, 3.42, 5.23, 3.61, 0.165, 0.0806}}},
     {{{5.68, 0.789, 1.74, 0.849, 0.183, 0.00248}, {6.77, 0.898, 0.666, 0.697, 0.147, 0.0315},
       {4.36, 0.446, 0, 0, 0.145}, {6.13, 0.835, 0, 0, 0.175}},
      {{5.79, 0.816, 1.77, 0.899, 0.176, 0.00683}, {6.73, 0.916, 0.628, 0.745, 0.14, 0.0321},
       {4.36, 0.465, 0, 0, 0.14}, {6.12, 0.89, 0, 0, 0.171}},
      {{7.24, 0.831, 3.38, 0.87, 0.159, 0.00228}, {10.1, 0.92, 2.51, 0.752, 0.117, 0.0276},
       {5.84, 0.478, 0, 0, 0.146}, {9.08, 0.878, 0, 0, 0.153}},
      {{0}, {8.33, 1.21, 4.36, 1.32, 0.158, 0.0262}},
      {{0}, {10.3, 2.27, 6, 2.48, 0.172, 0.0981}}}}};
  return tile_us(fits[fp64][strang][mode][kind], halo, tiles,
                 pass_bytes(forward_mb(cells, fp64, mode)), cu_count);
}

// ... of a marching pass of `depth` steps over segments of `rows` rows (rows_mean on
// average) in `blocks` workgroups
inline double march_pass_us(bool fp64, bool strang, int mode, int depth, int deepest, int rows,
                            double rows_mean, double blocks, double cells, int cu_count) {
  static const MarchFit fits[2][2][5][2] = {  // [fp64][strang][phase mode][K = 1, deepest]
    {{{{2.25, 0.267, 0.0583, 0.116, 0.0953}, {2.24, 0.632, 0.219, 0.0205, 0.128}},
      {{1.99, 0.31, 0.0638, 0.107, 0.104}, {1.14, 0.841, 0.315, 0.0111, 0.0898}},
      {{2.58, 0.393, 0.182, 0.0724, 0.118}, {1.12, 1.04, 0.338, 0.0127, 0.055}},
      {{3.63, 0.507, 0.403, 0.0624, 0.111}, {1.46, 1.08, 0.522, 0.0212, 0.0696}},
      {{3.24, 0.605, 0.398, 0.0622, 0.0972}, {0, 1.44, 0.665, 0.0244, 0.0628}}},
     {{{0.823, 0.438, 0.0656, 0.107, 0.0868}, {4.28, 0.581, 0.222, 0.0225, 0.123}},
      {{1.31, 0.432, 0.0982, 0.0838, 0.0909}, {3.03, 0.722, 0.266, 0.0256, 0.102}},
      {{1.77, 0.621, 0.187, 0.0427, 0.123}, {3, 0.907, 0.387, 0.00336, 0.105}},
      {{3.7, 0.63, 0.437, 0.0361, 0.132}, {3.7, 0.63, 0.437, 0.0361, 0.132}},
      {{3.5, 0.693, 0.449, 0.0349, 0.125}, {3.5, 0.693, 0.449, 0.0349, 0.125}}}},
    {{{{5.43, 0.227, 0.175, 0.145, 0.0879}, {2.44, 0.785, 0.429, 0.0525, 0.136}},
      {{4.8, 0.265, 0.163, 0.148, 0.0867}, {1.34, 0.889, 0.451, 0.0457, 0.139}},
      {{5.06, 0.406, 0.345, 0.103, 0.123}, {0, 1.34, 0.884, 0.00595, 0.0852}},
      {{5.14, 0.565, 0.707, 0.0894, 0.114}, {1.72, 1.31, 1.27, 0.0229, 0.0814}},
      {{5.81, 0.56, 0.846, 0.0766, 0.114}, {0, 1.78, 1.11, 0.0208, 0.0941}}},
     {{{3.52, 0.476, 0.278, 0.123, 0.0826}, {1.93, 0.903, 0.391, 0.0426, 0.158}},
      {{3.07, 0.514, 0.302, 0.117, 0.0874}, {1.76, 0.915, 0.422, 0.0383, 0.157}},
      {{4.35, 0.591, 0.463, 0.0766, 0.122}, {0, 1.36, 0.817, 0, 0.102}},
      {{4.82, 0.758, 0.7, 0.0612, 0.133}, {4.82, 0.758, 0.7, 0.0612, 0.133}},
      {{4.03, 1.1, 0.579, 0.079, 0.127}, {4.03, 1.1, 0.579, 0.079, 0.127}}}}};
  return march_us(fits[fp64][strang][mode], depth, deepest, depth * (strang ? 2 : 1), rows,
                  rows_mean, blocks, pass_bytes(forward_mb(cells, fp64, mode)), cu_count);
}

// The reverse passes of a 2-D plane (phase modes 0 to 2), fitted to the same planes; a
// tile pass hides part of its bytes behind its steps (1.5-norm of both).  A tile holds 16
// (small) or 24 rows, so planes a few rows thin lose here too (2^20 x 2, a pass of one
// reverse step: FP32 152 against 75 us, FP64 362 against 172).  Errors 5 to 7 %; a call
// marches where that is predicted to be 3 % faster.  Of 2800 measured calls of 1 to 120
// reverse steps 457 ran over 3 % slower than marching, at worst 1.7 times; by this rule
// 66 do, at worst 1.2 times.
inline PassBytes reverse_bytes(double cells, bool fp64, int mode) {
  return pass_bytes(cells * ((fp64 ? 256 : 128) + 16 + (mode == 2 ? 8 : 0)) / 1e6);
}
inline double rev_tile_pass_us(bool fp64, int mode, bool big, int steps, double tiles,
                               double cells, int cu_count) {
  static const TileFit fits[2][3][2] = {  // [fp64][phase mode][big]
    {{{3.13, 1.03, 0.371, 0.723, 0.137, 0.0719}, {3.54, 1.49, 0.589, 1.05, 0.128, 0.07}},
     {{3.06, 1.32, 0.482, 0.866, 0.134, 0.0636}, {3.53, 1.84, 0.576, 1.3, 0.123, 0.0683}},
     {{3.57, 1.29, 0.801, 0.888, 0.136, 0.0587}, {4.45, 1.85, 1.16, 1.3, 0.121, 0.0743}}},
    {{{4.78, 1.24, 2.65, 1.25, 0.238, 0.0259}, {6.09, 1.76, 3.67, 1.73, 0.233, 0.0518}},
     {{4.6, 1.39, 2.67, 1.36, 0.239, 0.0192}, {5.89, 1.88, 3.76, 1.81, 0.232, 0.0455}},
     {{5.37, 1.33, 3.73, 1.26, 0.236, 0.0187}, {6.91, 1.84, 4.98, 1.77, 0.229, 0.0482}}}};
  const TileFit& f = fits[fp64][mode][big];
  const PassBytes b = reverse_bytes(cells, fp64, mode);
  const double more =
      std::max(0.0, per_unit(tiles, cu_count) - 1.0) * (f.n0 + f.n1 * steps);
  const double memory = f.m * b.mb + f.o * b.beyond;
  return f.t0 + f.t1 * steps +
         std::cbrt(std::pow(more * std::sqrt(more) + memory * std::sqrt(memory), 2.0));
}
inline double rev_march_pass_us(bool fp64, int mode, int depth, int deepest, int rows,
                                double rows_mean, double blocks, double cells, int cu_count) {
  static const MarchFit fits[2][3][2] = {  // [fp64][phase mode][K = 1, deepest]
    {{{4.49, 0.339, 0.36, 0.0824, 0.134}, {2.61, 1.38, 1.44, 0.00245, 0.0569}},
     {{4.7, 0.372, 0.417, 0.0734, 0.137}, {2.4, 1.54, 1.63, 0, 0.0414}},
     {{4.9, 0.469, 0.498, 0.065, 0.135}, {2.13, 1.65, 1.75, 0.00383, 0.037}}},
    {{{5.01, 0.882, 1.11, 0.116, 0.0535}, {6.79, 1.06, 1.23, 0.0921, 0.0834}},
     {{5, 0.894, 1.13, 0.115, 0.0537}, {6.99, 1.09, 1.26, 0.0904, 0.0831}},
     {{5.63, 1.12, 1.4, 0.102, 0.0515}, {6.85, 1.38, 1.52, 0.0909, 0.0649}}}};
  return march_us(fits[fp64][mode], depth, deepest, depth, rows, rows_mean, blocks,
                  reverse_bytes(cells, fp64, mode), cu_count);
}

}  // namespace dirac
