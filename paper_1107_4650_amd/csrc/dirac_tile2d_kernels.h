// dirac_tile2d_kernels.h -- 2-D passes held in a workgroup's registers.
// Internal to libdirac.
//
// A workgroup of W waves holds a tile of 64 columns by W * RW rows (RW rows
// per wave, one cell per lane and row) with its phase factors in registers,
// advances it by K full steps and writes the cells K steps (2K transports per
// axis with second-order steps) away from the tile's edges.  The x transport
// is a DPP shift, the y transport passes the movers of a wave's first and
// last row to its neighbours through LDS (double buffered: one barrier per y
// transport).  The cells beyond a wave's tile that a transport lacks only
// reach cells that are not written.  Per cell the arithmetic and its order are
// those of the marching passes, so the bits are the same.
//
// Why beside the marching passes (march2d): a marching wave issues its rows
// one after the other, 18 iterations of 5 stages however small the plane,
// and at two waves per SIMD it cannot use the second FP32 issue slot (a wave
// issues one FP32 instruction in 4.9 cycles, four waves one in 2.4).  Tiles
// need 16 registers per cell (FP32) and run 4 to 8 waves per SIMD.  Per step
// with a potential, marching -> tiles: 256^2 FP32 4.06 -> 1.20 us, 1024^2
// 6.7 -> 4.6 us, 2048^2 17.0 -> 14.0 us; 256^2 FP64 4.9 -> 1.7 us; second
// order at 2048^2 FP32 28.4 -> 25.7 us.  Large planes are bound by VALU issue
// (the halo makes a tile of 48 rows and K = 7 do 1.8 times the work it writes;
// 71 % of the issue slots at 2.4 GHz and 3.1 TB/s counted at 2048^2); small ones
// by the launch and the first load (about 5 us) and by the barrier and LDS
// latency of a step (0.7 us).  With a vector potential a step is bound by some
// 150 FP64 operations per cell, the halo counts for more and the tiles win on
// planes of up to 768^2 cells only (pulse, FP32: 256^2 7.3 -> 2.8 us per step,
// 768^2 11.1 -> 9.0, 1024^2 13.7 marching against 15.6).
// On a small plane of alpha_x and alpha_y the step is the issue of a unit's
// sixteen waves while other units idle: the two uncoupled pairs of a spinor
// go to workgroups of their own (256^2, FP32, 100 steps: 119 -> 97 us).
#pragma once
#include "dirac_device.h"
#include "dirac_launch.h"
#include "dirac_sweep_impl.h"

namespace dirac {

// one y mover of every lane of a wave, in 16-byte parts (conflict-free
// 128-bit LDS accesses for both state types)
template <typename T, CellPart P = kAll> struct MovLds {
  static constexpr int kParts = sizeof(Mov<T>) / 16;
  uint4 q[kParts][64];
  __device__ __forceinline__ void put(int lane, const Mov<T>& m) {
    const uint4* s = reinterpret_cast<const uint4*>(m.v);
#pragma unroll
    for (int p = 0; p < kParts; ++p) q[p][lane] = s[p];
  }
  __device__ __forceinline__ void get(int lane, Mov<T>& m) const {
    uint4* d = reinterpret_cast<uint4*>(m.v);
#pragma unroll
    for (int p = 0; p < kParts; ++p) d[p] = q[p][lane];
  }
};

// ... of a pair on the plane of alpha_x and alpha_y: one complex number
template <typename T, CellPart P> struct MovPair {
  static constexpr int at = P == kSecond ? 2 : 0;
  struct alignas(2 * sizeof(T)) Complex { T re, im; };
  Complex q[64];
  __device__ __forceinline__ void put(int lane, const Mov<T>& m) {
    q[lane] = Complex{m.v[at], m.v[at + 1]};
  }
  __device__ __forceinline__ void get(int lane, Mov<T>& m) const {
    zero(m);
    const Complex c = q[lane];
    m.v[at] = c.re;
    m.v[at + 1] = c.im;
  }
};
template <typename T> struct MovLds<T, kFirst> : MovPair<T, kFirst> {};
template <typename T> struct MovLds<T, kSecond> : MovPair<T, kSecond> {};

// r (at most 2^31 + a tile) wrapped around a periodic box, or clamped to the box
__device__ __forceinline__ int64_t tile_index(int64_t r, int64_t n, int periodic) {
  if (!periodic) return r < 0 ? 0 : (r >= n ? n - 1 : r);
  // one wrap reaches the halo of any box of a tile or more; the division
  // only runs for smaller boxes
  if (r < 0) r += n;
  if (r >= n) r -= n;
  if (r < 0 || r >= n) {
    const int m = static_cast<int>(r) % static_cast<int>(n);
    r = m < 0 ? m + static_cast<int>(n) : m;
  }
  return r;
}

// the pass on tile (strip, seg) of the plane: strips of 64 - 2 a.halo written
// columns, tile rows of W * RW - 2 a.halo.  P: the components held (a pair on the
// plane of alpha_x and alpha_y only, without a vector potential)
template <typename T, class S, int W, int RW, int AX0, int AX1, int MODE, CellPart P = kAll>
__device__ __forceinline__ void tile2d(const T* __restrict__ src, T* __restrict__ dst,
                                       const double* __restrict__ V, const TileArgs& a, int lane,
                                       int wv, int64_t strip, int64_t seg,
                                       MovLds<T, P> (&sr)[2][W], MovLds<T, P> (&sl)[2][W]) {
  static_assert(P == kAll || (AX0 == 0 && AX1 == 1 && MODE <= 2), "pairs do not couple");
  using C = PartCell<AX0, P>;
  constexpr bool TWO = sizeof(T) == 8;
  const int64_t nx = a.nx, ny = a.ny;
  const int X = a.halo;  // transports per axis of the pass
  const int64_t x = strip * (64 - 2 * X) - X + lane;
  const int64_t y0 = seg * (W * RW - 2 * X) - X + wv * RW;  // this wave's first row
  const int64_t col = tile_index(x, nx, a.periodic);
  const bool xin = x >= 0 && x < nx;
  // wave-uniform: some cell of the wave lies beyond a zero wall
  const int64_t xs = strip * (64 - 2 * X) - X;
  const bool walls = !a.periodic && (xs < 0 || xs + 63 >= nx || y0 < 0 || y0 + RW > ny);
  constexpr bool PULSE = MODE == 4;           // ... with a pulse
  constexpr bool FIELD = MODE == 3 || PULSE;  // local step with a vector potential
  Site<T> s[RW];
  double v[RW], at[FIELD ? RW : 1][3];
  uint32_t yin = 0;  // bit j: row y0 + j lies in the box
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    const int64_t q = tile_index(y0 + j, ny, a.periodic) * nx + col;
    C::load(src, q, s[j]);
    v[j] = (MODE == 2 || (FIELD && V != nullptr)) ? V[q] : 0.0;
    if constexpr (FIELD) {
      at[j][0] = a.At[q];
      at[j][1] = a.At[a.cells + q];
      at[j][2] = a.At[2 * a.cells + q];
    }
    if (y0 + j >= 0 && y0 + j < ny) yin |= 1u << j;
  }
  yin = __builtin_amdgcn_readfirstlane(yin);
  // the rows' phase factors, U (static field), or scalar phase and profile
  // (pulse: U is formed per step)
  using FT = typename std::conditional<FIELD, typename FactorOf<MODE>::type,
                                       typename Stored<T>::type>::type;
  FT f[RW];
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    if constexpr (PULSE) {
      f[j] = pulse_row<TWO>(v[j], at[j][0], at[j][1], at[j][2], a.ph);
    } else if constexpr (FIELD) {
      f[j] = field_factors<TWO, false>(v[j], at[j][0], at[j][1], at[j][2], a.ph);
      field_fix<TWO>(f[j], v[j], at[j][0], at[j][1], at[j][2], a.ph);
    } else {
      Factors fd = factors_of<MODE, TWO>(v[j], a.ph);
      factors_fix<MODE, TWO>(fd, v[j], a.ph);
      f[j] = Stored<T>::of(fd);
    }
    if (walls && (!((yin >> j) & 1u) || !xin)) zero(s[j]);
  }
  const int below = wv > 0 ? wv - 1 : 0, above = wv < W - 1 ? wv + 1 : W - 1;
  // One transport pair and its local work per stage.  EDGE: zero the cells
  // beyond a zero wall after every stage, as the marching passes do.
  // FAR: form U with the general sine and cosine where an angle needs them.
  auto advance = [&](auto edge, auto far) {
    constexpr bool EDGE = decltype(edge)::value;
    constexpr bool FAR = decltype(far)::value;
    int buf = 0;
    for (int k = 0; k < a.steps; ++k) {
      const double F = PULSE ? a.F[k] : 1.0;
#pragma unroll
      for (int st = 0; st < S::kStages; ++st, buf ^= 1) {
        Mov<T> r[RW], l[RW];
        if (S::pre_x(st)) {
#pragma unroll
          for (int j = 0; j < RW; ++j) {
            Site<T> o;
            x_transport_inner<T, AX0>(s[j], o);
            s[j] = o;
            if (TWO) Axis<AX1, T>::movers(s[j], r[j], l[j]);
          }
        }
        if (!TWO || !S::pre_x(st)) {
#pragma unroll
          for (int j = 0; j < RW; ++j) Axis<AX1, T>::movers(s[j], r[j], l[j]);
        }
        sr[buf][wv].put(lane, r[RW - 1]);
        sl[buf][wv].put(lane, l[0]);
        __syncthreads();
        Mov<T> rb, la;  // from the row below the wave's first, above its last
        sr[buf][below].get(lane, rb);
        sl[buf][above].get(lane, la);
#pragma unroll
        for (int j = 0; j < RW; ++j) {
          Axis<AX1, T>::combine(j > 0 ? r[j - 1] : rb, j < RW - 1 ? l[j + 1] : la, s[j]);
          if (S::phase(st)) {
            if constexpr (PULSE)
              apply_field(s[j], field_with<TWO, FAR>(f[j].pr, f[j].pi, F * f[j].px, F * f[j].py,
                                                     F * f[j].pz, a.ph));
            else if constexpr (FIELD)
              apply_field(s[j], f[j]);
            else
              apply_local<MODE>(s[j], f[j], a.ph);
          }
          if (S::post_x(st)) {
            Site<T> o;
            x_transport_inner<T, AX0>(s[j], o);
            s[j] = o;
          }
          if (EDGE && walls && (!((yin >> j) & 1u) || !xin)) zero(s[j]);
          // one row's FP64 temporaries at a time (interleaved rows spill)
          if (FIELD) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  // waves of two rows run a loop without the wall test where no cell lies
  // beyond a wall; with more rows per wave that loop spills (the test's branch
  // keeps the compiler from interleaving the rows' temporaries), so those
  // waves test in every stage
  if constexpr (PULSE) {
    // the largest angle of the pass decides for the whole wave
    double Fm = 0.0;
    for (int k = 0; k < a.steps; ++k) Fm = fmax(Fm, fabs(a.F[k]));
    bool far = false;
#pragma unroll
    for (int j = 0; j < RW; ++j)
      far = far || angle_far<TWO>(Fm * f[j].px, Fm * f[j].py, Fm * f[j].pz, a.ph);
    if (__any(far))
      advance(std::true_type{}, std::true_type{});
    else
      advance(std::true_type{}, std::false_type{});
  } else if (RW > 2 || walls) {
    advance(std::true_type{}, std::false_type{});
  } else {
    advance(std::false_type{}, std::false_type{});
  }
  if (!xin || lane < X || lane > 63 - X) return;
#pragma unroll
  for (int j = 0; j < RW; ++j) {
    const int t = wv * RW + j;  // tile row
    if (((yin >> j) & 1u) && t >= X && t < W * RW - X)
      C::store(dst, (y0 + j) * nx + x, s[j]);
  }
}

template <typename T, class S, int W, int RW, int AX0, int AX1, int MODE>
__global__ __launch_bounds__(64 * W, tile2d_waves(sizeof(T) == 8, RW, MODE)) void k_tile2d(
    const T* __restrict__ src, T* __restrict__ dst, const double* __restrict__ V, TileArgs a) {
  __shared__ MovLds<T> sr[2][W], sl[2][W];  // right movers up, left movers down
  int64_t blk = blockIdx.x;
  if (a.xcd_remap) blk = (blk % 8) * (gridDim.x / 8) + blk / 8;
  if (blk >= a.ntiles) return;  // the whole workgroup
  tile2d<T, S, W, RW, AX0, AX1, MODE>(src, dst, V, a, threadIdx.x & 63, wave_in_block(),
                                      blk % a.nstrips, blk / a.nstrips, sr, sl);
}

// the pass with the two pairs of a plane of alpha_x and alpha_y in workgroups of
// their own (blockIdx.y)
template <typename T, class S, int W, int RW, int MODE>
__global__ __launch_bounds__(64 * W, 4) void k_tile2d_pairs(const T* __restrict__ src,
                                                            T* __restrict__ dst,
                                                            const double* __restrict__ V,
                                                            TileArgs a) {
  union Movers {
    MovLds<T, kFirst> first[2][W];
    MovLds<T, kSecond> second[2][W];
  };
  __shared__ Movers sr, sl;
  int64_t blk = blockIdx.x;
  if (a.xcd_remap) blk = (blk % 8) * (gridDim.x / 8) + blk / 8;
  if (blk >= a.ntiles) return;  // the whole workgroup
  const int64_t strip = blk % a.nstrips, seg = blk / a.nstrips;
  if (blockIdx.y == 0)
    tile2d<T, S, W, RW, 0, 1, MODE, kFirst>(src, dst, V, a, threadIdx.x & 63, wave_in_block(),
                                            strip, seg, sr.first, sl.first);
  else
    tile2d<T, S, W, RW, 0, 1, MODE, kSecond>(src, dst, V, a, threadIdx.x & 63, wave_in_block(),
                                             strip, seg, sr.second, sl.second);
}

template <typename T, class S, int KIND>
const void* tile2d_pairs(int mode) {
  constexpr TileShape t = tile_shape(sizeof(T) == 8, KIND);
  switch (mode) {
    case 0: return reinterpret_cast<const void*>(&k_tile2d_pairs<T, S, t.waves, t.rows, 0>);
    case 1: return reinterpret_cast<const void*>(&k_tile2d_pairs<T, S, t.waves, t.rows, 1>);
    case 2: return reinterpret_cast<const void*>(&k_tile2d_pairs<T, S, t.waves, t.rows, 2>);
    default: return nullptr;
  }
}

template <typename T, class S, bool BIG, int AX0, int AX1>
const void* tile2d_mode(int mode) {
  constexpr TileShape t = tile_shape(sizeof(T) == 8, BIG);
  constexpr TileShape f = tile_shape(sizeof(T) == 8, BIG, true);
  constexpr bool kField = BIG || std::is_same<S, LieStep>::value;
  switch (mode) {
    case 0: return reinterpret_cast<const void*>(&k_tile2d<T, S, t.waves, t.rows, AX0, AX1, 0>);
    case 1: return reinterpret_cast<const void*>(&k_tile2d<T, S, t.waves, t.rows, AX0, AX1, 1>);
    case 2: return reinterpret_cast<const void*>(&k_tile2d<T, S, t.waves, t.rows, AX0, AX1, 2>);
    case 3:
      if constexpr (kField)
        return reinterpret_cast<const void*>(&k_tile2d<T, S, f.waves, f.rows, AX0, AX1, 3>);
      else
        return nullptr;
    case 4:
      if constexpr (kField)
        return reinterpret_cast<const void*>(&k_tile2d<T, S, f.waves, f.rows, AX0, AX1, 4>);
      else
        return nullptr;
    default: return nullptr;
  }
}

template <typename T, class S, bool BIG>
const void* tile2d_axes(int axes_code, int mode) {
  switch (axes_code) {
    case 10: return tile2d_mode<T, S, BIG, 0, 1>(mode);
    case 20: return tile2d_mode<T, S, BIG, 0, 2>(mode);
    case 21: return tile2d_mode<T, S, BIG, 1, 2>(mode);
    default: return nullptr;
  }
}

template <typename T, class S>
const void* tile2d_kind(TileKind kind, int axes_code, int mode) {
  switch (kind) {
    case kTileSmall: return tile2d_axes<T, S, false>(axes_code, mode);
    case kTileBig: return tile2d_axes<T, S, true>(axes_code, mode);
    case kTilePairs: return axes_code == 10 ? tile2d_pairs<T, S, kTilePairs>(mode) : nullptr;
    case kTilePairsBig:
      return axes_code == 10 ? tile2d_pairs<T, S, kTilePairsBig>(mode) : nullptr;
  }
  return nullptr;
}

template <typename T>
const void* kernel_tile2d(bool strang, TileKind kind, int axes_code, int mode) {
  return strang ? tile2d_kind<T, StrangStep>(kind, axes_code, mode)
                : tile2d_kind<T, LieStep>(kind, axes_code, mode);
}

// the instance groups (nullptr for combinations that are not built)
const void* kernel_tile2d_f32(bool strang, TileKind kind, int axes_code, int mode);
const void* kernel_tile2d_f64(bool strang, TileKind kind, int axes_code, int mode);

}  // namespace dirac
