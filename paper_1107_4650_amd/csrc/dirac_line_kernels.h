// dirac_line_kernels.h -- passes of many steps over a 1-D line, held in a
// workgroup's registers.  Internal to libdirac.
//
// A workgroup of W waves holds W * 48 + 16 consecutive cells, one per lane:
// wave w the 64 cells from 48 w on, so neighbouring waves share 16.  An x
// transport is a DPP shift inside the wave, valid one lane further in from both
// ends; every kLineSync transports the waves pass the 8 valid cells next to
// the shared ones to each other through LDS and every lane is valid again.
// After X transports the cells X and more from the ends of the workgroup's span
// are written.  Per cell the arithmetic and its order are those of one_row, so the
// bits are the same.
//
// What bounds it: on short lines the launch (2.7-3.6 us a pass) and the latency
// of a step in one wave per SIMD, so passes are deep and the two uncoupled pairs
// of a spinor go to workgroups of their own (24 instead of 48 operations per
// step); on long ones the issue of the step's operations, so the workgroup is
// wide, which lets a pass be deep at little halo.  The exchange every 8
// transports keeps the overlap of the waves at 16 of 64 lanes whatever the depth
// of the pass, where waves that exchange nothing lose a lane at both ends per
// transport (24 steps: 16 of 64 lanes written).  Per lowest-order step, FP64, 4
// components: 4096 cells 0.142 us (waves without exchange, 24 steps a pass:
// 0.248), 65536 cells 0.30 (0.61), 2^20 cells 2.06 (5 steps a pass: 6.9).
#pragma once
#include <type_traits>

#include "dirac_device.h"
#include "dirac_launch.h"
#include "dirac_sweep_impl.h"

namespace dirac {

// what neighbouring waves hand over: the kLineSync valid cells next to the
// shared ones at the left, then at the right end of every wave
// ([buffer][16-byte part][wave][cell])
template <typename T, int W, int NR>
struct LineEnds {
  static constexpr int kParts = NR * static_cast<int>(sizeof(T)) / 16;
  uint4 q[2][kParts][W * 2 * kLineSync];
};

template <typename T, class S, int W, int AX, int MODE, CellPart P>
__device__ __forceinline__ void line_pass(const T* __restrict__ src, T* __restrict__ dst,
                                          const double* __restrict__ V, const LineArgs& a,
                                          LineEnds<T, W, PartCell<AX, P>::NR>& ends) {
  using C = PartCell<AX, P>;
  constexpr bool TWO = sizeof(T) == 8;
  constexpr int H = kLineSync, OWN = 64 - 2 * H;
  constexpr int NR = C::NR, PT = LineEnds<T, W, NR>::kParts;
  const int lane = threadIdx.x & 63;
  const int wv = wave_in_block();
  const int64_t x0 = int64_t(blockIdx.x) * a.own - a.halo;  // first cell of the span
  const int pos = wv * OWN + lane;  // cell of the span
  const Lanes c = lanes_of(a.nx, a.periodic, x0 + wv * OWN, lane);
  Site<T> m;
  C::load(src, c.col, m);
  const double v = (MODE == 2) ? V[c.col] : 0.0;
  if (c.out) zero(m);
  Factors fd = factors_of<MODE, TWO>(v, a.ph);
  factors_fix<MODE, TWO>(fd, v, a.ph);
  const typename Stored<T>::type f = Stored<T>::of(fd);
  // what this lane gives to and takes from the exchange
  const bool right = lane >= 32;
  const bool gives = right ? (lane >= 64 - 2 * H && lane < 64 - H) : (lane >= H && lane < 2 * H);
  const int give_at = wv * 2 * H + (right ? lane - (64 - 3 * H) : lane - H);
  const bool takes = right ? (lane >= 64 - H && wv < W - 1) : (lane < H && wv > 0);
  const int take_at = right ? (wv + 1) * 2 * H + lane - (64 - H) : (wv - 1) * 2 * H + H + lane;
  auto advance = [&](auto edge) {
    constexpr bool EDGE = decltype(edge)::value;  // some cell of the wave lies beyond a wall
    auto transport = [&]() {
      Site<T> o;
      x_transport_inner<T, AX>(m, o);
      m = o;
      if (EDGE && !c.inside) zero(m);
    };
    int left = a.steps;
    for (int buf = 0;; buf ^= 1) {
      const int n = left < H / S::kXPerStep ? left : H / S::kXPerStep;
#pragma unroll 4
      for (int k = 0; k < n; ++k) {
        transport();
        apply_local<MODE>(m, f, a.ph);
        if (S::kXPerStep == 2) transport();
      }
      left -= n;
      if (left == 0) return;
      union {
        T r[NR];
        uint4 q[PT];
      } u;
      if (gives) {
#pragma unroll
        for (int k = 0; k < NR; ++k) u.r[k] = m.v[C::real_of(k)];
#pragma unroll
        for (int k = 0; k < PT; ++k) ends.q[buf][k][give_at] = u.q[k];
      }
      __syncthreads();
      if (takes) {
#pragma unroll
        for (int k = 0; k < PT; ++k) u.q[k] = ends.q[buf][k][take_at];
#pragma unroll
        for (int k = 0; k < NR; ++k) m.v[C::real_of(k)] = u.r[k];
      }
    }
  };
  // wave-uniform; every wave of the workgroup meets the same barriers in both
  if (c.full)
    advance(std::false_type{});
  else
    advance(std::true_type{});
  const bool mine = lane >= (wv > 0 ? H : 0) && lane < (wv < W - 1 ? 64 - H : 64);
  if (c.inside && mine && pos >= a.halo && pos < a.halo + a.own) C::store(dst, c.x, m);
}

// P = kFirst: the workgroups of blockIdx.y = 0 and 1 advance the two pairs
template <typename T, class S, int W, int AX, int MODE, CellPart P>
__global__ __launch_bounds__(64 * W) void k_line(const T* __restrict__ src, T* __restrict__ dst,
                                                 const double* __restrict__ V, LineArgs a) {
  __shared__ LineEnds<T, W, PartCell<AX, P>::NR> ends;
  if constexpr (P == kFirst) {
    if (blockIdx.y == 0)
      line_pass<T, S, W, AX, MODE, kFirst>(src, dst, V, a, ends);
    else
      line_pass<T, S, W, AX, MODE, kSecond>(src, dst, V, a, ends);
  } else {
    line_pass<T, S, W, AX, MODE, P>(src, dst, V, a, ends);
  }
}

template <typename T, class S, int W, CellPart P, int AX>
const void* line_mode(int mode) {
  switch (mode) {
    case 0: return reinterpret_cast<const void*>(&k_line<T, S, W, AX, 0, P>);
    case 1: return reinterpret_cast<const void*>(&k_line<T, S, W, AX, 1, P>);
    case 2: return reinterpret_cast<const void*>(&k_line<T, S, W, AX, 2, P>);
    default: return nullptr;
  }
}

template <typename T, class S, int W, CellPart P>
const void* line_axis(int axis, int mode) {
  switch (axis) {
    case 0: return line_mode<T, S, W, P, 0>(mode);
    case 1: return line_mode<T, S, W, P, 1>(mode);
    case 2: return line_mode<T, S, W, P, 2>(mode);
    default: return nullptr;
  }
}

// the k_line instance of a kind and a stored cell of nc components, nullptr if
// not built
template <typename T, class S>
const void* line_step(LineKind kind, int axis, int mode, int nc) {
  constexpr int SMALL = kLineWaves, BIG = kLineWavesBig;
  if (nc == 2)
    return kind == kLineBig     ? line_axis<T, S, BIG, kPair>(axis, mode)
           : kind == kLineSmall ? line_axis<T, S, SMALL, kPair>(axis, mode)
                                : nullptr;
  return kind == kLineBig     ? line_axis<T, S, BIG, kAll>(axis, mode)
         : kind == kLineSmall ? line_axis<T, S, SMALL, kAll>(axis, mode)
                              : line_axis<T, S, SMALL, kFirst>(axis, mode);
}

template <typename T>
const void* kernel_line(bool strang, LineKind kind, int axis, int mode, int nc) {
  return strang ? line_step<T, StrangStep>(kind, axis, mode, nc)
                : line_step<T, LieStep>(kind, axis, mode, nc);
}

}  // namespace dirac
