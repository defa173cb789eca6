// Brick decomposition shared by the interpolation and its adjoint: a
// workgroup owns a brick of cells, finds its particles as z-runs of the
// sorted cell list, and touches one node more per axis (plus a two-node halo
// for the gradient).
#pragma once

#include "p3m_internal.h"

namespace p3m {
namespace brick {

constexpr int kThreads = 256;

// v / D for 0 <= v < 4096 by one 24-bit product (the compiler's division by a
// constant takes a 32-bit high product, eight times as long).
template <int D>
struct SmallDiv {
  static constexpr unsigned kM = (1u << 19) / D + 1;
  static constexpr bool exact() {
    for (unsigned v = 0; v < 4096; ++v)
      if ((v * kM) >> 19 != v / D) return false;
    return true;
  }
};
template <int D>
__device__ __forceinline__ int small_div(int v) {
  static_assert(SmallDiv<D>::exact(), "divisor too large for the product");
  return (int)(__umul24((unsigned)v, SmallDiv<D>::kM) >> 19);
}

// The potential of a brick of BX x BX x BZ cells with the two-node gradient
// halo, into LDS: (BX + 5)^2 z-rows, each from four nodes below the brick to
// four above its end, so that a row is whole aligned 16-byte pieces in both
// memories (grids are a multiple of 16 nodes, so a piece never straddles the
// periodic face). Node (x, y, z) relative to the brick's first is at
// phi_at(x, y, z), -2 <= x, y <= BX + 2, -2 <= z <= BZ + 2.
template <int BX, int BZ>
struct PhiRows {
  static constexpr int kX = BX + 5, kZ = BZ + 8;
  static constexpr int kSize = kX * kX * kZ;
  __device__ static int at(int x, int y, int z) { return ((x + 2) * kX + (y + 2)) * kZ + (z + 4); }
};

template <typename T, int BX, int BZ>
__device__ __forceinline__ void load_phi(T* ph, const T* __restrict__ phi, int lg, int bx0,
                                         int by0, int bz0) {
  using R = PhiRows<BX, BZ>;
  constexpr int kV = 16 / sizeof(T), kPieces = R::kZ / kV;      // values a piece, pieces a row
  static_assert(BZ % 16 == 0, "rows of aligned pieces");
  const int mask = (1 << lg) - 1;
  for (int i = threadIdx.x; i < R::kX * R::kX * kPieces; i += kThreads) {
    const int row = small_div<kPieces>(i), v = i - row * kPieces;
    const int nx = small_div<R::kX>(row), ny = row - nx * R::kX;
    const int gx = (bx0 - 2 + nx) & mask, gy = (by0 - 2 + ny) & mask,
              gz = (bz0 - 4 + v * kV) & mask;
    const int4 w = *reinterpret_cast<const int4*>(phi + ((((int64_t)gx << lg) | gy) << lg | gz));
    *reinterpret_cast<int4*>(ph + row * R::kZ + v * kV) = w;
  }
}

// Interpolation bricks of BX x BX x BZ cells: BX^2 z-runs of BZ cells each.
// A deeper brick along z makes a wave's particles longer runs of consecutive
// cells, so that for inputs stored in cell-like order (a lattice) the
// per-particle stores in input order fill longer pieces of cache lines.
template <int BX, int BZ>
struct InterpRuns {
  static constexpr int kR = BX * BX;
  int lo[kR];
  int pre[kR + 1];
};

template <int BX, int BZ>
__device__ inline void load_interp_runs(InterpRuns<BX, BZ>& R, const int32_t* __restrict__ start,
                                        int lg, int bx0, int by0, int bz0) {
  constexpr int kR = InterpRuns<BX, BZ>::kR;
  static_assert(kR <= 64, "one wave scans the run counts");
  const int t = threadIdx.x;
  if (t < kR) {
    int cx = bx0 + t / BX, cy = by0 + t % BX;
    int c0 = (((cx << lg) | cy) << lg) | bz0;
    int lo = start[c0];
    R.lo[t] = lo;
    R.pre[t + 1] = start[c0 + BZ] - lo;           // c0 + BZ <= ng^3: start has ng^3 + 1
  }
  __syncthreads();
  if (t < 64) {
    int v = (t < kR) ? R.pre[t + 1] : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int u = __shfl_up(v, o, 64);
      if (t >= o) v += u;
    }
    if (t < kR) R.pre[t + 1] = v;
    if (t == 0) R.pre[0] = 0;
  }
  __syncthreads();
}

template <int BX, int BZ>
__device__ __forceinline__ int find_interp_run(const InterpRuns<BX, BZ>& R, int f) {
  int lo = 0, hi = InterpRuns<BX, BZ>::kR;        // invariant: pre[lo] <= f < pre[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (R.pre[mid] <= f) lo = mid; else hi = mid;
  }
  return lo;
}

}  // namespace brick
}  // namespace p3m
