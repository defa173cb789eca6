// Cloud-in-cell mass deposit and the fused finite-difference gradient +
// cloud-in-cell interpolation of the long-range (PM) force.
//
// Both kernels work on bricks of grid cells. A particle in cell c
// (offset t = (x - c h)/h in [0,1) per axis) touches the nodes c and c + 1 of
// each axis with weights 1 - t and t (nodes at c h, periodic), so a brick's
// particles touch one node more per axis than it has cells.
//
// Deposit: each brick's nodes add the corner sums of the cells around them (no
// atomics; see k_deposit_cells). The density is rho = sum m W / h^3.
//
// Interpolation (bricks of BX x BX x BZ cells, 4 x 4 x 16): the brick's
// potential plus a two-node halo, (BX + 5)^2 (BZ + 5) values, is staged in
// LDS; the central-difference gradient (order 4:
// [8(phi(c+1) - phi(c-1)) - (phi(c+2) - phi(c-2))] / 12h, or order 2) is formed
// on the (BX + 1)^2 (BZ + 1) nodes in LDS, and each particle takes
// a = -sum_nodes W * grad. The result goes to the sorted-order PM buffer (to be
// combined with the pair sum) or, for the PM-only call, straight to the
// force array in input order as m * a.
#include "brick.h"

namespace p3m {
namespace {

using namespace brick;

// Deposit by cells: the workgroup owns the BX x BY x BZ nodes of its brick
// (every grid node belongs to exactly one brick, so each is written once, with
// no atomics and in a fixed order). A node takes, per axis, the upper-corner
// share of the cell below it and the lower-corner share of its own, so the
// brick needs the cells [-1, B) around it on each axis. One thread a cell sums
// the cell's particles into its eight corners, which go to LDS; then one
// thread a node adds the one corner it takes from each of its eight cells.
// Each particle is read once a brick that sees its cell (1.7 times on
// average) and its weights are formed once. (A node that looped over the
// particles of its eight cells read and weighted each particle eight times:
// 256^3 lattice FP32 362 -> 185 us, clustered 862 -> 373; the cotangent's
// deposit on 2M clustered particles, FP32, 697 -> 213. What is left is the loop over
// a cell's particles, as long as the wave's fullest cell.) NC = 1: mass, scaled by 1 / h^3
// (the density); NC = 3: mass times each component of a cotangent (the
// adjoint's deposit), unscaled, to out[c * ng^3 + node].
//
// A cell with more than kHeavy particles is summed by a whole wave (the lanes
// split its particles), so that a crowded cell does not hold up its brick.
constexpr int kHeavy = 16;

template <typename T, int NC>
__device__ __forceinline__ void add_corners(T (&m)[8 * NC], typename Vec<T>::v4 p,
                                            const typename Vec<T>::v4* __restrict__ lam, int s,
                                            T inv_h) {
  const T tx = p.x * inv_h, ty = p.y * inv_h, tz = p.z * inv_h;
  const T wx[2] = {T(1) - tx, tx}, wy[2] = {T(1) - ty, ty}, wz[2] = {T(1) - tz, tz};
  typename Vec<T>::v4 l;
  if constexpr (NC == 3) l = lam[s];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const T w = wx[q >> 2] * wy[(q >> 1) & 1] * wz[q & 1];
    if constexpr (NC == 1) {
      m[q] += p.w * w;
    } else {
      const T mw = p.w * w;
      m[3 * q] += mw * l.x;
      m[3 * q + 1] += mw * l.y;
      m[3 * q + 2] += mw * l.z;
    }
  }
}

template <typename T, int NC, int BX, int BY, int BZ>
__global__ void __launch_bounds__(kThreads)
k_deposit_cells(const typename Vec<T>::v4* __restrict__ rec,
                const typename Vec<T>::v4* __restrict__ lam, const int32_t* __restrict__ start,
                int ng, int lg, T inv_h, T scale, T* __restrict__ out) {
  constexpr int CY = BY + 1, CZ = BZ + 1, kC = (BX + 1) * CY * CZ;
  __shared__ T corner[8 * NC][kC];
  __shared__ int heavy[kC];
  __shared__ int nheavy;
  const int mask = ng - 1, nbz = ng / BZ, nby = ng / BY;
  const int b = blockIdx.x;
  const int bz0 = (b % nbz) * BZ, by0 = ((b / nbz) % nby) * BY, bx0 = (b / (nbz * nby)) * BX;
  const auto cell_of = [&](int e) {
    const int row = small_div<CZ>(e), ex = small_div<CY>(row);
    const int gx = (bx0 - 1 + ex) & mask, gy = (by0 - 1 + row - ex * CY) & mask,
              gz = (bz0 - 1 + e - row * CZ) & mask;
    return (((gx << lg) | gy) << lg) | gz;
  };
  if (threadIdx.x == 0) nheavy = 0;
  __syncthreads();
  for (int e = threadIdx.x; e < kC; e += kThreads) {
    const int c = cell_of(e);
    const int s0 = start[c], s1 = start[c + 1];
    if (s1 - s0 > kHeavy) {
      heavy[atomicAdd(&nheavy, 1)] = e;
      continue;
    }
    T m[8 * NC];
#pragma unroll
    for (int q = 0; q < 8 * NC; ++q) m[q] = T(0);
    for (int s = s0; s < s1; ++s) add_corners<T, NC>(m, rec[s], lam, s, inv_h);
#pragma unroll
    for (int q = 0; q < 8 * NC; ++q) corner[q][e] = m[q];
  }
  __syncthreads();
  const int nh = nheavy, lane = threadIdx.x & 63;
  for (int k = threadIdx.x >> 6; k < nh; k += kThreads / 64) {
    const int e = heavy[k], c = cell_of(e);
    const int s0 = start[c], s1 = start[c + 1];
    T m[8 * NC];
#pragma unroll
    for (int q = 0; q < 8 * NC; ++q) m[q] = T(0);
    for (int s = s0 + lane; s < s1; s += 64) add_corners<T, NC>(m, rec[s], lam, s, inv_h);
#pragma unroll
    for (int q = 0; q < 8 * NC; ++q) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m[q] += __shfl_xor(m[q], o, 64);
      if (lane == 0) corner[q][e] = m[q];
    }
  }
  __syncthreads();
  const int64_t ncell = (int64_t)1 << (3 * lg);
  for (int node = threadIdx.x; node < BX * BY * BZ; node += kThreads) {
    const int k = node % BZ, j = (node / BZ) % BY, i = node / (BZ * BY);
    T acc[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[q] = T(0);
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      const int e = ((i + (d >> 2)) * CY + (j + ((d >> 1) & 1))) * CZ + (k + (d & 1));
#pragma unroll
      for (int q = 0; q < NC; ++q) acc[q] += corner[NC * (7 - d) + q][e];
    }
    const int64_t g = (((int64_t)(bx0 + i) << lg | (by0 + j)) << lg) | (bz0 + k);
#pragma unroll
    for (int q = 0; q < NC; ++q) out[q * ncell + g] = acc[q] * scale;
  }
}

// Node gradients of a brick in LDS: FP32 as float4 (a corner is one 16-byte
// read), FP64 as three arrays.
template <typename T, int N> struct NodeGrad;
template <int N> struct NodeGrad<float, N> {
  float4 g[N];
  __device__ void put(int i, float x, float y, float z) { g[i] = make_float4(x, y, z, 0.f); }
  __device__ float4 get(int i) const { return g[i]; }
};
template <int N> struct NodeGrad<double, N> {
  double x[N], y[N], z[N];
  __device__ void put(int i, double a, double b, double c) { x[i] = a; y[i] = b; z[i] = c; }
  __device__ double4 get(int i) const { return make_double4(x[i], y[i], z[i], 0.0); }
};

template <typename T, int BX, int BZ>
__global__ void __launch_bounds__(kThreads)
k_interp(const typename Vec<T>::v4* __restrict__ rec, const int32_t* __restrict__ skey,
         const int32_t* __restrict__ start, int ng, int lg, T inv_h, const T* __restrict__ phi,
         T c1, T c2, typename Vec<T>::v4* __restrict__ acc_out, const int32_t* __restrict__ perm,
         int64_t n, void* __restrict__ force, int force_fp32,
         const typename Vec<T>::v4* __restrict__ acc_pp) {
  constexpr int X1 = BX + 1, Z1 = BZ + 1;        // nodes touched per axis
  using PR = PhiRows<BX, BZ>;
  __shared__ __align__(16) T ph[PR::kSize];
  __shared__ __align__(16) NodeGrad<T, X1 * X1 * Z1> gr;
  __shared__ InterpRuns<BX, BZ> R;
  const int mask = ng - 1, nbz = ng / BZ, nbx = ng / BX;
  const int b = blockIdx.x;
  const int bz0 = (b % nbz) * BZ, by0 = ((b / nbz) % nbx) * BX, bx0 = (b / (nbz * nbx)) * BX;
  load_phi<T, BX, BZ>(ph, phi, lg, bx0, by0, bz0);
  load_interp_runs(R, start, lg, bx0, by0, bz0);  // contains __syncthreads
  for (int i = threadIdx.x; i < X1 * X1 * Z1; i += kThreads) {
    const int row = small_div<Z1>(i), nz = i - row * Z1;
    const int nx = small_div<X1>(row), ny = row - nx * X1;
    const int q = PR::at(nx, ny, nz);
    constexpr int sx = PR::kX * PR::kZ, sy = PR::kZ, sz = 1;
    gr.put(i, c1 * (ph[q + sx] - ph[q - sx]) + c2 * (ph[q + 2 * sx] - ph[q - 2 * sx]),
           c1 * (ph[q + sy] - ph[q - sy]) + c2 * (ph[q + 2 * sy] - ph[q - 2 * sy]),
           c1 * (ph[q + sz] - ph[q - sz]) + c2 * (ph[q + 2 * sz] - ph[q - 2 * sz]));
  }
  __syncthreads();
  const int total = R.pre[InterpRuns<BX, BZ>::kR];
  for (int f = threadIdx.x; f < total; f += kThreads) {
    int r = find_interp_run(R, f);
    int s = R.lo[r] + (f - R.pre[r]);
    typename Vec<T>::v4 p = rec[s];
    int lx = r / BX, ly = r % BX, lz = (skey[s] & mask) - bz0;
    T tx = p.x * inv_h, ty = p.y * inv_h, tz = p.z * inv_h;
    T wx[2] = {T(1) - tx, tx}, wy[2] = {T(1) - ty, ty}, wz[2] = {T(1) - tz, tz};
    T ax = 0, ay = 0, az = 0;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          T w = wx[a] * wy[c] * wz[d];
          int q = ((lx + a) * X1 + (ly + c)) * Z1 + (lz + d);
          const typename Vec<T>::v4 g = gr.get(q);
          ax += w * g.x;
          ay += w * g.y;
          az += w * g.z;
        }
    if (acc_out) {
      typename Vec<T>::v4 o;
      o.x = -ax; o.y = -ay; o.z = -az; o.w = T(0);
      acc_out[s] = o;
    } else {
      int64_t i = perm ? perm[s] : s;      // (no permutation: cell order)
      double m = (double)p.w;
      // acc_pp: the pair sum's sorted acceleration, added here (the P3M call
      // whose mesh part ran beside the pair sum)
      double gx = -(double)ax, gy = -(double)ay, gz = -(double)az;
      if (acc_pp) {
        const typename Vec<T>::v4 a = acc_pp[s];
        gx += (double)a.x; gy += (double)a.y; gz += (double)a.z;
      }
      if (force_fp32) {
        float* F = (float*)force;
        F[i] = (float)(m * gx);
        F[n + i] = (float)(m * gy);
        F[2 * n + i] = (float)(m * gz);
      } else {
        double* F = (double*)force;
        F[i] = m * gx;
        F[n + i] = m * gy;
        F[2 * n + i] = m * gz;
      }
    }
  }
}

}  // namespace

template <typename T, int NC, int BX, int BY, int BZ>
void deposit_bricks(p3m_plan* P, const void* lam, T scale, void* out) {
  const unsigned nb = (unsigned)(P->ncell / (BX * BY * BZ));
  k_deposit_cells<T, NC, BX, BY, BZ><<<nb, kThreads, 0, P->stream>>>(
      (const typename Vec<T>::v4*)P->ws.rec, (const typename Vec<T>::v4*)lam, P->ws.start, P->ng,
      P->lg, T(1.0 / P->h), scale, (T*)out);
}

template <typename T>
hipError_t launch_deposit(p3m_plan* P) {
  // Bricks of 4 x 4 x 16 nodes in FP32 (14 KB of corner sums), 4 x 4 x 8 in
  // FP64: 128^3 lattice 24 us (8^3 27, 8 x 8 x 16 32, 4 x 4 x 8 28), FP64 32
  // us (4 x 4 x 16 34, 8^3 38); 2M clustered 53 and 73 us (8^3 62 and 99).
  constexpr int BZ = sizeof(T) == 4 ? 16 : 8;
  deposit_bricks<T, 1, 4, 4, BZ>(P, nullptr, T(1.0 / (P->h * P->h * P->h)), P->ws.grid);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deposit3(p3m_plan* P, const void* lam, void* grids) {
  // 4 x 4 x 16 nodes in FP32 (41 KB of corner sums), 4 x 4 x 8 in FP64 (43 KB:
  // three blocks a CU; 4 x 4 x 16 takes 82 KB, one block). FP64 mesh adjoint,
  // us, 4 x 4 x 16, 4 x 4 x 8, 4^3: 100001 particles on 128^3 331, 282, 285; 2M
  // on 128^3 790, 715, 739, clustered 2305, 1845, 2056; 1M on 256^3 2416, 2039,
  // 2108.
  constexpr int BZ = sizeof(T) == 4 ? 16 : 8;
  deposit_bricks<T, 3, 4, 4, BZ>(P, lam, T(1), grids);
  return hipGetLastError();
}

// One interpolation launch over bricks of BX x BX x BZ cells (one workgroup
// per brick); the grid's edge must be a multiple of BX and BZ.
template <typename T, int BX, int BZ>
hipError_t launch_interp_bricks(p3m_plan* P, int64_t n, void* force_out, int force_fp32,
                                const void* acc_pp, T c1, T c2, void* sorted_out) {
  Workspace& W = P->ws;
  const int nb = (int)(P->ncell / (BX * BX * BZ));
  typename Vec<T>::v4* acc = (typename Vec<T>::v4*)sorted_out;
  k_interp<T, BX, BZ><<<nb, kThreads, 0, P->stream>>>(
      (const typename Vec<T>::v4*)W.rec, W.skey, W.start, P->ng, P->lg, T(1.0 / P->h),
      (const T*)W.grid, c1, c2, acc, P->cell_order ? nullptr : W.perm, n, force_out, force_fp32,
      (const typename Vec<T>::v4*)acc_pp);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_interp(p3m_plan* P, int64_t n, void* force_out, int force_fp32,
                         const void* acc_pp, void* sorted_out) {
  double h = P->h;
  T c1, c2;
  if (P->prm.fd_order == 2) {
    c1 = T(1.0 / (2.0 * h));
    c2 = T(0);
  } else {
    c1 = T(8.0 / (12.0 * h));
    c2 = T(-1.0 / (12.0 * h));
  }
  // Bricks of 4 x 4 x 16 cells (grids are at least 16 cells on a side): a
  // wave's particles are 4 runs of 16 cells. Measured at 128^3 against 8^3
  // bricks: FP32 65 -> 47 us (4 x 4 x 32: the same; 2 x 2 x 64: 55), FP64
  // 77 -> 62 us (4 x 4 x 32: 72, its LDS costing occupancy; 2 x 2 x 32: 72).
  // no force: the sorted mesh acceleration, to sorted_out (default: ws.acc_pm)
  if (!force_out && !sorted_out) sorted_out = P->ws.acc_pm;
  return launch_interp_bricks<T, 4, 16>(P, n, force_out, force_fp32, acc_pp, c1, c2,
                                        force_out ? nullptr : sorted_out);
}

template hipError_t launch_deposit<float>(p3m_plan*);
template hipError_t launch_deposit<double>(p3m_plan*);
template hipError_t launch_deposit3<float>(p3m_plan*, const void*, void*);
template hipError_t launch_deposit3<double>(p3m_plan*, const void*, void*);
template hipError_t launch_interp<float>(p3m_plan*, int64_t, void*, int, const void*, void*);
template hipError_t launch_interp<double>(p3m_plan*, int64_t, void*, int, const void*, void*);

}  // namespace p3m
