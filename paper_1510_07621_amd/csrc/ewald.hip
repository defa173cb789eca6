// PP gravity with a tabulated Ewald correction (the guide's PP-with-Ewald
// kick: CONCEPT User's Guide, Ch. 5 entries use_Ewald and ewald_gridsize;
// Ch. 8 test kick_PP_with_Ewald), for small-N validation of the P3M path.
//
// Periodic field of a unit point mass at the origin with its images in a
// neutralising background, as a multiple of -G:
//   e(r) = sum_n r_n g(|r_n|) + (4 pi / L^3) sum_{k != 0} (k / k^2) e^{-k^2/(4 a^2)} sin(k . r),
//   g(s) = (erfc(a s) + (2 a s / sqrt(pi)) e^{-a^2 s^2}) / s^3,  r_n = r + n L,
// independent of the splitting a (here a = 2 / L, real images to erfc(7),
// Fourier terms to e^{-40}). The correction c(r) = e(r) - r / |r|^3 (the
// periodic images and the background, without the minimum-image Newtonian
// term) is smooth over the minimum-image cell and odd in each coordinate,
// so one octant [0, L/2]^3 of the ewald_gridsize^3 node grid (spacing
// L / ewald_gridsize) holds it: node (i, j, k), 0 <= i, j, k <= E/2. Between
// nodes it is trilinear in |r_d|, with the sign of r_d per component.
//
// The pair sum: F_i = -G m_i sum_{j != i} m_j [ r / (|r|^2 + eps^2)^(3/2) + c(r) ],
// r the minimum-image separation, all pairs, in FP64. A pair at zero
// separation contributes nothing.
#include <algorithm>

#include "p3m_internal.h"

namespace p3m {
namespace {

constexpr int kEwI = 64;                       // i-particles per block of the pair sum
constexpr int kEwWaves = 16;                   // waves per block, each on a share of the j's
constexpr int kEwThreads = kEwI * kEwWaves;

// c(r) at one octant node, in FP64.
__global__ void __launch_bounds__(256)
k_ewald_table(int E, double box, double4* __restrict__ tab) {
  const int H = E / 2 + 1;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= H * H * H) return;
  const int i = idx / (H * H), j = (idx / H) % H, k = idx % H;
  const double h = box / E;
  const double rx = i * h, ry = j * h, rz = k * h;
  const double a = 2.0 / box;
  const double kTwoOverSqrtPi = 1.1283791670955126;
  double cx = 0, cy = 0, cz = 0;
  if (i | j | k) {
    // real space: every image within erfc(7); the minimum image (n = 0) with
    // its Newtonian part removed, written so that small |r| does not cancel
    const double span = 7.0 / a;
    const int nmax = (int)ceil(span / box) + 1;
    for (int nx = -nmax; nx <= nmax; ++nx)
      for (int ny = -nmax; ny <= nmax; ++ny)
        for (int nz = -nmax; nz <= nmax; ++nz) {
          const double px = rx + nx * box, py = ry + ny * box, pz = rz + nz * box;
          const double s2 = px * px + py * py + pz * pz;
          const double s = sqrt(s2);
          if (s > span) continue;
          const double as = a * s;
          const double gauss = kTwoOverSqrtPi * as * exp(-as * as);
          double f;
          if (nx == 0 && ny == 0 && nz == 0)
            f = (gauss - erf(as)) / (s2 * s);     // erfc - 1 = -erf
          else
            f = (erfc(as) + gauss) / (s2 * s);
          cx += px * f;
          cy += py * f;
          cz += pz * f;
        }
    // Fourier space: (4 pi / L^3) sum (k / k^2) e^{-k^2/(4 a^2)} sin(k . r)
    const double kf = 2.0 * M_PI / box;
    const int mmax = (int)ceil(sqrt(40.0) * 2.0 * a / kf);
    const double pref = 4.0 * M_PI / (box * box * box);
    for (int mx = -mmax; mx <= mmax; ++mx)
      for (int my = -mmax; my <= mmax; ++my)
        for (int mz = -mmax; mz <= mmax; ++mz) {
          const int m2 = mx * mx + my * my + mz * mz;
          if (m2 == 0) continue;
          const double k2 = kf * kf * m2;
          const double w = exp(-k2 / (4.0 * a * a));
          if (w < 4e-18) continue;
          const double sn = sin(kf * (mx * rx + my * ry + mz * rz));
          const double c = pref * w / k2 * sn;
          cx += c * kf * mx;
          cy += c * kf * my;
          cz += c * kf * mz;
        }
  }
  tab[idx] = make_double4(cx, cy, cz, 0.0);
}

// The node table regrouped for the interpolation: entry (i, j, k), k < E/2,
// holds c at nodes (i, j, k) and (i, j, k + 1) as three double2 (48 bytes,
// 16-byte aligned), so the two z-corners of a trilinear cell come in three
// aligned 16-byte loads instead of the four that two padded double4 nodes
// take.
__global__ void __launch_bounds__(256)
k_ewald_zpairs(int E, const double4* __restrict__ tab, double2* __restrict__ zp) {
  const int H = E / 2 + 1;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= H * H * (H - 1)) return;
  const int col = idx / (H - 1), k = idx % (H - 1);
  const double4 a = tab[col * H + k], b = tab[col * H + k + 1];
  zp[3 * idx + 0] = make_double2(a.x, a.y);
  zp[3 * idx + 1] = make_double2(a.z, b.x);
  zp[3 * idx + 2] = make_double2(b.y, b.z);
}

// Trilinear c(r) from the octant table (z-pair layout), r a minimum-image
// separation.
__device__ __forceinline__ double3 ewald_corr(const double2* __restrict__ zp, int E,
                                              double inv_h, double dx, double dy, double dz) {
  const int H = E / 2 + 1;
  // clamped to the octant (also keeps a non-finite input inside the table)
  const double top = H - 1.0;
  const double ux = fmin(fabs(dx) * inv_h, top), uy = fmin(fabs(dy) * inv_h, top),
               uz = fmin(fabs(dz) * inv_h, top);
  const int ix = min((int)ux, H - 2), iy = min((int)uy, H - 2), iz = min((int)uz, H - 2);
  const double tx = ux - ix, ty = uy - iy, tz = uz - iz;
  double3 c = make_double3(0.0, 0.0, 0.0);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const double wxy = (a ? tx : 1.0 - tx) * (b ? ty : 1.0 - ty);
      const double2* e = zp + 3 * (((ix + a) * H + (iy + b)) * (H - 1) + iz);
      const double2 v0 = e[0], v1 = e[1], v2 = e[2];
      const double w0 = wxy * (1.0 - tz), w1 = wxy * tz;
      c.x += w0 * v0.x + w1 * v1.y;
      c.y += w0 * v0.y + w1 * v2.x;
      c.z += w0 * v1.x + w1 * v2.y;
    }
  c.x = dx < 0 ? -c.x : c.x;
  c.y = dy < 0 ? -c.y : c.y;
  c.z = dz < 0 ? -c.z : c.z;
  return c;
}

__device__ __forceinline__ double min_image(double d, double box, double inv_box) {
  return d - box * rint(d * inv_box);
}

// All pairs, j tiles in LDS. A block holds kEwI i-particles, one per lane,
// and kEwWaves waves that each take their own contiguous share of every j
// tile, so a small n still spreads over every CU with several waves per SIMD
// to cover the latency of the table's gathers. The i- and j-particles are
// both taken in cell order (order[s] is the input index of sorted slot s): a
// block's i's sit in a few neighbouring cells, so for one broadcast j its
// lanes' separations fall on nearby table nodes that share cache lines, and
// consecutive j's are neighbours, so consecutive steps revisit those lines.
// The waves' partial sums are added in wave order at the end (no atomics),
// so the summation order is the sorted order. Within a cell that order is
// the binning's atomic rank, which may differ between calls: the result can
// change at rounding level from call to call, like the P3M force.
__global__ void __launch_bounds__(kEwThreads)
k_pp_ewald(int64_t n, const double* __restrict__ pos, const double* __restrict__ mass,
           double ms, double box, double eps2, double negG, const double2* __restrict__ tab,
           int E, const int32_t* __restrict__ order, void* __restrict__ force,
           int force_fp32) {
  __shared__ double4 tile[kEwThreads];
  __shared__ double red[3][kEwWaves][kEwI];
  const int lane = threadIdx.x % kEwI, wave = threadIdx.x / kEwI;
  const int64_t slot = (int64_t)blockIdx.x * kEwI + lane;
  const bool live = slot < n;
  const int64_t i = live ? (int64_t)order[slot] : -1;
  const double xi = live ? pos[i] : 0.0, yi = live ? pos[n + i] : 0.0,
               zi = live ? pos[2 * n + i] : 0.0;
  const double inv_box = 1.0 / box, inv_h = E / box;
  double ax = 0, ay = 0, az = 0;
  for (int64_t j0 = 0; j0 < n; j0 += kEwThreads) {
    const int64_t jl = j0 + threadIdx.x;
    __syncthreads();
    if (jl < n) {
      const int64_t j = order[jl];
      tile[threadIdx.x] = make_double4(pos[j], pos[n + j], pos[2 * n + j], mass ? mass[j] : ms);
    }
    __syncthreads();
    // this wave's entries [tb, tb + cnt) of the tile (cnt <= 0 past the end)
    const int tb = wave * kEwI;
    const int64_t jb = j0 + tb;
    const int cnt = (int)min<int64_t>(kEwI, n - jb);
    for (int t = 0; t < cnt; ++t) {
      const double4 pj = tile[tb + t];
      const double dx = min_image(xi - pj.x, box, inv_box);
      const double dy = min_image(yi - pj.y, box, inv_box);
      const double dz = min_image(zi - pj.z, box, inv_box);
      const double r2 = dx * dx + dy * dy + dz * dz;
      if (!live || jb + t == slot || r2 == 0.0) continue;
      const double inv = rsqrt(r2 + eps2);
      const double w = inv * inv * inv;
      const double3 c = ewald_corr(tab, E, inv_h, dx, dy, dz);
      ax += pj.w * (dx * w + c.x);
      ay += pj.w * (dy * w + c.y);
      az += pj.w * (dz * w + c.z);
    }
  }
  red[0][wave][lane] = ax;
  red[1][wave][lane] = ay;
  red[2][wave][lane] = az;
  __syncthreads();
  if (wave != 0 || !live) return;
  ax = ay = az = 0;
#pragma unroll
  for (int w = 0; w < kEwWaves; ++w) {
    ax += red[0][w][lane];
    ay += red[1][w][lane];
    az += red[2][w][lane];
  }
  const double m = mass ? mass[i] : ms;
  const double fx = negG * m * ax, fy = negG * m * ay, fz = negG * m * az;
  if (force_fp32) {
    float* F = (float*)force;
    F[i] = (float)fx;
    F[n + i] = (float)fy;
    F[2 * n + i] = (float)fz;
  } else {
    double* F = (double*)force;
    F[i] = fx;
    F[n + i] = fy;
    F[2 * n + i] = fz;
  }
}

// All pairs once: both terms of a pair are odd in the separation, so the force
// on j is minus the one on i. The particles of the cell order are cut into
// blocks of 64 and superblocks of kRotWaves blocks; a workgroup takes a pair
// (I, J >= I) of superblocks, wave w the block w of I, one i a lane. For each
// block of J a lane also holds one j, and the j's go round the wave lane by
// lane (DPP wave_rol, their sums with them): in step s lane l evaluates i_l
// with j_(l + s). Each particle's sum over a superblock has one writer, row J
// of `part` for the i's and row I for the j's (the waves' shares of a j added
// in wave order in LDS first), and k_ewald_combine adds the rows in order. A
// superblock with itself is evaluated from both sides, without the j's share.
// blockIdx.y: a share of the 64 steps, with rows of its own, for sets with too
// few superblock pairs.
//
// What bounds the sum is the vector cache's rate of handing out a trilinear
// cell's corners, 192 bytes a lane and pair: 60 accesses of the cache for a
// 16-byte load of 64 lanes (TCP_TOTAL_CACHE_ACCESSES), 12 loads a step, and
// 560 cycles a step and CU, of which arithmetic needs 180. Each pair once
// halves the corners fetched. k_pp_ewald, then this kernel, 64^3 table: 32768
// uniform particles 13.76 -> 7.80 ms, 20001 8.91 -> 4.10, 5000 1.12 -> 0.38;
// 32768 clustered, 32^3 table 8.91 -> 5.12. (The table's columns of a tile
// copied to LDS instead: 11.7 ms from both sides, bank conflicts taking 60 %
// of the LDS time.)
constexpr int kRotWaves = 8;
constexpr int kRotSuper = 64 * kRotWaves;     // particles of a superblock

__device__ __forceinline__ int wave_next(int v) {      // the next lane's value, round the wave
  return __builtin_amdgcn_update_dpp(0, v, 0x134, 0xF, 0xF, false);
}
__device__ __forceinline__ double wave_next(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = wave_next((int)b), hi = wave_next((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__global__ void __launch_bounds__(kRotSuper, 4)
k_pp_ewald_blocks(int64_t n, const double* __restrict__ pos, const double* __restrict__ mass,
                  double ms, double box, double eps2, const double2* __restrict__ tab, int E,
                  int nsuper, const int32_t* __restrict__ order, double* __restrict__ part) {
  __shared__ double red[3][kRotWaves][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the superblock pair: the blockIdx.x-th of (0, 0), (0, 1), .., (1, 1), ..
  int I = 0, J = blockIdx.x;
  while (J >= nsuper - I) {
    J -= nsuper - I;
    ++I;
  }
  J += I;
  const int steps = 64 / gridDim.y, s0 = steps * blockIdx.y;
  const double inv_box = 1.0 / box, inv_h = E / box;
  const auto load = [&](int64_t slot, double& x, double& y, double& z, double& m) {
    x = y = z = m = 0.0;                 // past the end: no mass
    if (slot < n) {
      const int64_t p = order[slot];
      x = pos[p];
      y = pos[n + p];
      z = pos[2 * n + p];
      m = mass ? mass[p] : ms;
    }
  };
  const int64_t islot = (int64_t)I * kRotSuper + threadIdx.x;
  double xi, yi, zi, mi;
  load(islot, xi, yi, zi, mi);
  double ax = 0, ay = 0, az = 0;
  for (int b = 0; b < kRotWaves; ++b) {
    const int64_t j0 = (int64_t)J * kRotSuper + 64 * b;
    if (j0 >= n) break;                  // (uniform)
    int jl = (lane + s0) & 63;           // the j this lane starts with
    double xj, yj, zj, mj, bx = 0, by = 0, bz = 0;
    load(j0 + jl, xj, yj, zj, mj);
    for (int s = 0; s < steps; ++s) {
      const double dx = min_image(xi - xj, box, inv_box);
      const double dy = min_image(yi - yj, box, inv_box);
      const double dz = min_image(zi - zj, box, inv_box);
      const double r2 = dx * dx + dy * dy + dz * dz;
      // (a pair at zero separation: finite weight times zero, and c(0) = 0; a
      // j without mass, as the places past the end at the origin have none:
      // finite weight times no mass, however close the pair. With a test on jl
      // instead the compiler issues the corners' loads later: 7.82 -> 9.16 ms
      // for 32768 particles and a 64^3 table)
      const double inv = rsqrt_pos((r2 > 0.0) & (mj != 0.0) ? r2 + eps2 : 1.0);
      const double w = inv * inv * inv;
      const double3 c = ewald_corr(tab, E, inv_h, dx, dy, dz);
      const double tx = dx * w + c.x, ty = dy * w + c.y, tz = dz * w + c.z;
      ax += mj * tx;
      ay += mj * ty;
      az += mj * tz;
      bx -= mi * tx;
      by -= mi * ty;
      bz -= mi * tz;
      xj = wave_next(xj);
      yj = wave_next(yj);
      zj = wave_next(zj);
      mj = wave_next(mj);
      bx = wave_next(bx);
      by = wave_next(by);
      bz = wave_next(bz);
      jl = wave_next(jl);
    }
    if (I == J) continue;                // (uniform)
    __syncthreads();                     // the last block's shares are read
    red[0][wave][jl] = bx;
    red[1][wave][jl] = by;
    red[2][wave][jl] = bz;
    __syncthreads();
    if (threadIdx.x < 3 * 64 && j0 + lane < n) {
      double sum = 0;
#pragma unroll
      for (int v = 0; v < kRotWaves; ++v) sum += red[wave][v][lane];
      part[3 * (((int64_t)blockIdx.y * nsuper + I) * n + j0 + lane) + wave] = sum;
    }
  }
  if (islot < n) {
    double* out = part + 3 * (((int64_t)blockIdx.y * nsuper + J) * n + islot);
    out[0] = ax;
    out[1] = ay;
    out[2] = az;
  }
}

// F of each particle, in input order, from the rows of sums.
__global__ void __launch_bounds__(256)
k_ewald_combine(int64_t n, const double* __restrict__ part, int rows,
                const int32_t* __restrict__ order, const double* __restrict__ mass, double ms,
                double negG, void* __restrict__ force, int force_fp32) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= 3 * n) return;
  const int64_t slot = k / 3;
  const int d = (int)(k - 3 * slot);
  const int64_t i = order[slot];
  double a = 0;
#pragma unroll 8
  for (int r = 0; r < rows; ++r) a += part[(int64_t)r * 3 * n + k];
  const double f = negG * (mass ? mass[i] : ms) * a;
  if (force_fp32)
    ((float*)force)[d * n + i] = (float)f;
  else
    ((double*)force)[d * n + i] = f;
}

// The interpolated correction at given minimum-image separations.
__global__ void __launch_bounds__(256)
k_ewald_eval(int64_t npts, const double* __restrict__ r, double box,
             const double2* __restrict__ tab, int E, double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npts) return;
  const double inv_box = 1.0 / box;
  const double dx = min_image(r[p], box, inv_box), dy = min_image(r[npts + p], box, inv_box),
               dz = min_image(r[2 * npts + p], box, inv_box);
  const double3 c = ewald_corr(tab, E, E / box, dx, dy, dz);
  out[p] = c.x;
  out[npts + p] = c.y;
  out[2 * npts + p] = c.z;
}

}  // namespace

static int ewald_supers(int64_t n) { return (int)((n + kRotSuper - 1) / kRotSuper); }

int64_t ewald_part_size(int64_t n_max) {
  const int64_t n = std::min(n_max, kEwaldBlocksMax);
  return 3 * n * std::max<int64_t>(kEwaldRows, ewald_supers(n));
}

hipError_t launch_ewald_table(p3m_plan* P) {
  const int E = P->prm.ewald_gridsize, H = E / 2 + 1;
  const int total = H * H * H;
  k_ewald_table<<<(total + 255) / 256, 256, 0, P->stream>>>(E, P->prm.box,
                                                           (double4*)P->ws.ewald_tab);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int pairs = H * H * (H - 1);
  k_ewald_zpairs<<<(pairs + 255) / 256, 256, 0, P->stream>>>(
      E, (const double4*)P->ws.ewald_tab, (double2*)P->ws.ewald_zpair);
  return hipGetLastError();
}

hipError_t launch_pp_ewald(p3m_plan* P, int64_t n, const double* pos, const double* mass,
                           double ms, const int32_t* order, void* force, int force_fp32) {
  if (n <= kEwaldBlocksMax) {
    const int nsuper = ewald_supers(n);
    const int pairs = nsuper * (nsuper + 1) / 2;
    // Shares of the 64 steps: what a set of few superblocks waits for is a
    // block's steps in line. From both sides, up to 8 shares, up to 32, us:
    // 200 particles 55, 61, 27; 400 96, 102, 39; 1100 232, 119, 72; 2000 378,
    // 122, 77.
    int shares = 1;
    while (shares < 32 && pairs * shares < 1024 && 2 * shares * nsuper <= kEwaldRows) shares *= 2;
    k_pp_ewald_blocks<<<dim3((unsigned)pairs, (unsigned)shares), kRotSuper, 0, P->stream>>>(
        n, pos, mass, ms, P->prm.box, P->eps * P->eps, (const double2*)P->ws.ewald_zpair,
        P->prm.ewald_gridsize, nsuper, order, P->ws.ewald_part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_ewald_combine<<<(unsigned)((3 * n + 255) / 256), 256, 0, P->stream>>>(
        n, P->ws.ewald_part, nsuper * shares, order, mass, ms, -P->prm.G, force, force_fp32);
    return hipGetLastError();
  }
  const unsigned blocks = (unsigned)((n + kEwI - 1) / kEwI);
  k_pp_ewald<<<blocks, kEwThreads, 0, P->stream>>>(
      n, pos, mass, ms, P->prm.box, P->eps * P->eps, -P->prm.G,
      (const double2*)P->ws.ewald_zpair, P->prm.ewald_gridsize, order, force, force_fp32);
  return hipGetLastError();
}

hipError_t launch_ewald_eval(p3m_plan* P, int64_t npts, const double* r, double* out) {
  k_ewald_eval<<<(unsigned)((npts + 255) / 256), 256, 0, P->stream>>>(
      npts, r, P->prm.box, (const double2*)P->ws.ewald_zpair, P->prm.ewald_gridsize, out);
  return hipGetLastError();
}

}  // namespace p3m
