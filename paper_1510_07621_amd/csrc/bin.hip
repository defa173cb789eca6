// Counting-sort binning of particles into the cells of the PM grid, and the
// work list of the pair loop.
//
// Cells are the grid's own cells (side h = box / grid_n), indexed
// c = (cx * ng + cy) * ng + cz (z fastest), so each (cx, cy) column of cells is
// one contiguous run of particles after sorting. Steps:
//   1. keys + histogram: cell of each particle; atomic count per cell, whose
//      return value is the particle's rank inside the cell;
//   2. exclusive scan of the counts inside tiles of 2048 cells, and the tiles'
//      totals;
//   3. one launch of three kinds of blocks, each adding the totals of the
//      tiles before a cell's own to its place in the tile: the first slot of
//      every cell (start); scatter + pack, each particle to slot start[c] +
//      rank as a record of its offset from the cell's lower corner (in the
//      path's precision) and its mass, with its input index (perm) and cell
//      (skey); and the pair loop's work items.
// Small sets wait for launches, not for these kernels' work: about 5 us a
// launch from end to end, so that eight kernels in line (scan of the tiles,
// of their totals, add, scatter, three for the items) cost a 4096-particle
// force call 40 us.
// The order inside a cell follows the atomic ranks, so it can differ between
// runs; every later step is a sum, so only rounding depends on it.
#include "p3m_internal.h"

namespace p3m {
namespace {

constexpr int kThreads = 256;
constexpr int kScanItems = 8;                       // per thread
constexpr int kScanTile = kThreads * kScanItems;    // per block
static_assert(kScanItems == 8, "k_scan_tiles moves a thread's values as two int4");
constexpr int kFuseTiles = 1024;    // tiles whose totals each block of the last pass scans

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// Cell coordinate of t = x / h, clamped into [0, ng) (NaN -> 0).
__device__ __forceinline__ int cell_coord(double t, int ng) {
  t = fmax(floor(t), 0.0);
  t = fmin(t, (double)(ng - 1));
  return (int)t;
}

// Consecutive lanes of a wave in the same cell (input already in cell order,
// as a caller that keeps its particles in the order of the last binning
// hands it) share one atomic: the run's first lane adds the run's length
// and each lane's rank is the old count plus its place in the run. With
// input in random order every lane is a run of one. The cells are kept
// (key) for the adjoint's sort of the cotangents only.
__global__ void __launch_bounds__(256)
k_bin_count(int64_t n, const double* __restrict__ pos, int ng, int lg, double inv_h,
            int32_t* __restrict__ key, int32_t* __restrict__ rank,
            int32_t* __restrict__ count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = i < n;
  int c = -1;
  if (valid) {
    int cx = cell_coord(pos[i] * inv_h, ng);
    int cy = cell_coord(pos[n + i] * inv_h, ng);
    int cz = cell_coord(pos[2 * n + i] * inv_h, ng);
    c = (((cx << lg) | cy) << lg) | cz;
    if (key) key[i] = c;
  }
  const int lane = threadIdx.x & 63;
  const int prev = __shfl_up(c, 1, 64);
  const bool head = valid && (lane == 0 || prev != c);
  const unsigned long long heads = __ballot(head);
  // runs end at the next head or at the first lane past n
  const unsigned long long bounds = heads | ~__ballot(valid);
  const unsigned long long upto = lane == 63 ? ~0ull : (2ull << lane) - 1;
  const int start = valid ? 63 - __builtin_clzll(heads & upto) : lane;
  int base = 0;
  if (head) {
    const unsigned long long above = lane == 63 ? 0ull : bounds >> (lane + 1);
    const int len = above ? __builtin_ctzll(above) + 1 : 64 - lane;
    base = atomicAdd(&count[c], len);
  }
  base = __shfl(base, start, 64);
  if (valid) rank[i] = base + (lane - start);
}

// ---- exclusive scan of the cell counts: tiles, then the tiles' totals ----

__device__ __forceinline__ int wave_inclusive(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

// Exclusive scan of one value per thread over the block; returns the block total.
__device__ __forceinline__ int block_exclusive(int v, int* __restrict__ wsum, int& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int inc = wave_inclusive(v);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int base = 0, tot = 0;
  for (int k = 0; k < nw; ++k) {
    int s = wsum[k];
    if (k < w) base += s;
    tot += s;
  }
  __syncthreads();
  total = tot;
  return base + inc - v;
}

// Each tile's exclusive scan and its total; the counts are cleared as they
// are read, so that the next binning starts from zero without a fill pass.
// (Values move as two int4: in and out are 16-byte aligned allocations.)
__global__ void __launch_bounds__(kThreads)
k_scan_tiles(int32_t* __restrict__ in, int32_t* __restrict__ out, int64_t len,
             int32_t* __restrict__ tile_sum) {
  __shared__ int wsum[kThreads / 64];
  int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  // a thread's kScanItems values are 32-byte aligned (in and out are device
  // allocations): whole slices move as two int4, the ragged end one by one
  const bool whole = base + kScanItems <= len;
  int v[kScanItems];
  if (whole) {
    const int4 a = reinterpret_cast<const int4*>(in + base)[0];
    const int4 b = reinterpret_cast<const int4*>(in + base)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    reinterpret_cast<int4*>(in + base)[0] = int4{0, 0, 0, 0};
    reinterpret_cast<int4*>(in + base)[1] = int4{0, 0, 0, 0};
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) v[k] = (base + k < len) ? in[base + k] : 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
      if (base + k < len) in[base + k] = 0;
  }
  int local = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) local += v[k];
  int total;
  int run = block_exclusive(local, wsum, total);
  int e[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    e[k] = run;
    run += v[k];
  }
  if (whole) {
    reinterpret_cast<int4*>(out + base)[0] = int4{e[0], e[1], e[2], e[3]};
    reinterpret_cast<int4*>(out + base)[1] = int4{e[4], e[5], e[6], e[7]};
  } else {
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
      if (base + k < len) out[base + k] = e[k];
  }
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// Single block: exclusive scan of the tile sums in place.
__global__ void __launch_bounds__(1024)
k_scan_sums(int32_t* __restrict__ sums, int nt) {
  __shared__ int wsum[1024 / 64];
  int carry = 0;
  for (int b = 0; b < nt; b += blockDim.x) {
    int i = b + threadIdx.x;
    int v = i < nt ? sums[i] : 0;
    int total;
    int ex = block_exclusive(v, wsum, total);
    if (i < nt) sums[i] = carry + ex;
    carry += total;
  }
}

// ---- the last pass: cell starts, sorted records, work items ----

// What k_bin_finish works on. lstart: each cell's slot within its tile;
// tile: the tiles' totals (NSUM > 0) or their exclusive scan (NSUM 0).
template <typename T>
struct FinishArgs {
  int64_t n;
  const double* __restrict__ pos;
  const double* __restrict__ mass;
  double mass_scalar;
  int ng, lg;
  double h, inv_h;
  const int32_t* __restrict__ rank;
  const int32_t* __restrict__ lstart;
  const int32_t* __restrict__ tile;
  int nt;
  int64_t ncell;
  int32_t* __restrict__ start;
  int32_t* __restrict__ perm;
  int32_t* __restrict__ skey;
  typename Vec<T>::v4* __restrict__ rec;
  int scatter_blocks, start_blocks;     // then the blocks of the work items
  int G, lgG;
  int64_t ngroup;
  int chunk;
  int2* __restrict__ items;
};

// Where the items of the groups from g on begin: g places and one for every
// whole chunk of the particles in the groups before g (x slabs, then y rows
// of the slab, then z; group g's own slab and row column by column).
template <typename T, typename F>
__device__ __forceinline__ int64_t items_before(const FinishArgs<T>& A, const F& first,
                                                int64_t g) {
  if (g >= A.ngroup) return A.ngroup + A.n / A.chunk;
  const int lgd = A.lg - A.lgG, md = (1 << lgd) - 1;
  const int gz = (int)(g & md), gy = (int)((g >> lgd) & md), gx = (int)(g >> (2 * lgd));
  const auto cell = [&](int x, int y, int z) { return (((x << A.lg) | y) << A.lg) | z; };
  int64_t before = first(cell(gx * A.G, 0, 0));
  for (int x = gx * A.G; x < (gx + 1) * A.G; ++x) {
    before += first(cell(x, gy * A.G, 0)) - first(cell(x, 0, 0));
    if (gz)
      for (int y = gy * A.G; y < (gy + 1) * A.G; ++y)
        before += first(cell(x, y, gz * A.G)) - first(cell(x, y, 0));
  }
  return g + before / A.chunk;
}

// NSUM > 0: each block scans the tiles' totals itself, NSUM a thread (one
// launch less; up to kFuseTiles tiles, 128^3 cells, where a block's share is
// 4 KB from the L2). 0: scanned by k_scan_sums.
template <typename T, int NSUM>
__global__ void __launch_bounds__(kThreads)
k_bin_finish(FinishArgs<T> A) {
  __shared__ int off[NSUM ? NSUM * kThreads : 1];
  __shared__ int wsum[kThreads / 64];
  if constexpr (NSUM > 0) {
    int v[NSUM], local = 0, total;
#pragma unroll
    for (int k = 0; k < NSUM; ++k) {
      const int t = (int)threadIdx.x * NSUM + k;
      v[k] = t < A.nt ? A.tile[t] : 0;
      local += v[k];
    }
    int run = block_exclusive(local, wsum, total);
#pragma unroll
    for (int k = 0; k < NSUM; ++k) {
      off[threadIdx.x * NSUM + k] = run;
      run += v[k];
    }
    __syncthreads();
  }
  const auto offset = [&](int t) { return NSUM ? off[t] : A.tile[t]; };
  const auto first = [&](int64_t c) {       // first slot of cell c; of c = ncell: n
    return c < A.ncell ? A.lstart[c] + offset((int)(c / kScanTile)) : (int)A.n;
  };
  int b = blockIdx.x;
  if (b < A.scatter_blocks) {
    const int64_t n = A.n, i = (int64_t)b * kThreads + threadIdx.x;
    if (i >= n) return;
    // the cell again, as k_bin_count formed it: the positions are read anyway
    const double x = A.pos[i], y = A.pos[n + i], z = A.pos[2 * n + i];
    const int cx = cell_coord(x * A.inv_h, A.ng), cy = cell_coord(y * A.inv_h, A.ng),
              cz = cell_coord(z * A.inv_h, A.ng);
    const int c = (((cx << A.lg) | cy) << A.lg) | cz;
    const int dst = first(c) + A.rank[i];
    typename Vec<T>::v4 r;
    r.x = (T)(x - cx * A.h);
    r.y = (T)(y - cy * A.h);
    r.z = (T)(z - cz * A.h);
    r.w = (T)(A.mass ? A.mass[i] : A.mass_scalar);
    A.rec[dst] = r;
    // (a deposit reads neither: for particles in random order each of these
    // stores is a cache line of its own. Power spectrum of 16.7M clustered
    // particles on 256^3 2408 -> 1926 us, 2M on 128^3 in FP64 323 -> 272, of a
    // 128^3 lattice, whose lines are shared, 135.6 -> 133.5)
    if (A.perm) {
      A.perm[dst] = (int32_t)i;
      A.skey[dst] = c;
    }
    return;
  }
  b -= A.scatter_blocks;
  if (b < A.start_blocks) {
    // one tile: whole tiles as int4 (consecutive threads, consecutive 16
    // bytes), the ragged last tile one value at a time
    const int64_t base = (int64_t)b * kScanTile;
    const int add = offset(b);
    if (base + kScanTile <= A.ncell) {
      const int4* in = reinterpret_cast<const int4*>(A.lstart + base);
      int4* out = reinterpret_cast<int4*>(A.start + base);
      for (int k = threadIdx.x; k < kScanTile / 4; k += kThreads) {
        int4 q = in[k];
        q.x += add; q.y += add; q.z += add; q.w += add;
        out[k] = q;
      }
    } else {
      for (int64_t c = base + threadIdx.x; c < A.ncell; c += kThreads)
        A.start[c] = A.lstart[c] + add;
    }
    if (b == 0 && threadIdx.x == 0) A.start[A.ncell] = (int)A.n;
    return;
  }
  b -= A.start_blocks;
  // One group a thread: its chunks (the particles of its G x G z-runs over the
  // chunk), in group order. All groups before g together have at most
  // g + (their particles) / chunk items, so the block's list begins there (no
  // block needs another's counts), and the places up to the next block's
  // beginning are marked empty. (Appended by atomics, the blocks' order was
  // free and neighbouring groups no longer ran together: 128^3 lattice FP32
  // 2.39 -> 2.46 ms.)
  const int64_t g0 = (int64_t)b * kThreads;
  const int64_t base = items_before(A, first, g0);
  const int64_t next = items_before(A, first, min(g0 + kThreads, A.ngroup));
  const int64_t g = g0 + threadIdx.x;
  int nc = 0, total;
  if (g < A.ngroup) {
    const int lgd = A.lg - A.lgG, md = (1 << lgd) - 1;
    const int gz = (int)(g & md), gy = (int)((g >> lgd) & md), gx = (int)(g >> (2 * lgd));
    int cnt = 0;
    for (int x = 0; x < A.G; ++x)
      for (int y = 0; y < A.G; ++y) {
        const int c0 = ((((gx * A.G + x) << A.lg) | (gy * A.G + y)) << A.lg) | (gz * A.G);
        cnt += first(c0 + A.G) - first(c0);
      }
    nc = (cnt + A.chunk - 1) / A.chunk;
  }
  const int64_t at = base + block_exclusive(nc, wsum, total);
  for (int c = 0; c < nc; ++c) A.items[at + c] = make_int2((int)g, c);
  for (int64_t i = base + total + threadIdx.x; i < next; i += kThreads)
    A.items[i] = make_int2(-1, 0);
}

inline unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

int scan_tiles(int64_t ncell) { return (int)((ncell + kScanTile - 1) / kScanTile); }

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t b = (n + kThreads - 1) / kThreads;
  unsigned blocks = (unsigned)(b < 65536 ? b : 65536);
  k_fill_i32<<<blocks, kThreads, 0, s>>>(p, n, v);
  return hipGetLastError();
}

// How a call's particles are cut into work items: chunks of `chunk`
// i-particles, each summed by item_waves waves that share its stencil. A
// whole item (64 particles, one wave) takes 150 to 300 us from end to end, so
// a set with fewer items than wave slots leaves most of the chip idle and
// lasts that long whatever its size; a cut item stages its stencil for fewer
// particles, which costs more in all. Short-range calls, binning included, us,
// as (chunk, waves):
//   n <= 8192, (16, 8): 4096 on 16^3, FP32 (64, 1) 290, (16, 4) 44, (16, 8)
//     39; FP64 adjoint (16, 4) 81, (16, 8) 72
//   n <= 24576, (16, 4): 16000 on 16^3, FP32 (32, 4) 141, (16, 4) 102, (16, 8)
//     120; FP64 274, 192, 202
//   n <= 65536, (32, 4), FP64 (16, 4): 32768 on 32^3, FP32 (32, 2) 117, (32, 4)
//     84, (16, 4) 87; FP64 (32, 4) 152, (16, 4) 150, adjoint 242, 221
//   n <= 3 2^17, (32, 2), FP64 (32, 4): 64^3 on 64^3, FP32 (32, 1) 405, (32, 2)
//     372, (32, 4) 379; FP64 (32, 2) 829, (32, 4) 791, adjoint 1303, 1245
//   n <= 3 2^18, (32, 2): 80^3 on 64^3, FP32 (32, 1) 1083, (32, 2) 1056; FP64
//     2620, 2526
//   n <= 3 2^20, (32, 1): the last items end sooner and their boxes clip more:
//     2M clustered on 128^3 FP32 (64, 1) 2887, (32, 1) 2761, FP64 6844, 6426;
//     128^3 lattice 2402, 2290 and 5618, 5584
//   above, (64, 1): 16.7M clustered FP32, both sides: 41.6 against 43.1 ms
// Groups that are sparse (under 16 particles on average) have one item each,
// enough of them to fill the chip: sharing those measured slower (FP32 300007
// on 128^3: (32, 1) 279, (32, 2) 302).
static void pair_split(p3m_plan* P, int64_t n) {
  const bool f64 = P->prm.precision == P3M_FP64;
  P->item_waves = 1;
  P->chunk = n <= int64_t{3} << 20 ? 32 : kChunk;
  if (n < 16 * P->ngroup) return;
  if (n <= 8192) {
    P->item_waves = 8;
    P->chunk = 16;
  } else if (n <= 65536) {
    P->item_waves = 4;
    if (f64 || n <= 24576) P->chunk = 16;
  } else if (n <= int64_t{3} << 17) {
    P->item_waves = f64 ? 4 : 2;
  } else if (n <= int64_t{3} << 18) {
    P->item_waves = 2;
  }
}

template <typename T>
static hipError_t launch_finish(p3m_plan* P, int64_t n, const double* pos, const double* mass,
                                double mass_scalar, Items items) {
  Workspace& W = P->ws;
  FinishArgs<T> A{};
  A.n = n;
  A.pos = pos;
  A.mass = mass;
  A.mass_scalar = mass_scalar;
  A.ng = P->ng;
  A.lg = P->lg;
  A.h = P->h;
  A.inv_h = 1.0 / P->h;
  A.rank = W.rank;
  A.lstart = W.lstart;
  A.tile = W.scan_tmp;
  A.nt = scan_tiles(P->ncell);
  A.ncell = P->ncell;
  A.start = W.start;
  A.perm = items == Items::kRecords ? nullptr : W.perm;
  A.skey = W.skey;
  A.rec = (typename Vec<T>::v4*)W.rec;
  A.scatter_blocks = (int)blocks_for(n, kThreads);
  A.start_blocks = A.nt;
  A.G = P->G;
  A.lgG = P->lgG;
  A.ngroup = P->ngroup;
  A.chunk = P->chunk;
  A.items = W.items;
  const unsigned blocks = (unsigned)(A.scatter_blocks + A.start_blocks) +
                          (items <= Items::kNone ? 0 : blocks_for(P->ngroup, kThreads));
  if (A.nt <= kThreads)
    k_bin_finish<T, 1><<<blocks, kThreads, 0, P->stream>>>(A);
  else if (A.nt <= kFuseTiles)
    k_bin_finish<T, kFuseTiles / kThreads><<<blocks, kThreads, 0, P->stream>>>(A);
  else
    k_bin_finish<T, 0><<<blocks, kThreads, 0, P->stream>>>(A);
  return hipGetLastError();
}

hipError_t launch_bin(p3m_plan* P, int64_t n, const double* pos, const double* mass,
                      double mass_scalar, Items items) {
  Workspace& W = P->ws;
  hipStream_t s = P->stream;
  hipError_t e;
  P->chunk = kChunk;
  P->item_waves = 1;
  if (items == Items::kCut) pair_split(P, n);
  // The counts start at zero: cleared by the previous binning's scan, or
  // here when that binning did not get as far (a failed launch)
  if (P->count_dirty && (e = launch_fill_i32(W.count, P->ncell, 0, s)) != hipSuccess) return e;
  P->count_dirty = 1;
  k_bin_count<<<blocks_for(n, kThreads), kThreads, 0, s>>>(n, pos, P->ng, P->lg, 1.0 / P->h,
                                                           W.key, W.rank, W.count);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int nt = scan_tiles(P->ncell);
  k_scan_tiles<<<nt, kThreads, 0, s>>>(W.count, W.lstart, P->ncell, W.scan_tmp);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  P->count_dirty = 0;
  if (nt > kFuseTiles) {
    k_scan_sums<<<1, 1024, 0, s>>>(W.scan_tmp, nt);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return P->prm.precision == P3M_FP32
             ? launch_finish<float>(P, n, pos, mass, mass_scalar, items)
             : launch_finish<double>(P, n, pos, mass, mass_scalar, items);
}

}  // namespace p3m
