// Short-range force without a plan: pp_force_noalloc, for callers that
// cannot allocate device memory. Its workspace (binning arrays, work list,
// stencil rows, split tables, sorted records) is carved from one file-scope
// device array of fixed size; the stencil and the split table are computed
// on the host (once while the parameters stay) and handed over in the
// arguments of the call's first kernels, 960 words each: one launch for the 260
// words of an FP32 table and up to 700 stencil rows (one word a row), two for
// an FP64 table's 910 words and more than 50 rows, at most six. The arithmetic
// is that of pp_force (the same kernels), with every pair evaluated from
// both sides.
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>

#include "p3m_internal.h"

namespace {

constexpr size_t kScratchBytes = size_t{12} << 20;
constexpr int kMaxDevices = 64;
constexpr int kMaxRows = 4096;

// The workspace of every pp_force_noalloc call on a device. In host code the
// name stands for the host-side shadow of the symbol; device addresses come
// from hipGetSymbolAddress, one per device.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kTabWords = 2 * p3m::kSplitCoef64 * (p3m::kSplitBins + 1);   // the longer table

// The stencil rows and the split table of a set of parameters, as the words
// k_setup unpacks. The last set is kept, by its values: a program that calls
// in a loop keeps its parameters, and the fit of the table takes 0.2 (FP32)
// to 0.6 ms (FP64) of host time, the call's kernels 0.1 ms.
struct HostTables {
  bool valid = false;
  int precision = 0, G = 0;
  double cutoff_rs = 0, soft_rs = 0, radius = 0;
  p3m::SplitMap map{};
  int nrows = 0, ntab = 0;
  uint32_t words[kMaxRows + kTabWords];     // rows, then the table
};

std::mutex g_mutex;                       // the address table and the tables below
void* g_scratch[kMaxDevices] = {};
HostTables g_tables;
int32_t g_rows[4 * kMaxRows];

// Makes g_tables those of plan P (P->nrows <= kMaxRows checked before).
void make_tables(const p3m_plan& P) {
  HostTables& H = g_tables;
  const p3m_params& q = P.prm;
  const double soft = q.softening / P.r_s, radius = P.r_c / P.h;
  if (H.valid && H.precision == q.precision && H.G == P.G && H.cutoff_rs == q.cutoff_rs &&
      H.soft_rs == soft && H.radius == radius)
    return;
  H.valid = false;
  H.precision = q.precision;
  H.G = P.G;
  H.cutoff_rs = q.cutoff_rs;
  H.soft_rs = soft;
  H.radius = radius;
  H.nrows = P.nrows;
  // a row's four values in a byte each: at most 32 cells of reach (r_c below
  // half a box of at most 64 cells) on either side of the group
  p3m::stencil_rows(P.G, radius, g_rows, P.nrows);
  for (int r = 0; r < P.nrows; ++r) {
    uint32_t w = 0;
    for (int c = 0; c < 4; ++c) w |= (uint32_t)(uint8_t)(int8_t)g_rows[4 * r + c] << (8 * c);
    H.words[r] = w;
  }
  if (q.precision == P3M_FP32) {
    float tab[4 * (p3m::kSplitBins + 1)];
    H.map = p3m::split_table(q.cutoff_rs, soft, p3m::kSplitBins, tab);
    H.ntab = sizeof(tab) / 4;
    std::memcpy(H.words + H.nrows, tab, sizeof(tab));
  } else {
    double tab[p3m::kSplitCoef64 * (p3m::kSplitBins + 1)];
    H.map = p3m::split_table64(q.cutoff_rs, soft, tab);
    H.ntab = sizeof(tab) / 4;
    std::memcpy(H.words + H.nrows, tab, sizeof(tab));
  }
  H.valid = true;
}

// Words [at, at + count) of the rows and the table, carried in the kernel's
// arguments (a captured call replays with them, and no copy is queued).
constexpr int kSetupWords = 960;
struct SetupArgs {
  int4* rows;
  uint32_t* tab;
  int nrows, at, count;
  int32_t* clear;             // cell counts to clear (the first launch), or null
  int nclear;
  uint32_t words[kSetupWords];
};
static_assert(sizeof(SetupArgs) <= 4096, "kernel arguments");

__global__ void __launch_bounds__(256) k_setup(SetupArgs A) {
  const int stride = gridDim.x * blockDim.x, first = blockIdx.x * blockDim.x + threadIdx.x;
  for (int i = first; i < A.count; i += stride) {
    const uint32_t w = A.words[i];
    const int k = A.at + i;
    if (k < A.nrows)
      A.rows[k] = make_int4((int8_t)w, (int8_t)(w >> 8), (int8_t)(w >> 16), (int8_t)(w >> 24));
    else
      A.tab[k - A.nrows] = w;
  }
  if (A.clear)
    for (int i = first; i < A.nclear; i += stride) A.clear[i] = 0;
}

// The tables of g_tables into the plan's workspace, and the cell counts
// cleared (the array keeps the last call's contents).
hipError_t launch_setup(p3m_plan* P) {
  const HostTables& H = g_tables;
  const int total = H.nrows + H.ntab;
  for (int at = 0; at < total; at += kSetupWords) {
    SetupArgs A;
    A.rows = P->ws.rows;
    A.tab = H.precision == P3M_FP32 ? (uint32_t*)P->ws.split_tab : (uint32_t*)P->ws.split_tab64;
    A.nrows = H.nrows;
    A.at = at;
    A.count = total - at < kSetupWords ? total - at : kSetupWords;
    A.clear = at == 0 ? P->ws.count : nullptr;
    A.nclear = (int)P->ncell;
    std::memcpy(A.words, H.words + at, 4 * (size_t)A.count);
    const unsigned blocks = (unsigned)(at == 0 && P->ncell > 4096 ? P->ncell / 1024 : 4);
    k_setup<<<blocks, 256, 0, P->stream>>>(A);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  P->count_dirty = 0;
  return hipSuccess;
}

// Device address of this device's scratch array (looked up once per device,
// with that device current).
hipError_t scratch_address(int dev, unsigned char** out) {
  if (!g_scratch[dev]) {
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[dev] = ptr;
  }
  *out = (unsigned char*)g_scratch[dev];
  return hipSuccess;
}

// Carves the plan's workspace from the scratch array at base; returns the
// bytes used (the caller checks them against kScratchBytes first with
// base == nullptr).
size_t carve(p3m_plan* P, unsigned char* base, int64_t n) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    unsigned char* p = base ? base + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return p;
  };
  const size_t real = P->prm.precision == P3M_FP32 ? sizeof(float) : sizeof(double);
  const int64_t nn = n > 0 ? n : 1;
  p3m::Workspace& W = P->ws;
  W.rank = (int32_t*)take(sizeof(int32_t) * nn);
  W.perm = (int32_t*)take(sizeof(int32_t) * nn);
  W.skey = (int32_t*)take(sizeof(int32_t) * nn);
  W.count = (int32_t*)take(sizeof(int32_t) * (P->ncell + 1));
  W.start = (int32_t*)take(sizeof(int32_t) * (P->ncell + 1));
  W.scan_tmp = (int32_t*)take(sizeof(int32_t) * p3m::scan_tiles(P->ncell));
  W.lstart = (int32_t*)take(sizeof(int32_t) * P->ncell);
  W.items = (int2*)take(sizeof(int2) * P->max_items);
  W.rows = (int4*)take(sizeof(int4) * P->nrows);
  W.rec = take(4 * real * nn);
  W.split_tab = (float*)take(sizeof(float) * 4 * (p3m::kSplitBins + 1));
  W.split_tab64 = (double*)take(sizeof(double) * p3m::kSplitCoef64 * (p3m::kSplitBins + 1));
  return off;
}

int status_of(hipError_t e) {
  if (e == hipSuccess) return P3M_OK;
  if (e == hipErrorOutOfMemory) return P3M_ENOMEM;
  return P3M_EHIP;
}

}  // namespace

extern "C" int pp_force_noalloc(const p3m_params* params, int64_t n, const double* pos,
                                const double* mass, double mass_scalar, void* force,
                                int32_t force_fp32, void* hip_stream) {
  if (!params || n < 0) return P3M_EINVAL;
  if (n > P3M_NOALLOC_MAX_N || params->grid_n > P3M_NOALLOC_MAX_GRID) return P3M_ESIZE;
  p3m_plan P;
  int st = p3m::plan_geometry(*params, n, &P);
  if (st != P3M_OK) return st;
  if (n == 0) return P3M_OK;
  if (!pos || !force) return P3M_EINVAL;
  if (!mass && !std::isfinite(mass_scalar)) return P3M_EINVAL;
  const size_t fbytes = (size_t)(3 * n) * (force_fp32 ? sizeof(float) : sizeof(double));
  const auto lo = [](const void* p) { return (uintptr_t)p; };
  if ((lo(force) < lo(pos) + 3 * n * sizeof(double) && lo(pos) < lo(force) + fbytes) ||
      (mass && lo(force) < lo(mass) + n * sizeof(double) && lo(mass) < lo(force) + fbytes))
    return P3M_EINVAL;
  if (P.nrows > kMaxRows || carve(&P, nullptr, n) > kScratchBytes) return P3M_ESIZE;
  P.stream = (hipStream_t)hip_stream;
  P.timing_slot = -1;

  std::lock_guard<std::mutex> lock(g_mutex);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return status_of(e);
  if (dev < 0 || dev >= kMaxDevices) return P3M_EINVAL;
  unsigned char* base = nullptr;
  if ((e = scratch_address(dev, &base)) != hipSuccess) return status_of(e);
  P.device = dev;
  carve(&P, base, n);
  make_tables(P);
  p3m::plan_set_split(&P, g_tables.map);
  if ((e = launch_setup(&P)) != hipSuccess) return status_of(e);
  if ((e = p3m::launch_bin(&P, n, pos, mass, mass_scalar, p3m::Items::kCut)) != hipSuccess)
    return status_of(e);
  e = params->precision == P3M_FP32
          ? p3m::launch_pairs<float>(&P, n, false, force, force_fp32 ? 1 : 0, mass == nullptr)
          : p3m::launch_pairs<double>(&P, n, false, force, force_fp32 ? 1 : 0, mass == nullptr);
  return status_of(e);
}
