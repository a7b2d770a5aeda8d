// Dense reconstruction C x_1 U_1 ... x_p U_p (eq. (reconstructed), Sec. 2.2) from
// factors the caller holds on the device, for callers that cannot allocate device
// memory: the intermediates of the n-mode product chain live in a fixed array of this
// library (`scratch`), so the call allocates nothing.
//
// In host code `scratch` names a host-side stand-in, not a device address: its device
// address is looked up once per device with hipGetSymbolAddress (with that device
// current) and only that pointer is handed to kernels. Each GPU holds its own copy of
// the array until the process ends; calls that overlap on one GPU race for it.
#include "tdb_common.h"
#include "tdb_kernels.h"
#include "noalloc.h"
#include "ttm.h"

#include <mutex>

namespace tdb {

static __device__ __align__(256) double scratch[NOALLOC_SCRATCH_DOUBLES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// The device address of `scratch` on the current device, looked up on the first call
// made with that device current.
static hipError_t scratch_on_current_device(double** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<double*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

NoallocPlan noalloc_plan(int p, const long long* dims, const int* ranks) {
  NoallocPlan pl{};
  pl.p = p;
  // contract the modes in order of increasing N_n / r_n (ties by mode), so that the
  // intermediates stay small; the last product writes the output
  for (int k = 0; k < p; ++k) pl.order[k] = k;
  for (int i = 1; i < p; ++i)
    for (int j = i; j > 0; --j) {
      const int x = pl.order[j - 1], y = pl.order[j];
      const double rx = (double)dims[x] / ranks[x], ry = (double)dims[y] / ranks[y];
      if (rx > ry || (rx == ry && x > y)) { pl.order[j - 1] = y; pl.order[j] = x; } else break;
    }
  long long cd[TDB_P];
  for (int k = 0; k < p; ++k) cd[k] = ranks[k];
  pl.max_inter = 0;
  for (int q = 0; q + 1 < p; ++q) {
    cd[pl.order[q]] = dims[pl.order[q]];
    long long sz = 1;
    for (int k = 0; k < p; ++k) sz *= cd[k];
    if (sz > pl.max_inter) pl.max_inter = sz;
  }
  return pl;
}

hipError_t noalloc_reconstruct(const NoallocPlan& pl, const long long* dims, const int* ranks, const double* C,
                               const double* const* U, int out_f32, void* out, hipStream_t s) {
  if (pl.p == 3) {
    // third-order states whose factors fit the LDS of a block: one launch, no scratch
    Rec3Args a{};
    for (int n = 0; n < 3; ++n) {
      a.N[n] = dims[n];
      a.r[n] = a.ldU[n] = ranks[n];
      a.U[n] = U[n];
    }
    a.C = C;
    a.out = out;
    if (rec3_ok<double>(a)) return out_f32 ? launch_rec3<double, float>(a, s) : launch_rec3<double, double>(a, s);
  }
  double* base = nullptr;
  hipError_t e = scratch_on_current_device(&base);
  if (e != hipSuccess) return e;
  double* half[2] = {base, base + NOALLOC_SCRATCH_DOUBLES / 2};
  const int p = pl.p;
  long long cd[TDB_P];
  for (int k = 0; k < p; ++k) cd[k] = ranks[k];
  const double* in = C;
  for (int q = 0; q < p; ++q) {
    const int k = pl.order[q];
    long long A = 1, B = 1;
    for (int j = 0; j < k; ++j) A *= cd[j];
    for (int j = k + 1; j < p; ++j) B *= cd[j];
    TtmGroup g{};
    g.n = 1;
    TtmJob& j = g.j[0];
    j.X = in;
    j.M = U[k];
    j.ms_i = 1;
    j.ms_o = ranks[k];
    j.A = A;
    j.Bsz = B;
    j.Nin = ranks[k];
    j.Nout = (int)dims[k];
    if (q + 1 < p) {
      j.Y = half[q & 1];
      in = half[q & 1];
      e = launch_ttm_group<double, double, double>(g, s);
    } else {
      j.Y = out;
      e = out_f32 ? launch_ttm_group<double, double, float>(g, s) : launch_ttm_group<double, double, double>(g, s);
    }
    if (e != hipSuccess) return e;
    cd[k] = dims[k];
  }
  return hipSuccess;
}

}  // namespace tdb
