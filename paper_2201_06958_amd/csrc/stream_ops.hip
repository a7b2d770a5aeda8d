// Elementwise passes over snapshots: the check for non-finite values and the
// second-order stage derivatives; the sum of the error pass's partials; and the copy of
// core and bases to the host.
#include "tdb_common.h"
#include "tdb_kernels.h"

namespace tdb {

__global__ void __launch_bounds__(256) k_err_final(const double* partials, int nb, CtrlState* ctrl) {
  __shared__ double red[16];
  double se = 0.0, sv = 0.0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) {
    se += partials[2 * i];
    sv += partials[2 * i + 1];
  }
  se = block_sum(se, red);
  sv = block_sum(sv, red);
  if (threadIdx.x == 0) {
    ctrl->eps2 = se;
    ctrl->nu2 = sv;
  }
}

hipError_t launch_err_final(const double* partials, int nblocks, CtrlState* ctrl, hipStream_t s) {
  hipLaunchKernelGGL(k_err_final, dim3(1), dim3(256), 0, s, partials, nblocks, ctrl);
  return hipGetLastError();
}

__global__ void k_flag_clear(int* flag) { *flag = 0; }

template <typename T>
__global__ void __launch_bounds__(256) k_nonfinite(const T* __restrict__ x, long long n, int* flag) {
  int bad = 0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    bad |= isfinite(x[i]) ? 0 : 1;
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

template <typename T>
hipError_t launch_nonfinite_check(const T* x, long long n, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_flag_clear, dim3(1), dim3(1), 0, s, flag);
  long long blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL((k_nonfinite<T>), dim3((unsigned)blocks), dim3(256), 0, s, x, n, flag);
  return hipGetLastError();
}
template hipError_t launch_nonfinite_check<float>(const float*, long long, int*, hipStream_t);
template hipError_t launch_nonfinite_check<double>(const double*, long long, int*, hipStream_t);

// The two stage derivatives of the second-order difference (Sec. 2.3): D1 at t_k by
// the central difference and D2 at t_{k+1} by the one-sided second-order difference,
// from the snapshots at t_{k-1} (Vm), t_k (V0) and t_{k+1} (V1). Formed in FP64 and
// stored in the data type; c = 1 / (2 dt). A grid-stride loop, one element per
// thread per pass (the loads of the three snapshots are coalesced).
template <typename T>
__global__ void __launch_bounds__(256) k_fd2(const T* __restrict__ Vm, const T* __restrict__ V0,
                                             const T* __restrict__ V1, T* __restrict__ D1, T* __restrict__ D2,
                                             long long n, double c) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const double a = (double)Vm[i], b = (double)V0[i], x = (double)V1[i];
    D1[i] = (T)((x - a) * c);
    D2[i] = (T)((3.0 * x - 4.0 * b + a) * c);
  }
}

template <typename T>
hipError_t launch_fd2(const T* Vm, const T* V0, const T* V1, T* D1, T* D2, long long n, double dt, hipStream_t s) {
  long long blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL((k_fd2<T>), dim3((unsigned)blocks), dim3(256), 0, s, Vm, V0, V1, D1, D2, n, 0.5 / dt);
  return hipGetLastError();
}
template hipError_t launch_fd2<float>(const float*, const float*, const float*, float*, float*, long long, double,
                                      hipStream_t);
template hipError_t launch_fd2<double>(const double*, const double*, const double*, double*, double*, long long,
                                       double, hipStream_t);

// Bound by the host link at large states, by the launch at small ones.
__global__ void __launch_bounds__(256) k_pack(PackArgs a, double* __restrict__ out, long long t0, long long cnt) {
  for (long long t = (long long)blockIdx.x * 256 + threadIdx.x; t < cnt; t += (long long)gridDim.x * 256) {
    long long q = t0 + t - a.csz;
    if (q < 0) {
      out[t] = a.C[t0 + t];
      continue;
    }
    int n = 0;
    while (n + 1 < a.p && q >= a.N[n] * a.r[n]) {
      q -= a.N[n] * a.r[n];
      ++n;
    }
    const long long i = q / a.r[n];
    out[t] = a.U[n][i * a.ldU[n] + (q - i * a.r[n])];
  }
}

hipError_t launch_pack(const PackArgs& a, double* out, long long t0, long long cnt, hipStream_t s) {
  if (cnt <= 0) return hipSuccess;
  long long blocks = (cnt + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)blocks), dim3(256), 0, s, a, out, t0, cnt);
  return hipGetLastError();
}

}  // namespace tdb
