// Small FP64 work of a step on the per-mode path (orders 2 to 4): the core Grams and
// their inverses, the basis right-hand side and its Heun update, the W-orthonormal QR
// folded into the core, and the controller.
//
// The basis equation (basecont) is used in the form
//   U_dot_n = (K_n - U_n T_n) G_n^-1,  K_n = F_(n) C_(n)^T,  T_n = (W_n U_n)^T K_n,
// with G_n = C_(n) C_(n)^T: F_(n) P_n = K_n G_n^-1, so the pseudo-inverse P_n (as large as
// the core) is never formed, and K_n and T_n are sums that split over workgroups. Every
// split sum is added in a fixed order.
//
// All of these are bound by latency: at ranks (33, 13, 33, 3) one workgroup per mode (the
// earlier form) took 988 us for the preparation of a stage and 1 650 us for the QR.
#include "tdb_common.h"
#include "plain.h"
#include "lds_limit.h"
#include "device_util.h"
#include <math.h>

namespace tdb {

typedef wd4 pd4;

// ---------------------------------------------------------------- helpers
// Columns of the mode-n unfolding of a core: inner = prod_{k > n} r_k.
// (A core holds at most 64^4 entries and F_n at most 512 x 64^3, so 32 bits index both.)
__device__ __forceinline__ void unf_sizes(const PlainArgs& a, int n, unsigned& inner, unsigned& R) {
  inner = 1;
  R = 1;
  for (int k = 0; k < a.p; ++k) {
    if (k != n) R *= a.r[k];
    if (k > n) inner *= a.r[k];
  }
}

constexpr int BP = 16;            // block size of the factorisation
constexpr int PLD = TDB_RCAP + 1; // row stride of the LDS matrices

// Lower Cholesky factor of the symmetric n x n matrix A (LDS, row stride PLD), its inverse
// Li and, with Gi, Gi = Li^T Li (row stride n), by four waves in 16 x 16 blocks: the
// diagonal block by one wave in registers, every other block as a matrix product by one
// wave each. Rows and columns from n to the next multiple of 16 are set to the identity.
// Fails like the one-wave form (a pivot below TDB_PIVOT_FLOOR times the largest diagonal
// entry). Bound by the chain of diagonal blocks; at n = 33 the first form, with the
// products as loops over LDS entries, took 51 us in the kernel that holds it.
__device__ bool block_chol_inv(double* A, int n, double* Li, double* Gi) {
  __shared__ double dmax_s;
  __shared__ int bad_s;
  const int tid = threadIdx.x, nt = blockDim.x, wv = tid >> 6, lane = tid & 63;
  const int nb = (n + BP - 1) / BP, m = nb * BP;
  for (int i = tid >> 4; i < m; i += nt >> 4)
    for (int j = tid & 15; j < m; j += 16) {
      if (i >= n || j >= n) A[i * PLD + j] = i == j ? 1.0 : 0.0;
      Li[i * PLD + j] = 0.0;
    }
  if (tid < 64) {
    const double d = wave_max_d(tid < n ? A[tid * PLD + tid] : 0.0);
    if (tid == 0) { dmax_s = d; bad_s = 0; }
  }
  __syncthreads();
  const double dmax = dmax_s;
  for (int kb = 0; kb < nb; ++kb) {
    const int k0 = kb * BP;
    if (wv == 0 && !wave_chol16(A, Li, PLD, k0, n, dmax) && lane == 0) bad_s = 1;
    __syncthreads();
    if (bad_s) return false;
    // L_ik = A_ik L_kk^-T
    for (int ib = kb + 1 + wv; ib < nb; ib += 4) {
      double* ai = A + ib * BP * PLD + k0;
      const pd4 r = mm16<BP>([&](int i, int k) { return ai[i * PLD + k]; },
                             [&](int k, int j) { return Li[(k0 + j) * PLD + k0 + k]; }, (pd4){0, 0, 0, 0});
      each16(r, [&](int i, int j, double v) { ai[i * PLD + j] = v; });
    }
    __syncthreads();
    // A_ij -= L_ik L_jk^T
    const int left = nb - kb - 1;
    for (int q = wv; q < left * (left + 1) / 2; q += 4) {
      int bi = 0;
      while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
      const int i0 = (kb + 1 + bi) * BP, j0 = (kb + 1 + q - bi * (bi + 1) / 2) * BP;
      pd4 c;
#pragma unroll
      for (int i = 0; i < 4; ++i) c[i] = A[(i0 + (lane >> 4) + 4 * i) * PLD + j0 + (lane & 15)];
      c = mm16<BP>([&](int i, int k) { return -A[(i0 + i) * PLD + k0 + k]; },
                   [&](int k, int j) { return A[(j0 + j) * PLD + k0 + k]; }, c);
      each16(c, [&](int i, int j, double v) { A[(i0 + i) * PLD + j0 + j] = v; });
    }
    __syncthreads();
  }
  // L^-1: X_ij = -Linv_ii sum_{j <= k < i} L_ik X_kj; the blocks of one distance i - j are
  // independent, one wave each
  for (int d = 1; d < nb; ++d) {
    if (wv < nb - d) {
      const int j0 = wv * BP, ib = wv + d, i0 = ib * BP;
      pd4 r = {0, 0, 0, 0};
      for (int kb = wv; kb < ib; ++kb)
        r = mm16<BP>([&](int i, int k) { return A[(i0 + i) * PLD + kb * BP + k]; },
                     [&](int k, int j) { return Li[(kb * BP + k) * PLD + j0 + j]; }, r);
      each16(r, [&](int i, int j, double v) { Li[(i0 + i) * PLD + j0 + j] = v; });
      wave_fence();
      r = mm16<BP>([&](int i, int k) { return -Li[(i0 + i) * PLD + i0 + k]; },
                   [&](int k, int j) { return Li[(i0 + k) * PLD + j0 + j]; }, (pd4){0, 0, 0, 0});
      wave_fence();
      each16(r, [&](int i, int j, double v) { Li[(i0 + i) * PLD + j0 + j] = v; });
    }
    __syncthreads();
  }
  if (Gi) {
    for (int q = wv; q < nb * nb; q += 4) {
      const int i0 = q / nb * BP, j0 = q % nb * BP;
      pd4 r = {0, 0, 0, 0};
      for (int k0 = max(i0, j0); k0 < m; k0 += BP)
        r = mm16<BP>([&](int i, int k) { return Li[(k0 + k) * PLD + i0 + i]; },
                     [&](int k, int j) { return Li[(k0 + k) * PLD + j0 + j]; }, r);
      each16(r, [&](int i, int j, double v) {
        if (i0 + i < n && j0 + j < n) Gi[(i0 + i) * n + j0 + j] = v;
      });
    }
    __syncthreads();
  }
  return true;
}

// Sum of `cnt` partials of `len` values each, entry t, sixteen loads in flight at a time.
__device__ __forceinline__ double sum_parts(const double* __restrict__ p, long long t, int cnt, long long len) {
  double s = 0.0;
  for (int c = 0; c < cnt; c += 16) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(long long)min(c + u, cnt - 1) * len + t];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += c + u < cnt ? v[u] : 0.0;
  }
  return s;
}

// ---------------------------------------------------------------- core Grams
// Block (n, chunk): partial Gram of columns [chunk * glen, +glen) of C_(n), staged 64
// columns at a time, on the FP64 matrix cores (the blocks on and below the diagonal, one
// per wave in turn).
__global__ void __launch_bounds__(256) k_core_gram(PlainArgs a) {
  __shared__ double X[64 * PLD];
  int n = 0, ch = blockIdx.x;
  while (n + 1 < a.p && ch >= a.gch[n]) ch -= a.gch[n++];
  const int rn = a.r[n];
  unsigned inner, R;
  unf_sizes(a, n, inner, R);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, lm = lane & 15, lk = lane >> 4;
  const int nb = (rn + 15) >> 4, nblk = nb * (nb + 1) / 2;
  pd4 acc[3] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  const unsigned c0 = (unsigned)(ch * a.glen[n]), c1 = min(R, c0 + (unsigned)a.glen[n]);
  const unsigned k = threadIdx.x & 63, ib = threadIdx.x >> 6;
  for (unsigned cb = c0; cb < c1; cb += 64) {
    // a thread keeps its column, so the division is done once a chunk
    const unsigned c = min(cb + k, c1 - 1), o = c / inner, in = c - o * inner;
    const bool cv = cb + k < c1;
    const double* src = a.C + (o * rn) * inner + in;
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = src[min(ib + 4 * q, (unsigned)rn - 1) * inner];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const unsigned i = ib + 4 * q;
      if (i < 16u * nb) X[k * PLD + i] = (cv && i < (unsigned)rn) ? v[q] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int blk = wid + 4 * q;
      if (blk < nblk) {
        int bi = 0;
        while ((bi + 1) * (bi + 2) / 2 <= blk) ++bi;
        const int bj = blk - bi * (bi + 1) / 2;
#pragma unroll
        for (int kk = 0; kk < 64; kk += 4) {
          const double x = X[(kk + lk) * PLD + 16 * bi + lm], y = X[(kk + lk) * PLD + 16 * bj + lm];
          acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[q], 0, 0, 0);
        }
      }
    }
  }
  double* out = a.gpart[n] + (long long)ch * rn * rn;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int blk = wid + 4 * q;
    if (blk < nblk) {
      int bi = 0;
      while ((bi + 1) * (bi + 2) / 2 <= blk) ++bi;
      const int bj = blk - bi * (bi + 1) / 2;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * bi + lk + 4 * i, c = 16 * bj + lm;
        if (r < rn && c <= r) out[r * rn + c] = acc[q][i];
      }
    }
  }
}

// Block n: G_n from its partials, its inverse, and what the removal test needs of it.
// A failed test of a mode that evolves raises NUM_CORE, or NUM_NEXT when the core is
// the next step's.
__global__ void __launch_bounds__(256) k_core_fact(PlainArgs a, CtrlState* ctrl) {
  __shared__ double A[TDB_RCAP * PLD], Li[TDB_RCAP * PLD];
  __shared__ double red[16];
  const int n = blockIdx.x, rn = a.r[n];
  for (int t = threadIdx.x; t < rn * rn; t += 256) {
    const int i = t / rn, j = t - i * rn;
    if (j <= i) {
      const double s = sum_parts(a.gpart[n], t, a.gch[n], (long long)rn * rn);
      A[i * PLD + j] = s;
      A[j * PLD + i] = s;
    }
  }
  __syncthreads();
  const bool ok = block_chol_inv(A, rn, Li, a.Ginv[n]);
  double tr = 0.0, mx = 0.0;
  if (ok) {
    // (each thread reads the diagonal entries that some thread of this block wrote
    // before the last barrier)
    for (int i = threadIdx.x; i < rn; i += 256) {
      const double d = a.Ginv[n][i * rn + i];
      tr += d;
      mx = fmax(mx, d);
    }
  } else {
    for (int t = threadIdx.x; t < rn * rn; t += 256) a.Ginv[n][t] = 0.0;
    if (threadIdx.x == 0 && rn < a.N[n]) atomicOr(&ctrl->numeric, a.next ? NUM_NEXT : NUM_CORE);
  }
  tr = block_sum(tr, red);
  mx = block_max(mx, red);
  if (threadIdx.x == 0) {
    a.gstat[3 * n] = tr;
    a.gstat[3 * n + 1] = mx;
    a.gstat[3 * n + 2] = ok ? 1.0 : 0.0;
  }
}

// ---------------------------------------------------------------- fold with the core
// Block (n, 64 rows, chunk): partial K_n over columns [chunk * klen, +klen), FP64 products
// on the matrix cores (F_n is held in the compute type), 32 columns staged at a time with
// the next ones' loads in flight. PINV: the pseudo-inverse P_n (R x r_n, compute type) in
// the place of C_(n)^T, which gives H_n = F_(n) P_n itself.
template <typename T, bool PINV>
__global__ void __launch_bounds__(256) k_core_fold(PlainArgs a) {
  constexpr int KC = 32, LD = KC + 1;
  __shared__ double Fl[64 * LD], Cl[TDB_RCAP * LD];
  int n = 0, bx = blockIdx.x;
  for (;; ++n) {
    const int nb = a.r[n] < a.N[n] ? (int)((a.N[n] + 63) / 64) * a.kch[n] : 0;
    if (bx < nb) break;
    bx -= nb;
  }
  const int ch = bx % a.kch[n];
  const long long i0 = (long long)(bx / a.kch[n]) * 64, Nn = a.N[n];
  const int rn = a.r[n];
  unsigned inner, R;
  unf_sizes(a, n, inner, R);
  const T* F = static_cast<const T*>(a.F[n]);
  const unsigned c0 = (unsigned)(ch * a.klen[n]), c1 = min(R, c0 + (unsigned)a.klen[n]);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, lm = lane & 15, lk = lane >> 4;
  const int nb = (rn + 15) >> 4;
  pd4 acc[4] = {{0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}, {0, 0, 0, 0}};
  T fv[8];
  double cv[8];
  const unsigned k = threadIdx.x & 31, ib = threadIdx.x >> 5, ilast = (unsigned)(Nn - 1 - i0);
  // a thread keeps its column, so the division is done once for its 16 loads
  auto load = [&](unsigned cb) {
    const unsigned c = min(cb + k, c1 - 1), o = c / inner, in = c - o * inner;
    const T* fs = F + (o * (unsigned)Nn + (unsigned)i0) * inner + in;
    const double* cs = a.C + (o * rn) * inner + in;
    const T* ps = static_cast<const T*>(a.P[n]) + (size_t)c * rn;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      fv[q] = fs[min(ib + 8 * q, ilast) * inner];
      cv[q] = PINV ? (double)ps[min(ib + 8 * q, (unsigned)rn - 1)] : cs[min(ib + 8 * q, (unsigned)rn - 1) * inner];
    }
  };
  load(c0);
  for (unsigned cb = c0; cb < c1; cb += KC) {
    __syncthreads();
    const bool cok = cb + k < c1;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const unsigned i = ib + 8 * q;
      Fl[i * LD + k] = (cok && i <= ilast) ? (double)fv[q] : 0.0;
      Cl[i * LD + k] = (cok && i < (unsigned)rn) ? cv[q] : 0.0;
    }
    __syncthreads();
    if (cb + KC < c1) load(cb + KC);
#pragma unroll
    for (int kk = 0; kk < KC; kk += 4) {
      const double x = Fl[(16 * wid + lm) * LD + kk + lk];
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (b < nb) acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, Cl[(16 * b + lm) * LD + kk + lk], acc[b], 0, 0, 0);
    }
  }
  double* out = a.kpart[n] + (long long)ch * Nn * rn;
#pragma unroll
  for (int b = 0; b < 4; ++b)
    if (b < nb) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const long long i = i0 + 16 * wid + lk + 4 * q;
        const int c = 16 * b + lm;
        if (i < Nn && c < rn) out[i * rn + c] = acc[b][q];
      }
    }
}

// Mode and slab of a flat block index over the slabs of every mode; false past the end.
__device__ __forceinline__ bool slab_of(const PlainArgs& a, int& bx, int rows, int& n) {
  for (n = 0; n < a.p; ++n) {
    const int nb = (int)((a.N[n] + rows - 1) / rows);
    if (bx < nb) return true;
    bx -= nb;
  }
  return false;
}

// Block (n, slab): K_n of the slab's rows from its partials, and the slab's part of T_n.
__global__ void __launch_bounds__(256) k_basis_sum(PlainArgs a, CtrlState* ctrl) {
  __shared__ double Kl[PL_SLAB * PLD], Wl[PL_SLAB * PLD];
  // a singular core found while preparing this step belongs to its first stage
  if (a.stage == 1 && blockIdx.x == 0 && threadIdx.x == 0 && (ctrl->numeric & NUM_NEXT)) {
    atomicOr(&ctrl->numeric, NUM_CORE);
    atomicAnd(&ctrl->numeric, ~NUM_NEXT);
  }
  int bx = blockIdx.x, n;
  if (!slab_of(a, bx, PL_SLAB, n)) return;
  const int rn = a.r[n], nb = (rn + 15) >> 4;
  const long long Nn = a.N[n], i0 = (long long)bx * PL_SLAB;
  if (rn >= Nn) return;
  const int rows = (int)min((long long)PL_SLAB, Nn - i0);
  for (int i = threadIdx.x >> 4; i < PL_SLAB; i += 16)
    for (int j = threadIdx.x & 15; j < nb * 16; j += 16) {
      double k = 0.0, w = 0.0;
      if (i < rows && j < rn) {
        k = sum_parts(a.kpart[n], (i0 + i) * rn + j, a.kch[n], Nn * rn);
        a.K[n][(i0 + i) * rn + j] = k;
        w = a.w[n][i0 + i] * a.U[n][(i0 + i) * a.ldU[n] + j];
      }
      Kl[i * PLD + j] = k;
      Wl[i * PLD + j] = w;
    }
  __syncthreads();
  double* out = a.tpart[n] + (long long)bx * rn * rn;
  for (int q = threadIdx.x >> 6; q < nb * nb; q += 4) {
    const int r0 = q / nb * 16, c0 = q % nb * 16;
    const pd4 t = mm16<PL_SLAB>([&](int i, int k) { return Wl[k * PLD + r0 + i]; },
                                [&](int k, int j) { return Kl[k * PLD + c0 + j]; }, (pd4){0, 0, 0, 0});
    each16(t, [&](int i, int j, double v) {
      if (r0 + i < rn && c0 + j < rn) out[(r0 + i) * rn + c0 + j] = v;
    });
  }
}

// Block (n, slab): U_dot_n = (K_n - U_n T_n) G_n^-1 of the slab's rows and the Heun update
// (stage 1: k = U_dot, U* = U + dt k; stage 2: U <- U + dt/2 (k + U_dot)). The blocks
// after the slabs apply the same to the core. Stage 2 changes nothing when a stage found
// a singular core or non-finite data.
__global__ void __launch_bounds__(256) k_basis_rows(PlainArgs a, CtrlState* ctrl) {
  __shared__ double T[TDB_RCAP * PLD], Gi[TDB_RCAP * PLD];
  __shared__ double Ul[PL_SLAB * PLD], Vl[PL_SLAB * PLD];
  if (a.stage == 2 && ctrl->numeric) return;
  int bx = blockIdx.x, n;
  if (!slab_of(a, bx, PL_SLAB, n)) {
    const long long t = (long long)bx * 256 + threadIdx.x;
    if (t >= a.csz) return;
    const double cd = a.Cdot[t] * a.dscale;
    if (a.stage == 1) {
      // NaN or Inf anywhere in the data derivative reaches every entry of C_dot
      if (!isfinite(cd)) atomicOr(&ctrl->numeric, NUM_NONFINITE);
      a.kC[t] = cd;
      a.Cs[t] = a.C0[t] + a.dt * cd;
    } else {
      a.C0[t] = a.C0[t] + 0.5 * a.dt * (a.kC[t] + cd);
    }
    return;
  }
  const int rn = a.r[n], ld = a.ldU[n], nb = (rn + 15) >> 4;
  const long long Nn = a.N[n], i0 = (long long)bx * PL_SLAB;
  const int rows = (int)min((long long)PL_SLAB, Nn - i0);
  const bool full = rn >= Nn;
  auto update = [&](int i, int j, double ud) {
    const long long e = (i0 + i) * ld + j;
    if (a.stage == 1) {
      a.kU[n][e] = ud;
      a.Us[n][e] = a.U0[n][e] + a.dt * ud;
    } else {
      a.U0[n][e] += 0.5 * a.dt * (a.kU[n][e] + ud);
    }
  };
  if (full) {
    for (int t = threadIdx.x; t < rows * rn; t += 256) update(t / rn, t % rn, 0.0);
    return;
  }
  const int slabs = (int)((Nn + PL_SLAB - 1) / PL_SLAB);
  for (int i = threadIdx.x >> 4; i < nb * 16; i += 16)
    for (int j = threadIdx.x & 15; j < nb * 16; j += 16) {
      const bool in = i < rn && j < rn;
      T[i * PLD + j] = in ? sum_parts(a.tpart[n], i * rn + j, slabs, (long long)rn * rn) : 0.0;
      Gi[i * PLD + j] = in ? a.Ginv[n][i * rn + j] : 0.0;
    }
  for (int i = threadIdx.x >> 4; i < PL_SLAB; i += 16)
    for (int j = threadIdx.x & 15; j < nb * 16; j += 16) {
      const bool in = i < rows && j < rn;
      Ul[i * PLD + j] = in ? a.U[n][(i0 + i) * ld + j] : 0.0;
      Vl[i * PLD + j] = in ? a.K[n][(i0 + i) * rn + j] : 0.0;
    }
  __syncthreads();
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int q = wv; q < 2 * nb; q += 4) {
    const int r0 = q / nb * 16, c0 = q % nb * 16;
    pd4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = Vl[(r0 + (lane >> 4) + 4 * i) * PLD + c0 + (lane & 15)];
    for (int k0 = 0; k0 < nb * 16; k0 += 16)
      v = mm16<16>([&](int i, int k) { return -Ul[(r0 + i) * PLD + k0 + k]; },
                   [&](int k, int j) { return T[(k0 + k) * PLD + c0 + j]; }, v);
    each16(v, [&](int i, int j, double x) { Vl[(r0 + i) * PLD + c0 + j] = x; });
  }
  __syncthreads();
  for (int q = wv; q < 2 * nb; q += 4) {
    const int r0 = q / nb * 16, c0 = q % nb * 16;
    pd4 v = {0, 0, 0, 0};
    for (int k0 = 0; k0 < nb * 16; k0 += 16)
      v = mm16<16>([&](int i, int k) { return Vl[(r0 + i) * PLD + k0 + k]; },
                   [&](int k, int j) { return Gi[(k0 + k) * PLD + c0 + j]; }, v);
    each16(v, [&](int i, int j, double x) {
      if (r0 + i < rows && c0 + j < rn) update(r0 + i, c0 + j, x * a.dscale);
    });
  }
}

// H_n from its partials, and the Heun update of the core (as the reduction of a fused
// stream's tile partials does it), for the streams whose projections are formed by
// products.
__global__ void __launch_bounds__(256) k_chain_reduce(PlainArgs a, CtrlState* ctrl) {
  if (ctrl->hold || (a.stage == 2 && ctrl->numeric)) return;
  // a singular core found while preparing this step belongs to its first stage
  if (a.stage == 1 && blockIdx.x == 0 && threadIdx.x == 0 && (ctrl->numeric & NUM_NEXT)) {
    atomicOr(&ctrl->numeric, NUM_CORE);
    atomicAnd(&ctrl->numeric, ~NUM_NEXT);
  }
  long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  for (int n = 0; n < a.p; ++n) {
    const long long len = a.r[n] < a.N[n] ? a.N[n] * a.r[n] : 0;
    if (t < len) {
      a.H[n][t] = sum_parts(a.kpart[n], t, a.kch[n], len);
      return;
    }
    t -= len;
  }
  if (t >= a.csz) return;
  const double cd = a.Cdot[t] * a.dscale;
  if (a.stage == 1) {
    // every entry of the data derivative reaches every entry of C_dot, so NaN or Inf
    // anywhere in the snapshots shows here; the step is then not applied
    if (!isfinite(cd)) atomicOr(&ctrl->numeric, NUM_NONFINITE);
    a.kC[t] = cd;
    a.Cs[t] = a.C0[t] + a.dt * cd;
  } else {
    a.Cdot2[t] = cd;
    a.C0[t] += 0.5 * a.dt * (a.kC[t] + cd);
  }
}

// ---------------------------------------------------------------- QR and fold
// Block (n, slab): partial U_n^T W_n U_n of the slab's rows (lower triangle).
__global__ void __launch_bounds__(256) k_qr_gram(PlainArgs a, CtrlState* ctrl) {
  __shared__ double Ul[PL_QSLAB * PLD];
  if (ctrl->numeric & ~NUM_NEXT) return;
  int bx = blockIdx.x, n;
  if (!slab_of(a, bx, PL_QSLAB, n)) return;
  const int rn = a.r[n], nb = (rn + 15) >> 4;
  const long long Nn = a.N[n], i0 = (long long)bx * PL_QSLAB;
  const int rows = (int)min((long long)PL_QSLAB, Nn - i0);
  for (int i = threadIdx.x >> 4; i < PL_QSLAB; i += 16)
    for (int j = threadIdx.x & 15; j < nb * 16; j += 16)
      Ul[i * PLD + j] =
          (i < rows && j < rn) ? sqrt(a.w[n][i0 + i]) * a.U0[n][(i0 + i) * a.ldU[n] + j] : 0.0;
  __syncthreads();
  double* out = a.qpart[n] + (long long)bx * rn * rn;
  for (int q = threadIdx.x >> 6; q < nb * (nb + 1) / 2; q += 4) {
    int bi = 0;
    while ((bi + 1) * (bi + 2) / 2 <= q) ++bi;
    const int r0 = bi * 16, c0 = (q - bi * (bi + 1) / 2) * 16;
    const pd4 t = mm16<PL_QSLAB>([&](int i, int k) { return Ul[k * PLD + r0 + i]; },
                                 [&](int k, int j) { return Ul[k * PLD + c0 + j]; }, (pd4){0, 0, 0, 0});
    each16(t, [&](int i, int j, double v) {
      if (r0 + i < rn && c0 + j <= r0 + i) out[(r0 + i) * rn + c0 + j] = v;
    });
  }
}

// Block n: the factor L of U_n^T W_n U_n = L L^T (R_n = L^T) and its inverse; the identity
// when the step is not applied. After one round the bases are orthonormal to cond(U)^2
// roundings, so a second one matters only where the Gram is far from the identity;
// qneed then asks for it. The flags are read once a block, so that its waves take one branch,
// and without NUM_BASIS, which the other blocks of this launch may be raising.
__global__ void __launch_bounds__(256) k_qr_fact(PlainArgs a, CtrlState* ctrl) {
  __shared__ double A[TDB_RCAP * PLD], Li[TDB_RCAP * PLD];
  __shared__ double red[16];
  const int n = blockIdx.x, rn = a.r[n];
  const int slabs = (int)((a.N[n] + PL_QSLAB - 1) / PL_QSLAB);
  __shared__ int flags;
  if (threadIdx.x == 0)
    flags = __hip_atomic_load(&ctrl->numeric, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ~(NUM_NEXT | NUM_BASIS);
  __syncthreads();
  const bool skip = flags != 0;
  bool ok = false;
  double dev = 0.0;
  if (!skip) {
    for (int t = threadIdx.x; t < rn * rn; t += 256) {
      const int i = t / rn, j = t - i * rn;
      if (j <= i) {
        const double s = sum_parts(a.qpart[n], t, slabs, (long long)rn * rn);
        A[i * PLD + j] = s;
        A[j * PLD + i] = s;
        const double d = i == j ? s - 1.0 : s;
        dev += (i == j ? 1.0 : 2.0) * d * d;
      }
    }
    dev = block_sum(dev, red);
    ok = block_chol_inv(A, rn, Li, nullptr);
    if (!ok && threadIdx.x == 0) atomicOr(&ctrl->numeric, NUM_BASIS);
    if (!(dev <= 0.25) && threadIdx.x == 0) *a.qneed = 1;
  }
  for (int t = threadIdx.x; t < rn * rn; t += 256) {
    const int i = t / rn, j = t - i * rn;
    const double id = i == j ? 1.0 : 0.0;
    a.L[n][t] = ok ? (j <= i ? A[i * PLD + j] : 0.0) : id;
    a.Li[n][t] = ok ? (j <= i ? Li[i * PLD + j] : 0.0) : id;
  }
}

// Folds R = L^T into the core for one pair of modes (m, m + 1; m + 1 == p: one mode): a
// block takes some slices of the two modes in place. The blocks after those apply
// U_n <- U_n L_n^-T to the slabs of every basis (first launch only).
__global__ void __launch_bounds__(256) k_qr_fold2(PlainArgs a, int m, int spb, int cblocks, CtrlState* ctrl) {
  extern __shared__ __align__(16) unsigned char raw_f[];
  double* lds = reinterpret_cast<double*>(raw_f);
  if ((int)blockIdx.x >= cblocks) {
    int bx = (int)blockIdx.x - cblocks, n;
    if (!slab_of(a, bx, PL_SLAB, n)) return;
    const int rn = a.r[n];
    const long long Nn = a.N[n], i0 = (long long)bx * PL_SLAB;
    const int rows = (int)min((long long)PL_SLAB, Nn - i0);
    double *Ll = lds, *Ul = lds + rn * rn;
    for (int t = threadIdx.x; t < rn * rn; t += 256) Ll[t] = a.Li[n][t];
    for (int t = threadIdx.x; t < rows * rn; t += 256) Ul[t] = a.U0[n][(i0 + t / rn) * a.ldU[n] + t % rn];
    __syncthreads();
    for (int t = threadIdx.x; t < rows * rn; t += 256) {
      const int i = t / rn, j = t - i * rn;
      double s = 0.0;
      for (int k = 0; k <= j; ++k) s += Ll[j * rn + k] * Ul[i * rn + k];
      a.U0[n][(i0 + i) * a.ldU[n] + j] = s;
    }
    return;
  }
  const bool two = m + 1 < a.p;
  const int ra = a.r[m], rb = two ? a.r[m + 1] : 1;
  long long inner = 1, outer = 1;
  for (int k = 0; k < m; ++k) outer *= a.r[k];
  for (int k = m + (two ? 2 : 1); k < a.p; ++k) inner *= a.r[k];
  const long long slices = outer * inner;
  const long long s0 = (long long)blockIdx.x * spb;
  const int ns = (int)min((long long)spb, slices - s0);
  const int ssz = ra * rb, tot = ns * ssz;
  double *La = lds, *Lb = La + ra * ra, *X = Lb + rb * rb, *Y = X + spb * ssz;
  for (int t = threadIdx.x; t < ra * ra; t += 256) La[t] = a.L[m][t];
  for (int t = threadIdx.x; t < rb * rb; t += 256) Lb[t] = two ? a.L[m + 1][t] : 1.0;
  // consecutive threads along the slices, which are contiguous where inner > 1
  auto at = [&](int t, int& sl, int& x) {
    sl = t % ns;
    x = t / ns;
    const long long s = s0 + sl, o = s / inner, in = s - o * inner;
    return (o * ssz + x) * inner + in;
  };
  for (int t = threadIdx.x; t < tot; t += 256) {
    int sl, x;
    const long long e = at(t, sl, x);
    X[sl * ssz + x] = a.C0[e];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < tot; t += 256) {
    const int sl = t / ssz, x = t - sl * ssz, i = x / rb, j = x - i * rb;
    double s = 0.0;
    for (int k = i; k < ra; ++k) s += La[k * ra + i] * X[sl * ssz + k * rb + j];
    Y[t] = s;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < tot; t += 256) {
    int sl, x;
    const long long e = at(t, sl, x);
    const int i = x / rb, j = x - i * rb;
    double s = 0.0;
    for (int k = j; k < rb; ++k) s += Lb[k * rb + j] * Y[sl * ssz + i * rb + k];
    a.C0[e] = s;
  }
}

// ---------------------------------------------------------------- controller
// One block: the error and norm sums, the decision (Sec. 2.5). The removal test asks
// whether some mode's smallest core singular value fits the budget, sigma^2 <= B - eps^2.
// 1 / trace(G^-1) <= sigma^2 <= 1 / max diag(G^-1) settles it except in between, where the
// Cholesky factorisation of G - (B - eps^2) I decides.
__global__ void __launch_bounds__(256) k_plain_ctrl(PlainArgs a, const double* part, int nb, CtrlState* c) {
  __shared__ double A[TDB_RCAP * PLD], Li[TDB_RCAP * PLD];
  __shared__ double red[16];
  __shared__ int test;
  double se = 0.0, sv = 0.0;
  for (int i = threadIdx.x; i < nb; i += 256) {
    se += part[2 * i];
    sv += part[2 * i + 1];
  }
  se = block_sum(se, red);
  sv = block_sum(sv, red);
  if (threadIdx.x == 0) {
    c->eps2 = se;
    c->nu2 = sv;
    test = controller_pre(c) ? 1 : 0;
  }
  __syncthreads();
  if (!test) return;
  const double B = c->gamma_th > 0.0 ? (1.0 - c->gamma_th / 100.0) * c->nu2 : 0.25 * c->eps_th * c->eps_th;
  const double room = B - c->eps * c->eps;
  bool fits = false;
  for (int n = 0; n < a.p && !fits; ++n) {
    const int rn = a.r[n];
    const bool have = a.gstat[3 * n + 2] != 0.0;
    if (!(room >= 0.0)) continue;
    if (have && a.gstat[3 * n] * room < 1.0) continue;
    if (have && a.gstat[3 * n + 1] * room >= 1.0) { fits = true; continue; }
    __syncthreads();
    for (int t = threadIdx.x; t < rn * rn; t += 256) {
      const int i = t / rn, j = t - i * rn;
      if (j <= i) {
        const double s = sum_parts(a.gpart[n], t, a.gch[n], (long long)rn * rn) - (i == j ? room : 0.0);
        A[i * PLD + j] = s;
        A[j * PLD + i] = s;
      }
    }
    __syncthreads();
    fits = !block_chol_inv(A, rn, Li, nullptr);
  }
  if (fits && threadIdx.x == 0) c->decision = DEC_REMOVE;
}

// ---------------------------------------------------------------- launchers
static long long cols_of(const PlainArgs& a, int n) {
  long long R = 1;
  for (int k = 0; k < a.p; ++k)
    if (k != n) R *= a.r[k];
  return R;
}

// Columns per chunk: 128 for the Grams; for the folds 64 (two rounds of loads a block) up to
// 512 columns and 128 above (with 64 there the channel's 1 287 columns a mode made twice
// the partials to write and add: 2.73 against 2.55 ms for four steps); more only where
// that would make more chunks than the partial buffers hold.
void plain_chunks(PlainArgs& a) {
  for (int n = 0; n < a.p; ++n) {
    const long long R = cols_of(a, n);
    const long long g = ((R + PL_GCH - 1) / PL_GCH + 63) & ~63LL, k = ((R + PL_KCH - 1) / PL_KCH + 31) & ~31LL;
    a.glen[n] = (int)(g > 128 ? g : 128);
    const int kmin = R <= 512 ? 64 : 128;
    a.klen[n] = (int)(k > kmin ? k : kmin);
    a.gch[n] = (int)((R + a.glen[n] - 1) / a.glen[n]);
    a.kch[n] = (int)((R + a.klen[n] - 1) / a.klen[n]);
  }
}

hipError_t launch_plain_prep(const PlainArgs& a, CtrlState* ctrl, hipStream_t s) {
  int nb = 0;
  for (int n = 0; n < a.p; ++n) nb += a.gch[n];
  hipLaunchKernelGGL(k_core_gram, dim3(nb), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_core_fact, dim3(a.p), dim3(256), 0, s, a, ctrl);
  return hipGetLastError();
}

static int slabs_of(const PlainArgs& a, int rows) {
  int nb = 0;
  for (int n = 0; n < a.p; ++n) nb += (int)((a.N[n] + rows - 1) / rows);
  return nb;
}

template <typename T>
hipError_t launch_plain_rhs(const PlainArgs& a, CtrlState* ctrl, hipStream_t s) {
  int nb = 0;
  for (int n = 0; n < a.p; ++n)
    if (a.r[n] < a.N[n]) nb += (int)((a.N[n] + 63) / 64) * a.kch[n];
  if (nb) hipLaunchKernelGGL((k_core_fold<T, false>), dim3(nb), dim3(256), 0, s, a);
  const int sl = slabs_of(a, PL_SLAB);
  hipLaunchKernelGGL(k_basis_sum, dim3(sl), dim3(256), 0, s, a, ctrl);
  hipLaunchKernelGGL(k_basis_rows, dim3((unsigned)(sl + (a.csz + 255) / 256)), dim3(256), 0, s, a, ctrl);
  return hipGetLastError();
}
template hipError_t launch_plain_rhs<float>(const PlainArgs&, CtrlState*, hipStream_t);
template hipError_t launch_plain_rhs<double>(const PlainArgs&, CtrlState*, hipStream_t);

template <typename T>
hipError_t launch_chain_finish(const PlainArgs& a, CtrlState* ctrl, hipStream_t s) {
  int nb = 0;
  long long len = a.csz;
  for (int n = 0; n < a.p; ++n)
    if (a.r[n] < a.N[n]) {
      nb += (int)((a.N[n] + 63) / 64) * a.kch[n];
      len += a.N[n] * a.r[n];
    }
  if (nb) hipLaunchKernelGGL((k_core_fold<T, true>), dim3(nb), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_chain_reduce, dim3((unsigned)((len + 255) / 256)), dim3(256), 0, s, a, ctrl);
  return hipGetLastError();
}
template hipError_t launch_chain_finish<float>(const PlainArgs&, CtrlState*, hipStream_t);
template hipError_t launch_chain_finish<double>(const PlainArgs&, CtrlState*, hipStream_t);

hipError_t launch_plain_qr(const PlainArgs& a, CtrlState* ctrl, hipStream_t s) {
  hipLaunchKernelGGL(k_qr_gram, dim3(slabs_of(a, PL_QSLAB)), dim3(256), 0, s, a, ctrl);
  hipLaunchKernelGGL(k_qr_fact, dim3(a.p), dim3(256), 0, s, a, ctrl);
  for (int m = 0; m < a.p; m += 2) {
    const bool two = m + 1 < a.p;
    const int ra = a.r[m], rb = two ? a.r[m + 1] : 1;
    const long long slices = a.csz / ((long long)ra * rb);
    // enough slices a block to pay for staging the factors, at most 16 KB of them
    int spb = 1024 / (ra * rb);
    if (spb < 1) spb = 1;
    if (spb > slices) spb = (int)slices;
    const int cb = (int)((slices + spb - 1) / spb);
    size_t lds = ((size_t)ra * ra + (size_t)rb * rb + 2 * (size_t)spb * ra * rb) * 8;
    int extra = 0;
    if (m == 0) {
      extra = slabs_of(a, PL_SLAB);
      for (int n = 0; n < a.p; ++n) {
        const size_t l = ((size_t)a.r[n] * a.r[n] + (size_t)PL_SLAB * a.r[n]) * 8;
        if (l > lds) lds = l;
      }
    }
    // at most 128 KB (two factors and two slices of 64 x 64)
    hipError_t e = lds_limit(reinterpret_cast<const void*>(k_qr_fold2), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_qr_fold2, dim3(cb + extra), dim3(256), lds, s, a, m, spb, cb, ctrl);
  }
  return hipGetLastError();
}

hipError_t launch_plain_ctrl(const PlainArgs& a, const double* err_part, int nblocks, CtrlState* ctrl, hipStream_t s) {
  hipLaunchKernelGGL(k_plain_ctrl, dim3(1), dim3(256), 0, s, a, err_part, nblocks, ctrl);
  return hipGetLastError();
}

}  // namespace tdb
