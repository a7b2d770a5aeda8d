// Device helpers shared by the plain and fused kernels (internal).
#pragma once
#include "tdb_common.h"

namespace tdb {

// ---------------------------------------------------------------- Jacobi eigensolver
// Cyclic Jacobi on a symmetric rn x rn LDS matrix A with round-robin pairing
// (rn/2 disjoint rotations per round). On exit the diagonal of A holds the
// eigenvalues; if V != nullptr it accumulates the eigenvectors (columns).
static __device__ void jacobi_lds(double* A, double* V, int rn, int* pairs) {
  __shared__ int rotated;
  __shared__ double cs[TDB_RCAP], sn[TDB_RCAP];
  const int m = rn + (rn & 1);               // even size with a dummy index
  __shared__ double dmax_l;
  if (threadIdx.x == 0) {
    double mx = 0.0;
    for (int i = 0; i < rn; ++i) mx = fmax(mx, fabs(A[i * rn + i]));
    dmax_l = mx;
  }
  __syncthreads();
  const double tol = TDB_JACOBI_TOL * dmax_l;
  if (V)
    for (int t = threadIdx.x; t < rn * rn; t += blockDim.x) V[t] = (t / rn == t % rn) ? 1.0 : 0.0;
  __syncthreads();
  for (int sweep = 0; sweep < 40; ++sweep) {
    if (threadIdx.x == 0) rotated = 0;
    __syncthreads();
    for (int round = 0; round < m - 1; ++round) {
      // round-robin schedule: index m-1 fixed, others rotate
      for (int k = threadIdx.x; k < m / 2; k += blockDim.x) {
        int p_, q_;
        if (k == 0) { p_ = m - 1; q_ = round; }
        else { p_ = (round + k) % (m - 1); q_ = (round - k + (m - 1)) % (m - 1); }
        if (p_ > q_) { const int t = p_; p_ = q_; q_ = t; }
        pairs[2 * k] = p_;
        pairs[2 * k + 1] = q_;
        double c = 1.0, s = 0.0;
        if (q_ < rn) {
          const double apq = A[p_ * rn + q_];
          const double app = A[p_ * rn + p_], aqq = A[q_ * rn + q_];
          if (fabs(apq) > 1e-300 && fabs(apq) > tol) {
            const double theta = (aqq - app) / (2.0 * apq);
            const double tt = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
            c = 1.0 / sqrt(tt * tt + 1.0);
            s = tt * c;
            rotated = 1;
          }
        }
        cs[k] = c;
        sn[k] = s;
      }
      __syncthreads();
      // rows: A <- J^T A
      for (int t = threadIdx.x; t < (m / 2) * rn; t += blockDim.x) {
        const int k = t / rn, col = t % rn;
        const int p_ = pairs[2 * k], q_ = pairs[2 * k + 1];
        if (q_ >= rn || sn[k] == 0.0) continue;
        const double ap = A[p_ * rn + col], aq = A[q_ * rn + col];
        A[p_ * rn + col] = cs[k] * ap - sn[k] * aq;
        A[q_ * rn + col] = sn[k] * ap + cs[k] * aq;
      }
      __syncthreads();
      // columns: A <- A J, V <- V J
      for (int t = threadIdx.x; t < (m / 2) * rn; t += blockDim.x) {
        const int k = t / rn, row = t % rn;
        const int p_ = pairs[2 * k], q_ = pairs[2 * k + 1];
        if (q_ >= rn || sn[k] == 0.0) continue;
        const double ap = A[row * rn + p_], aq = A[row * rn + q_];
        A[row * rn + p_] = cs[k] * ap - sn[k] * aq;
        A[row * rn + q_] = sn[k] * ap + cs[k] * aq;
        if (V) {
          const double vp = V[row * rn + p_], vq = V[row * rn + q_];
          V[row * rn + p_] = cs[k] * vp - sn[k] * vq;
          V[row * rn + q_] = sn[k] * vp + cs[k] * vq;
        }
      }
      __syncthreads();
    }
    if (!rotated) break;
    __syncthreads();
  }
  __syncthreads();
}

static __device__ void jacobi_values(double* A, int rn, int* pairs) { jacobi_lds(A, nullptr, rn, pairs); }

// Eigenvalues of a symmetric rn x rn LDS matrix (rn <= 64) by cyclic Jacobi run by one
// wave (lanes 0..63 of the calling block, all of which must call it): round-robin
// pairing, rotations computed by one lane per pair, row and column updates spread
// over the lanes. Only wave-level ordering is needed, so no block barriers.
static __device__ void jacobi_wave(double* A, int rn, int* pairs) {
  __shared__ double cs_w[TDB_RCAP], sn_w[TDB_RCAP];
  __shared__ int rot_w;
  const int lane = threadIdx.x & 63;
  const int m = rn + (rn & 1);
  double mx = 0.0;
  for (int i = lane; i < rn; i += 64) mx = fmax(mx, fabs(A[i * rn + i]));
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
  const double tol = TDB_JACOBI_TOL * mx;
  for (int sweep = 0; sweep < 40; ++sweep) {
    if (lane == 0) rot_w = 0;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    for (int round = 0; round < m - 1; ++round) {
      for (int k = lane; k < m / 2; k += 64) {
        int p_, q_;
        if (k == 0) { p_ = m - 1; q_ = round; }
        else { p_ = (round + k) % (m - 1); q_ = (round - k + (m - 1)) % (m - 1); }
        if (p_ > q_) { const int t = p_; p_ = q_; q_ = t; }
        pairs[2 * k] = p_;
        pairs[2 * k + 1] = q_;
        double c = 1.0, s = 0.0;
        if (q_ < rn) {
          const double apq = A[p_ * rn + q_];
          const double app = A[p_ * rn + p_], aqq = A[q_ * rn + q_];
          if (fabs(apq) > 1e-300 && fabs(apq) > tol) {
            const double theta = (aqq - app) / (2.0 * apq);
            const double tt = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
            c = 1.0 / sqrt(tt * tt + 1.0);
            s = tt * c;
            rot_w = 1;
          }
        }
        cs_w[k] = c;
        sn_w[k] = s;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      for (int t = lane; t < (m / 2) * rn; t += 64) {
        const int k = t / rn, col = t % rn;
        const int p_ = pairs[2 * k], q_ = pairs[2 * k + 1];
        if (q_ >= rn || sn_w[k] == 0.0) continue;
        const double ap = A[p_ * rn + col], aq = A[q_ * rn + col];
        A[p_ * rn + col] = cs_w[k] * ap - sn_w[k] * aq;
        A[q_ * rn + col] = sn_w[k] * ap + cs_w[k] * aq;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
      for (int t = lane; t < (m / 2) * rn; t += 64) {
        const int k = t / rn, row = t % rn;
        const int p_ = pairs[2 * k], q_ = pairs[2 * k + 1];
        if (q_ >= rn || sn_w[k] == 0.0) continue;
        const double ap = A[row * rn + p_], aq = A[row * rn + q_];
        A[row * rn + p_] = cs_w[k] * ap - sn_w[k] * aq;
        A[row * rn + q_] = sn_w[k] * ap + cs_w[k] * aq;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    }
    if (!rot_w) break;
  }
}

// ---------------------------------------------------------------- controller
// Single thread (called by one thread): reads eps^2, nu^2 of the error pass and decides the step's event
// (Sec. 2.5): an add when eps exceeds the trigger, a removal check when the error
// slope over the window is negative with headroom and some mode's weakest direction
// fits in the budget, a restart on a numerical event.
// First part of the decision: error and norm, numerical events, additions, the slope
// window. Returns true when the removal test has to run (drop a direction if the error
// stays within budget without it): eps^2 + sigma_min^2 <= B for some core unfolding.
static __device__ bool controller_pre(CtrlState* c) {
  c->eps = sqrt_sum_sq(c->eps2);
  c->nu = sqrt_sum_sq(c->nu2);
  c->event = 0;
  c->eps_after = __builtin_nan("");
  c->rank_changed = 0;
  // a numerical event (the state was kept) comes before an error that is not finite
  // only because of it; non-finite data come first
  if (!(c->numeric & NUM_NONFINITE) && (c->numeric & (NUM_CORE | NUM_BASIS))) {
    c->decision = DEC_NUMERIC;
    return false;
  }
  if ((c->numeric & NUM_NONFINITE) || !isfinite(c->eps2) || !isfinite(c->nu2)) {
    // non-finite data: the step was not applied; the flags its stages raised on the
    // non-finite values go with it (a failure of the next step's core Gram, found on
    // the kept state, stays for that step)
    c->numeric &= NUM_NEXT;
    c->eps = __builtin_nan("");
    c->decision = DEC_NONFINITE;
    return false;
  }
  if (!c->adaptive) { c->decision = DEC_NONE; return false; }
  const double eps = c->eps;
  if (eps > c->eps_trig) { c->decision = DEC_ADD; return false; }
  const int nw = c->slope_window;
  c->window[c->whead] = eps;
  c->whead = (c->whead + 1) % TDB_WIN;
  c->wcount += 1;
  c->decision = DEC_NONE;
  if (c->wcount < nw) return false;
  const double last = c->window[(c->whead - 1 + TDB_WIN) % TDB_WIN];
  const double first = c->window[(c->whead - nw + TDB_WIN) % TDB_WIN];
  const double slope = (last - first) / ((nw - 1) * c->dt);
  if (!(slope < 0.0)) return false;
  if (eps > 0.5 * c->eps_th) return false;
  return true;
}

}  // namespace tdb

namespace tdb {

// floor(t / d) for 0 <= t < 2^22 and d >= 1, given inv = 1.0f / d: the float quotient
// is within one of the exact one (relative error below 2^-23), and the remainder
// corrects it.
__device__ __forceinline__ int small_div(int t, int d, float inv) {
  int q = (int)((float)t * inv);
  const int r = t - q * d;
  q += (r >= d) ? 1 : 0;
  q -= (r < 0) ? 1 : 0;
  return q;
}

// ===================================================================== block copies
// Copy n values from global memory into LDS (converted to the LDS type), with up to 16
// loads in flight per thread before any is stored, so that a short copy costs one
// memory round trip rather than one per loop iteration.
template <typename TS, typename TL>
__device__ __forceinline__ void g2l(TL* dst, const TS* src, int n) {
  for (int base = 0; base < n; base += 16 * (int)blockDim.x) {
    TS v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int t = base + u * (int)blockDim.x + (int)threadIdx.x;
      v[u] = t < n ? src[t] : (TS)0;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int t = base + u * (int)blockDim.x + (int)threadIdx.x;
      if (t < n) dst[t] = (TL)v[u];
    }
  }
}

// Up to five such copies in one pass (one round trip for all of them); a segment with
// n = 0 is skipped.
__device__ __forceinline__ void g2l5(double* d0, const double* s0, int n0, double* d1, const double* s1, int n1,
                                     double* d2, const double* s2, int n2, double* d3, const double* s3, int n3,
                                     double* d4, const double* s4, int n4) {
  const int e0 = n0, e1 = e0 + n1, e2 = e1 + n2, e3 = e2 + n3, e4 = e3 + n4;
  for (int base = 0; base < e4; base += 16 * (int)blockDim.x) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int t = base + u * (int)blockDim.x + (int)threadIdx.x;
      double x = 0.0;
      if (t < e0) x = s0[t];
      else if (t < e1) x = s1[t - e0];
      else if (t < e2) x = s2[t - e1];
      else if (t < e3) x = s3[t - e2];
      else if (t < e4) x = s4[t - e3];
      v[u] = x;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int t = base + u * (int)blockDim.x + (int)threadIdx.x;
      if (t < e0) d0[t] = v[u];
      else if (t < e1) d1[t - e0] = v[u];
      else if (t < e2) d2[t - e1] = v[u];
      else if (t < e3) d3[t - e2] = v[u];
      else if (t < e4) d4[t - e3] = v[u];
    }
  }
}

// ===================================================================== one-wave kernels
// The routines below are run by one full wave (64 lanes) of the calling block on small
// (rn <= 64) row-major matrices in LDS. Lanes own rows or columns; ordering between
// lanes only needs wave-level memory ordering, so no block barriers are used.
__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); }

__device__ __forceinline__ double wave_sum_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ double wave_max_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// ------------------------------------------------ Cholesky factor and inverse by one wave
// 1/sqrt(x) for x > 0 to full FP64 accuracy: the hardware estimate and two Newton steps.
__device__ __forceinline__ double rsqrt_nr(double x) {
  double r = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * x;
  r = fma(r, fma(-h * r, r, 0.5), r);
  r = fma(r, fma(-h * r, r, 0.5), r);
  return r;
}
// 1/x likewise.
__device__ __forceinline__ double rcp_nr(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  r = fma(r, fma(-x, r, 1.0), r);
  return r;
}

typedef double wd4 __attribute__((ext_vector_type(4)));

// acc += A B over K (a multiple of 4) by one wave on the FP64 16x16x4 matrix instructions:
// A(m, k) = fa(m, k), B(k, n) = fb(k, n) for m, n < 16. Entry i of the result is row
// lane / 16 + 4 i, column lane % 16.
template <int K, typename FA, typename FB>
__device__ __forceinline__ wd4 mm16(FA fa, FB fb, wd4 acc) {
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  double x[K / 4], y[K / 4];
#pragma unroll
  for (int k = 0; k < K / 4; ++k) {
    x[k] = fa(m, 4 * k + g);
    y[k] = fb(4 * k + g, m);
  }
#pragma unroll
  for (int k = 0; k < K / 4; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k], y[k], acc, 0, 0, 0);
  return acc;
}
template <typename FE>
__device__ __forceinline__ void each16(const wd4& acc, FE emit) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < 4; ++i) emit((lane >> 4) + 4 * i, lane & 15, acc[i]);
}

// Diagonal block at k0 of the symmetric n x n matrix A (LDS, row stride ld, lower triangle
// read): its Cholesky factor in place (zeros above) and the inverse of that in the same
// block of Li. Elimination of [A | I] with lane c holding column c (c < 16: A, c - 16: I) in
// registers: each step broadcasts one column to all lanes, which serves the factor and
// the inverse at once, and keeps the reciprocal of the pivot off the broadcasts. Rows and
// columns from n on are the identity's. S: steps taken, no fewer than the block's rows
// within n (a short block takes fewer dependent steps). Returns false if a pivot is not
// positive or is below TDB_PIVOT_FLOOR dmax.
template <int S>
__device__ __forceinline__ bool wave_chol_block(double* A, double* Li, int ld, int k0, int n, double dmax) {
  const int l = threadIdx.x & 63, c = l & 15;
  const bool isA = l < 16;
  double v[S];
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const int r = max(i, c), q = min(i, c);
    const bool in = isA && k0 + r < n;
    const double x = A[min(k0 + r, n - 1) * ld + min(k0 + q, n - 1)];
    v[i] = in ? x : (i == c ? 1.0 : 0.0);
  }
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const double w = v[k] * rcp_nr(lane_get(v[k], k));
#pragma unroll
    for (int i = k + 1; i < S; ++i) v[i] = fma(-lane_get(v[i], k), w, v[i]);
  }
  // the pivots, one a lane: tested and their roots taken at once (a branch or a root per
  // step would lengthen every step)
  double d = v[0];
#pragma unroll
  for (int i = 1; i < S; ++i) d = c == i ? v[i] : d;
  const bool bad = __any(isA && c < S && k0 + c < n && (!(d > TDB_PIVOT_FLOOR * dmax) || !(d > 0.0)));
  const double rl = rsqrt_nr(fmax(d, 1e-300));
  double rs[S];
#pragma unroll
  for (int i = 0; i < S; ++i) rs[i] = lane_get(rl, i);
  // lane c < 16: entries i <= c of column c are D L^T (row c of L); lane 16 + c: column c of
  // the inverse of the unit lower factor. One store per i for both, predicated per lane
  // (`lim` in a vector register: a scalar test would branch around every store)
  int lim = min(n - k0, S);
  asm volatile("" : "+v"(lim));
  double* dst = isA ? A + (k0 + c) * ld + k0 : Li + k0 * ld + k0 + c;
  const int step = isA ? 1 : ld;
  const bool mine = l < 32 && c < lim;
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const bool in = isA ? i <= c : i >= c;
    const double x = in ? v[i] * rs[i] : 0.0;
    if (mine && i < lim) dst[i * step] = x;
  }
  wave_fence();
  return !bad;
}
__device__ __forceinline__ bool wave_chol16(double* A, double* Li, int ld, int k0, int n, double dmax) {
  if (n - k0 <= 4) return wave_chol_block<4>(A, Li, ld, k0, n, dmax);
  if (n - k0 <= 8) return wave_chol_block<8>(A, Li, ld, k0, n, dmax);
  return wave_chol_block<16>(A, Li, ld, k0, n, dmax);
}

// Lower Cholesky factor of the SPD n x n matrix A (n <= 32, LDS, row stride ld) in place,
// zeros above, its inverse Li and, with Gi, the inverse Gi = Li^T Li of A, all of row
// stride ld, by one full wave (no lane may be masked off), for second-order streams. 16 x 16
// blocks: the diagonal blocks in registers, everything else as matrix products. Returns false
// if a pivot is not positive or is below TDB_PIVOT_FLOOR times the largest diagonal entry; Li
// and Gi are then not all formed.
// Bound by the dependent steps of the elimination. In registers of one lane per row, with
// a second substitution for the inverse, it took 6.0 us at n = 16 and 16.7 at 32; this form
// takes 3.5 and 9.2, and with the short last block's elimination cut to 4 or 8 steps 1.3 at
// n = 3 (3.1 with 16), 1.8 at 8, 5.6 at 17 (8.4) and at 20.
template <int NB>
__device__ __forceinline__ bool wave_chol_inv_nb(double* A, int n, int ld, double* Li, double* Gi) {
  const int l = threadIdx.x & 63;
  const double dmax = wave_max_d(l < n ? A[l * ld + l] : 0.0);
  auto at = [&](const double* M, int i, int j) {      // zero outside the matrix
    const double x = M[min(i, n - 1) * ld + min(j, n - 1)];
    return (i < n && j < n) ? x : 0.0;
  };
  bool ok = true;
#pragma unroll
  for (int kb = 0; kb < NB; ++kb) {
    const int k0 = 16 * kb;
    ok = wave_chol16(A, Li, ld, k0, n, dmax) && ok;
    // L_ik = A_ik L_kk^-T
#pragma unroll
    for (int ib = kb + 1; ib < NB; ++ib) {
      const int i0 = 16 * ib;
      const wd4 r = mm16<16>([&](int i, int k) { return at(A, i0 + i, k0 + k); },
                             [&](int k, int j) { return at(Li, k0 + j, k0 + k); }, (wd4){0, 0, 0, 0});
      wave_fence();
      each16(r, [&](int i, int j, double v) {
        if (i0 + i < n) { A[(i0 + i) * ld + k0 + j] = v; A[(k0 + j) * ld + i0 + i] = 0.0; }
      });
    }
    wave_fence();
    // A_ij -= L_ik L_jk^T
#pragma unroll
    for (int ib = kb + 1; ib < NB; ++ib)
#pragma unroll
      for (int jb = kb + 1; jb <= ib; ++jb) {
        const int i0 = 16 * ib, j0 = 16 * jb;
        wd4 c;
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = at(A, i0 + (l >> 4) + 4 * i, j0 + (l & 15));
        c = mm16<16>([&](int i, int k) { return -at(A, i0 + i, k0 + k); },
                     [&](int k, int j) { return at(A, j0 + j, k0 + k); }, c);
        each16(c, [&](int i, int j, double v) {
          if (i0 + i < n && j0 + j < n) A[(i0 + i) * ld + j0 + j] = v;
        });
      }
    wave_fence();
  }
  if (!ok) return false;
  // L^-1: X_ij = -Linv_ii sum_{j <= k < i} L_ik X_kj
#pragma unroll
  for (int d = 1; d < NB; ++d)
#pragma unroll
    for (int jb = 0; jb + d < NB; ++jb) {
      const int ib = jb + d, i0 = 16 * ib, j0 = 16 * jb;
      wd4 r = {0, 0, 0, 0};
#pragma unroll
      for (int kb = jb; kb < ib; ++kb)
        r = mm16<16>([&](int i, int k) { return at(A, i0 + i, 16 * kb + k); },
                     [&](int k, int j) { return at(Li, 16 * kb + k, j0 + j); }, r);
      each16(r, [&](int i, int j, double v) {
        if (i0 + i < n) { Li[(i0 + i) * ld + j0 + j] = v; Li[(j0 + j) * ld + i0 + i] = 0.0; }
      });
      wave_fence();
      r = mm16<16>([&](int i, int k) { return -at(Li, i0 + i, i0 + k); },
                   [&](int k, int j) { return at(Li, i0 + k, j0 + j); }, (wd4){0, 0, 0, 0});
      wave_fence();
      each16(r, [&](int i, int j, double v) {
        if (i0 + i < n) Li[(i0 + i) * ld + j0 + j] = v;
      });
      wave_fence();
    }
  if (Gi) {
#pragma unroll
    for (int ib = 0; ib < NB; ++ib)
#pragma unroll
      for (int jb = 0; jb <= ib; ++jb) {
        const int i0 = 16 * ib, j0 = 16 * jb;
        wd4 r = {0, 0, 0, 0};
#pragma unroll
        for (int kb = ib; kb < NB; ++kb)
          r = mm16<16>([&](int i, int k) { return at(Li, 16 * kb + k, i0 + i); },
                       [&](int k, int j) { return at(Li, 16 * kb + k, j0 + j); }, r);
        each16(r, [&](int i, int j, double v) {
          if (i0 + i < n && j0 + j < n) {
            Gi[(i0 + i) * ld + j0 + j] = v;
            if (ib != jb) Gi[(j0 + j) * ld + i0 + i] = v;
          }
        });
      }
  }
  wave_fence();
  return true;
}

// ------------------------------------------------ the same, operation by operation
// The forms for the state of a third-order stream: a stream that holds directions near the
// noise floor turns one rounding of these matrices into changes of its reconstruction that can
// be seen, so each entry goes through one fixed sequence of operations, whatever the split
// over lanes and matrix instructions: right-looking, one column after another,
//   l_jj = a_jj r, l_ij = a_ij r with r = rsqrt(a_jj), a_ik <- fma(-l_ij, l_kj, a_ik),
// and for each column of the inverse, x_j <- x_j r, x_i <- fma(-l_ij, x_j, x_i); above 32 rows
//   l_jj = sqrt(a_jj), l_ij = a_ij / l_jj, x_jj = 1 / l_jj, x_ij = -(sum_k l_ik x_kj) / l_ii.
// A 16x16x4 FP64 product is an ascending chain of fused multiply-adds, so it takes the place
// of any run of such updates.
// Bound by the dependent steps. With Gi: 1.0 us at n = 4, 1.6 at 8, 3.4 at 16, 5.9 at 18, 9.9 at
// 32, 26 at 33 and 54 at 64; one lane per row with the inverse as a second substitution took
// 5.7, 5.8, 6.0, 16.3 and 16.8, and with loops over LDS above 32 rows 95 and 388.

// Largest of the lanes' values (none of them NaN), in every lane.
__device__ __forceinline__ double wave_max_dpp(double v) {
  v = fmax(v, dpp_get<0xB1>(v));
  v = fmax(v, dpp_get<0x4E>(v));
  v = fmax(v, dpp_get<0x141>(v));
  v = fmax(v, dpp_get<0x140>(v));
  return fmax(fmax(lane_get(v, 0), lane_get(v, 16)), fmax(lane_get(v, 32), lane_get(v, 48)));
}

// Columns k0 .. k0 + S - 1 of the factor of A, n <= 32 (row-major, stride n): lane c < 32
// holds row c, lane 32 + c column c of the inverse, so that a step's broadcasts serve both.
// Li holds, in the rows of the panel, what the earlier panels have subtracted. RD: the
// inverse's rows are scaled by 1 / l_jj instead of r. Rows and columns from n on are the
// identity's. Returns false if a pivot is not positive or not above `floor`.
template <int S, bool RD>
__device__ __forceinline__ bool wave_panel(double* A, double* Li, int n, int k0, double floor) {
  const int l = threadIdx.x & 63, c = l & 31;
  const bool isX = l >= 32;
  double v[S], piv[S];
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const int q = k0 + j, qc = min(q, n - 1), cc = min(c, n - 1);
    const double x = *(isX ? Li + qc * n + cc : A + cc * n + qc);
    v[j] = (q < n && c < n && (isX ? c < k0 : c >= k0)) ? x : (c == q ? 1.0 : 0.0);
  }
#pragma unroll
  for (int k = 0; k < S; ++k) {
    piv[k] = lane_get(v[k], k0 + k);
    const double pv = fmax(piv[k], 1e-300), r = rsqrt_nr(pv), lk = pv * r;
    const double f = RD && isX ? 1.0 / lk : r;
    v[k] = (!isX && c == k0 + k) ? lk : v[k] * f;
#pragma unroll
    for (int j = k + 1; j < S; ++j) v[j] = fma(-v[k], lane_get(v[k], k0 + j), v[j]);
  }
  bool ok = true;
#pragma unroll
  for (int k = 0; k < S; ++k) ok = ok && (k0 + k >= n || (piv[k] > floor && piv[k] > 0.0));
  // one store per column for both, predicated per lane (`lim` in a vector register: a scalar
  // test would branch around every store)
  int lim = min(n - k0, S);
  asm volatile("" : "+v"(lim));
  double* dst = isX ? Li + k0 * n + c : A + c * n + k0;
  const int step = isX ? n : 1;
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const double x = (isX || k0 + j <= c) ? v[j] : 0.0;
    if (c < n && j < lim) dst[j * step] = x;
  }
  wave_fence();
  return ok;
}

// Gi = Li^T Li (n <= 16 NB, row stride n), sums over the rows in order.
template <int NB, typename PL>
__device__ __forceinline__ void wave_inv_gram(PL Li, PL Gi, int n) {
  auto at = [&](int i, int j) {
    const double x = Li[min(i, n - 1) * n + min(j, n - 1)];
    return (i < n && j < n) ? x : 0.0;
  };
#pragma unroll
  for (int ib = 0; ib < NB; ++ib)
#pragma unroll
    for (int jb = 0; jb <= ib; ++jb) {
      const int i0 = 16 * ib, j0 = 16 * jb;
      wd4 r = {0, 0, 0, 0};
#pragma unroll
      for (int kb = ib; kb < NB; ++kb)
        r = mm16<16>([&](int i, int k) { return at(16 * kb + k, i0 + i); },
                     [&](int k, int j) { return at(16 * kb + k, j0 + j); }, r);
      each16(r, [&](int i, int j, double v) {
        if (i0 + i < n && j0 + j < n) {
          Gi[(i0 + i) * n + j0 + j] = v;
          if (ib != jb) Gi[(j0 + j) * n + i0 + i] = v;
        }
      });
    }
}

template <int S, bool RD>
__device__ __forceinline__ bool wave_chol_inv_s(double* A, int n, double* Li, double* Gi) {
  const int l = threadIdx.x & 63;
  const double x = A[min(l, n - 1) * (n + 1)];
  const double floor = TDB_PIVOT_FLOOR * wave_max_dpp(l < n ? fmax(x, 0.0) : 0.0);
  const bool ok = wave_panel<S, RD>(A, Li, n, 0, floor);
  if (Gi && ok) wave_inv_gram<1, double*>(Li, Gi, n);
  wave_fence();
  return ok;
}
template <bool RD>
__device__ __forceinline__ bool wave_chol_inv_2(double* A, int n, double* Li, double* Gi) {
  const int l = threadIdx.x & 63;
  const double x = A[min(l, n - 1) * (n + 1)];
  const double floor = TDB_PIVOT_FLOOR * wave_max_dpp(l < n ? fmax(x, 0.0) : 0.0);
  bool ok = wave_panel<16, RD>(A, Li, n, 0, floor);
  auto at = [&](const double* M, int i, int j) {      // zero outside the matrix
    const double m = M[min(i, n - 1) * n + min(j, n - 1)];
    return (i < n && j < n) ? m : 0.0;
  };
  // A_11 -= L_10 L_10^T and X_10 = -L_10 X_00
  wd4 c;
#pragma unroll
  for (int i = 0; i < 4; ++i) c[i] = at(A, 16 + (l >> 4) + 4 * i, 16 + (l & 15));
  c = mm16<16>([&](int i, int k) { return -at(A, 16 + i, k); }, [&](int k, int j) { return at(A, 16 + j, k); }, c);
  const wd4 y = mm16<16>([&](int i, int k) { return -at(A, 16 + i, k); }, [&](int k, int j) { return at(Li, k, j); },
                         (wd4){0, 0, 0, 0});
  wave_fence();
  each16(c, [&](int i, int j, double v) {
    if (16 + i < n && 16 + j < n) A[(16 + i) * n + 16 + j] = v;
  });
  each16(y, [&](int i, int j, double v) {
    if (16 + i < n) Li[(16 + i) * n + j] = v;
  });
  wave_fence();
  ok = (n <= 20 ? wave_panel<4, RD>(A, Li, n, 16, floor)
                : n <= 24 ? wave_panel<8, RD>(A, Li, n, 16, floor) : wave_panel<16, RD>(A, Li, n, 16, floor)) && ok;
  if (Gi && ok) wave_inv_gram<2, double*>(Li, Gi, n);
  wave_fence();
  return ok;
}

// 32 < n <= 64 (out of line: rare and long). A in LDS, Li and Gi there too or anywhere (PL: the
// pointers' type; through plain pointers every access would be a flat one).
typedef __attribute__((address_space(3))) double lds_double;
template <bool GRAM, typename PL>
static __device__ __attribute__((noinline)) bool wave_chol_inv_big(lds_double* A, int n, PL Li, PL Gi) {
  const int l = threadIdx.x & 63, nb = (n + 15) >> 4;
  const double dx = A[min(l, n - 1) * (n + 1)];
  const double floor = TDB_PIVOT_FLOOR * wave_max_dpp(l < n ? fmax(dx, 0.0) : 0.0);
  auto at = [&](auto M, int i, int j) {
    const double m = M[min(i, n - 1) * n + min(j, n - 1)];
    return (i < n && j < n) ? m : 0.0;
  };
  bool ok = true;
  for (int kb = 0; kb < nb; ++kb) {
    // lane l: row l of the panel's columns
    const int k0 = 16 * kb;
    double v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const double x = A[min(l, n - 1) * n + min(k0 + j, n - 1)];
      v[j] = (l < n && k0 + j < n) ? x : (l == k0 + j ? 1.0 : 0.0);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (k0 + k >= n) break;
      const double piv = lane_get(v[k], k0 + k);
      ok = ok && piv > floor && piv > 0.0;
      const double lk = sqrt(fmax(piv, 1e-300));
      v[k] = l == k0 + k ? lk : v[k] / lk;
#pragma unroll
      for (int j = k + 1; j < 16; ++j) v[j] = fma(-v[k], lane_get(v[k], k0 + j), v[j]);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (l < n && k0 + j < n) A[l * n + k0 + j] = k0 + j <= l ? v[j] : 0.0;
    wave_fence();
    for (int ib = kb + 1; ib < nb; ++ib)
      for (int jb = kb + 1; jb <= ib; ++jb) {
        const int i0 = 16 * ib, j0 = 16 * jb;
        wd4 c;
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = at(A, i0 + (l >> 4) + 4 * i, j0 + (l & 15));
        c = mm16<16>([&](int i, int k) { return -at(A, i0 + i, k0 + k); },
                     [&](int k, int j) { return at(A, j0 + j, k0 + k); }, c);
        each16(c, [&](int i, int j, double x) {
          if (i0 + i < n && j0 + j < n) A[(i0 + i) * n + j0 + j] = x;
        });
      }
    wave_fence();
  }
  if (!ok) return false;
  for (int ib = 0; ib < nb; ++ib) {
    // rows i0 .. i0 + 15 of the inverse: the sums over the earlier rows, then lane l column l
    const int i0 = 16 * ib;
    for (int jb = 0; jb < ib; ++jb) {
      wd4 r = {0, 0, 0, 0};
      for (int kb = jb; kb < ib; ++kb)
        r = mm16<16>([&](int i, int k) { return at(A, i0 + i, 16 * kb + k); },
                     [&](int k, int j) { return at(Li, 16 * kb + k, 16 * jb + j); }, r);
      each16(r, [&](int i, int j, double x) {
        if (i0 + i < n) Li[(i0 + i) * n + 16 * jb + j] = x;
      });
    }
    wave_fence();
    // (the rows of the diagonal block, one a lane, so that a coefficient is a lane's value)
    double s[16], c[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const double x = Li[min(i0 + i, n - 1) * n + min(l, n - 1)];
      s[i] = l < i0 ? x : 0.0;
      c[i] = A[min(i0 + (l & 15), n - 1) * n + min(i0 + i, n - 1)];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i0 + i >= n) break;
      const double lii = lane_get(c[i], i);
      const double num = l == i0 + i ? 1.0 : -s[i];
      const double y = l <= i0 + i ? num / lii : 0.0;
      s[i] = y;
#pragma unroll
      for (int m = i + 1; m < 16; ++m) s[m] = fma(lane_get(c[i], m), y, s[m]);
    }
    wave_fence();
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (l < n && i0 + i < n) Li[(i0 + i) * n + l] = s[i];
    wave_fence();
  }
  if (GRAM) {
    if (n <= 48) wave_inv_gram<3, PL>(Li, Gi, n);
    else wave_inv_gram<4, PL>(Li, Gi, n);
  }
  wave_fence();
  return true;
}

// Lower Cholesky factor of the SPD n x n matrix A (n <= 64, LDS, row stride n) in place, zeros
// above, its inverse Li (RD: see wave_panel) and, unless RD, Gi = Li^T Li, by one full wave (no
// lane may be masked off); Li and Gi in LDS unless FAR. Returns false if a pivot is not positive or not above
// TDB_PIVOT_FLOOR times the largest diagonal entry; Gi is then not formed.
template <bool RD, bool FAR = false>
__device__ __forceinline__ bool wave_chol_inv(double* A, int n, double* Li, double* Gi) {
  if (n <= 4) return wave_chol_inv_s<4, RD>(A, n, Li, Gi);
  if (n <= 8) return wave_chol_inv_s<8, RD>(A, n, Li, Gi);
  if (n <= 16) return wave_chol_inv_s<16, RD>(A, n, Li, Gi);
  if (n <= 32) return wave_chol_inv_2<RD>(A, n, Li, Gi);
  // (RD: the caller wants no Gi)
  lds_double* a = (lds_double*)A;
  if (FAR) return wave_chol_inv_big<!RD>(a, n, Li, RD ? Li : Gi);
  return wave_chol_inv_big<!RD>(a, n, (lds_double*)Li, (lds_double*)(RD ? Li : Gi));
}

// Whether the symmetric n x n matrix A (n <= 64, LDS, row-major, lower triangle read) is
// positive definite: its Cholesky factorisation by one full wave, 16 x 16 blocks at a time,
// meets positive pivots only. A is overwritten; D: 16 n doubles of scratch. (Right-looking
// with one column a step the test of three modes took 9.9 us at n = 18, now 5.5.)
__device__ __forceinline__ bool wave_chol_pd(double* A, int n, double* D) {
  const int l = threadIdx.x & 63;
  auto at = [&](int i, int j) {
    const double x = A[min(i, n - 1) * n + min(j, n - 1)];
    return (i < n && j < n) ? x : 0.0;
  };
  for (int k0 = 0; k0 < n; k0 += 16) {
    // (the block's inverse factor: entry (i, j) at D[i n + j], so D - k0 n - k0 is its origin)
    if (!wave_chol16(A, D - k0 * n - k0, n, k0, n, 0.0)) return false;
    for (int i0 = k0 + 16; i0 < n; i0 += 16) {
      const wd4 r = mm16<16>([&](int i, int k) { return at(i0 + i, k0 + k); },
                             [&](int k, int j) { return (k0 + j < n && k0 + k < n) ? D[j * n + k] : 0.0; },
                             (wd4){0, 0, 0, 0});
      wave_fence();
      each16(r, [&](int i, int j, double v) {
        if (i0 + i < n) A[(i0 + i) * n + k0 + j] = v;
      });
    }
    wave_fence();
    for (int i0 = k0 + 16; i0 < n; i0 += 16)
      for (int j0 = k0 + 16; j0 <= i0; j0 += 16) {
        wd4 c;
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = at(i0 + (l >> 4) + 4 * i, j0 + (l & 15));
        c = mm16<16>([&](int i, int k) { return -at(i0 + i, k0 + k); },
                     [&](int k, int j) { return at(j0 + j, k0 + k); }, c);
        each16(c, [&](int i, int j, double v) {
          if (i0 + i < n && j0 + j < n) A[(i0 + i) * n + j0 + j] = v;
        });
      }
    wave_fence();
  }
  return true;
}

// Eigenvalues of the symmetric matrix A (destroyed), descending, into lam[0..rn):
// Householder reduction to tridiagonal form (lane i owns row i of the trailing block),
// then bisection on Sturm counts with one eigenvalue per lane. ws: LDS scratch of
// 4*rn doubles.
static __device__ void wave_eigvals(double* A, int rn, double* lam, double* ws) {
  const int lane = threadIdx.x & 63;
  double* d = ws;
  double* e2 = ws + rn;
  double* v = ws + 2 * rn;
  double* wv = ws + 3 * rn;
  for (int k = 0; k + 2 < rn; ++k) {
    const int m = rn - k - 1;
    const double x = lane < m ? A[(k + 1 + lane) * rn + k] : 0.0;
    const double ss = wave_sum_d(x * x);
    const double x0 = __shfl(x, 0, 64);
    double bk = 0.0, ek = x0;
    double vi = x;
    if (ss > 0.0) {
      const double xn = sqrt(ss);
      const double alpha = x0 > 0.0 ? -xn : xn;
      const double v0 = x0 - alpha;
      bk = 2.0 / (ss - x0 * x0 + v0 * v0);
      ek = alpha;
      if (lane == 0) vi = v0;
    }
    if (lane == 0) { d[k] = A[k * rn + k]; e2[k] = ek * ek; }
    if (lane < m) v[lane] = vi;
    wave_fence();
    if (bk != 0.0) {
      double p = 0.0;
      if (lane < m) {
        const double* row = A + (k + 1 + lane) * rn + (k + 1);
        for (int j = 0; j < m; ++j) p += row[j] * v[j];
        p *= bk;
      }
      const double Kc = 0.5 * bk * wave_sum_d(lane < m ? p * vi : 0.0);
      if (lane < m) wv[lane] = p - Kc * vi;
      wave_fence();
      if (lane < m) {
        double* row = A + (k + 1 + lane) * rn + (k + 1);
        const double wi = wv[lane];
        for (int j = 0; j < m; ++j) row[j] -= vi * wv[j] + wi * v[j];
      }
      wave_fence();
    }
  }
  if (lane == 0) {
    if (rn >= 2) {
      d[rn - 2] = A[(rn - 2) * rn + (rn - 2)];
      const double el = A[(rn - 1) * rn + (rn - 2)];
      e2[rn - 2] = el * el;
    }
    d[rn - 1] = A[(rn - 1) * rn + (rn - 1)];
  }
  wave_fence();
  // Gershgorin interval
  double lo = 1e300, hi = -1e300, mx = 0.0, me = 0.0;
  for (int i = lane; i < rn; i += 64) {
    const double off = (i > 0 ? sqrt(e2[i - 1]) : 0.0) + (i + 1 < rn ? sqrt(e2[i]) : 0.0);
    lo = fmin(lo, d[i] - off);
    hi = fmax(hi, d[i] + off);
    mx = fmax(mx, fabs(d[i]) + off);
    if (i + 1 < rn) me = fmax(me, e2[i]);
  }
  lo = -wave_max_d(-lo);
  hi = wave_max_d(hi);
  mx = wave_max_d(mx);
  me = wave_max_d(me);
  const double eps = 2.220446049250313e-16;
  const double pivmin = 2.2250738585072014e-308 * fmax(1.0, me);
  lo -= 4.0 * eps * mx + 2.0 * pivmin;
  hi += 4.0 * eps * mx + 2.0 * pivmin;
  // multisection: L lanes per eigenvalue evaluate Sturm counts at L interior points
  int L = 1;
  while (L < 16 && (2 * L) * rn <= 64) L *= 2;
  const int e = lane / L, sub = lane - (lane / L) * L;
  const int idx = rn - 1 - e;               // ascending index of the e-th largest
  double a = lo, b = hi;
  const double invL1 = 1.0 / (double)(L + 1);
  int its = 1;
  {
    int bits = 0;
    for (int q = L + 1; q > 1; q >>= 1) ++bits;      // floor(log2(L+1)) bits per round
    its = (56 + bits - 1) / bits + 1;
  }
  for (int it = 0; it < its; ++it) {
    const double x = a + (b - a) * ((double)(sub + 1) * invL1);
    int c = 0;
    if (e < rn) {
      double q = d[0] - x;
      if (fabs(q) < pivmin) q = -pivmin;
      c += q < 0.0;
      for (int i = 1; i < rn; ++i) {
        double r0 = __builtin_amdgcn_rcp(q);
        r0 = r0 * (2.0 - q * r0);
        r0 = r0 * (2.0 - q * r0);
        q = d[i] - x - e2[i - 1] * r0;
        if (fabs(q) < pivmin) q = -pivmin;
        c += q < 0.0;
      }
    }
    const unsigned long long mask = __ballot(c > idx);
    const unsigned grp = (unsigned)((mask >> (e * L)) & ((L == 64) ? ~0ull : ((1ull << L) - 1ull)));
    const int f = grp ? __builtin_ctz(grp) : L;   // first sub-point above the target
    const double na = (f == 0) ? a : a + (b - a) * ((double)f * invL1);
    const double nb = (f == L) ? b : a + (b - a) * ((double)(f + 1) * invL1);
    a = na;
    b = nb;
  }
  if (e < rn && sub == 0) lam[e] = 0.5 * (a + b);
  wave_fence();
}

}  // namespace tdb
