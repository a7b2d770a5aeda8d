// n-mode products on the matrix cores (internal; see ttm_ops.hip).
#pragma once
#include "tdb_common.h"

namespace tdb {

constexpr int TTM_JOBS = 4;

// One product Y[a, o, b] = sum_i M(i, o) X[a, i, b] on a C-ordered tensor viewed as
// (A, Nin, Bsz); with X0 the input is X - X0. M(i, o) = M[i * ms_i + o * ms_o], times
// mw[i] when mw is given.
struct TtmJob {
  const void* X;
  const void* X0;
  const double* M;
  const double* mw;
  void* Y;
  long long A, Bsz, ms_i, ms_o;
  int Nin, Nout;
};

// Products that do not depend on each other, in one launch.
struct TtmGroup {
  int n;
  int chain;   // every output one chain over the contracted rows in order
  TtmJob j[TTM_JOBS];
};

// Weighted error of the last product of a reconstruction R against the snapshot V (both
// laid out as Y): partials[2 * block] = sum w (V - R)^2, [2 * block + 1] = sum w V^2 with
// w = wa[a] wo[o] wb[b].
struct TtmErr {
  const void* V;
  const double *wa, *wo, *wb;
  double* partials;
};

// TX: input type, T: type of the products, TY: output type, S: type of the sums over more than a
// few rows.
template <typename TX, typename T, typename TY, typename S = T>
hipError_t launch_ttm_group(const TtmGroup& g, hipStream_t s);
// The product of `j` against the snapshot; *blocks receives the number of partial
// pairs, at most ttm_err_blocks() of the same job.
template <typename TX, typename T, typename TV>
hipError_t launch_ttm_err(const TtmJob& j, const TtmErr& e, int* blocks, hipStream_t s);
// An upper bound on launch_ttm_err's blocks for an output of `outer` x Nout x Bsz.
long long ttm_err_blocks(long long A, int Nout, long long Bsz);

// Reconstruction C x_1 U_1 x_2 U_2 x_3 U_3 of a third-order state (C dense and C-ordered,
// U[n] N[n] x r[n] with leading dimension ldU[n], all FP64) into out (TY, C-ordered) in one
// launch, T arithmetic. rec3_ok: whether the factors of a block fit the LDS.
struct Rec3Args {
  long long N[3];
  int r[3], ldU[3];
  const double* C;
  const double* U[3];
  void* out;
  int vec, rows;      // (set by the launcher) four values a store; rows of mode 1 a block
};
template <typename T>
bool rec3_ok(const Rec3Args& a);
template <typename T, typename TY>
hipError_t launch_rec3(const Rec3Args& a, hipStream_t s);

}  // namespace tdb
