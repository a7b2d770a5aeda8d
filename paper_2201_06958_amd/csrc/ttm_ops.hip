// n-mode products (tensor times matrix) on the matrix cores, for every path that
// contracts or expands one mode at a time: the projections of orders 2 and 4 (eqs.
// (Corecont), (basecont)), the HOSVD's core, and the reconstruction with or without the
// weighted error of eq. (error) behind it.
//
// A product over the middle index of (A, Nin, Bsz) is, for each a, a matrix product of
// M^T (Nout x Nin) with the Nin x Bsz slice, so the 16x16x4 matrix instructions take M as
// the A operand and 16 columns of the slice as the B operand. Products and sums are of the
// arithmetic type; FP32 products may be summed in FP64. One thread per output
// (the earlier form) read every operand from the caches once per output: 81 us a product
// on average for the 192 x 129 x 192 x 3 FP32 channel at ranks (33, 13, 33, 3).
#include "tdb_common.h"
#include "device_util.h"
#include "ttm.h"
#include <type_traits>

namespace tdb {

typedef float tf4 __attribute__((ext_vector_type(4)));
typedef double td4 __attribute__((ext_vector_type(4)));

template <typename T> struct Acc;
template <> struct Acc<float> {
  typedef tf4 v;
  static __device__ __forceinline__ v mma(float a, float b, v c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // row of result entry i in lane group kg
  static __device__ __forceinline__ int row(int kg, int i) { return 4 * kg + i; }
};
template <> struct Acc<double> {
  typedef td4 v;
  static __device__ __forceinline__ v mma(double a, double b, v c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int kg, int i) { return kg + 4 * i; }
};

// A run of 16 contracted rows: products and their sums within it in T, the sum over the runs
// in S. (With S = T the runs are one chain. FP32 products with FP64 sums: a third-order step of
// 192^3 FP32 at ranks 5 takes 189 us, 206 on the FP64 matrix cores, 184 with FP32 sums of
// whole modes, which were up to ten times as far off.)
template <typename T, typename S>
__device__ __forceinline__ void begin_run(const typename Acc<S>::v& acc, typename Acc<T>::v& run) {
  if constexpr (std::is_same<T, S>::value) run = acc;
  else run = (typename Acc<T>::v){0, 0, 0, 0};
}
template <typename T, typename S>
__device__ __forceinline__ void end_run(const typename Acc<T>::v& run, typename Acc<S>::v& acc) {
  if constexpr (std::is_same<T, S>::value) acc = run;
  else
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += (S)run[i];
}

// Columns a lane takes from one 16-byte load of X.
template <typename TX> constexpr int vec_of() { return 16 / (int)sizeof(TX); }

// LDS bytes of the staged part of M (rows of the contracted index, OT tiles of 16 outputs)
constexpr int TTM_MBYTES = 32768;
template <typename T, int OT> constexpr int mrows() { return (TTM_MBYTES / (OT * 16 * (int)sizeof(T))) & ~15; }
// contracted rows staged at a time when Bsz < 16
constexpr int TTM_KS = 64;

// M of rows k0..k0+kc (a multiple of 16) and outputs o0.. into LDS, zero past the
// matrix: 16 rows by one output sit together as [k % 4][k / 4], so that a lane finds the
// four entries it feeds to four matrix instructions side by side.
template <typename T, int OT>
__device__ __forceinline__ void stage_m(const TtmJob& j, int k0, int kc, int o0, T* Ml) {
  const int tot = kc * OT * 16;
  const bool kfast = j.ms_i == 1;
  for (int t = threadIdx.x; t < tot; t += 256) {
    const int k = kfast ? t % kc : t / (OT * 16);
    const int o = kfast ? t / kc : t % (OT * 16);
    const int gk = k0 + k, go = o0 + o;
    double v = 0.0;
    if (gk < j.Nin && go < j.Nout) {
      const long long e = (long long)gk * j.ms_i + (long long)go * j.ms_o;
      v = j.M[e];
      if (j.mw) v *= j.mw[gk];
    }
    Ml[((k >> 4) * (OT * 16) + o) * 16 + (k & 3) * 4 + ((k & 15) >> 2)] = (T)v;
  }
}

// Whether the sums of four waves over 16 V columns fit the LDS of the staged matrix.
template <typename T, int OT, int V> constexpr bool ks_fits() { return 1024 * OT * V * (int)sizeof(T) <= TTM_MBYTES; }

// Adds the four waves' accumulators of 16 V columns (in wave order, through 1024 OT V values
// of LDS) and hands each lane the sums of its V columns: fn(output, values), thread t's
// outputs being t / 16 + 16 q.
template <typename T, typename S, int OT, int V, typename Fn>
__device__ __forceinline__ void ks_sum(S* lds, const typename Acc<S>::v (&acc)[OT][V], Fn fn) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, c = lane & 15, kg = lane >> 4;
  constexpr int W = 256 * OT * V;
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int i = 0; i < 4; ++i) lds[wv * W + v * 256 * OT + (16 * t + Acc<T>::row(kg, i)) * 16 + c] = acc[t][v][i];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < OT; ++q) {
    const int e = (int)threadIdx.x + 256 * q;
    S val[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const S* l = lds + v * 256 * OT + e;
      val[v] = ((l[0] + l[W]) + l[2 * W]) + l[3 * W];
    }
    fn(e >> 4, val);
  }
}

// Columns with unit stride (Bsz >= 16): a wave takes 16 V consecutive columns of one
// slice and all the outputs of its block (o0 .. o0 + 16 OT). V columns a lane come from
// one load, so column tile v of the wave holds columns V c + v, c < 16, and the V tiles
// of a lane are stored together. The next rows' loads are issued before the current
// rows' products. Bound: memory for the first contractions of a stage (the slices are
// read once), latency for the later ones.
// KS: the four waves of a block share one unit and split its contracted rows (every
// fourth 16 of them), and their sums are added through LDS in wave order.
template <typename TX, typename T, typename S, int V, int RG, int OT, bool KS, typename Emit>
__device__ __forceinline__ void ttm_cols(const TtmJob& j, long long unit0, int o0, T* Ml, Emit emit) {
  typedef TX vx __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int c = lane & 15, kg = lane >> 4;
  const long long ncol = (j.Bsz + 16 * V - 1) / (16 * V);
  const long long units = j.A * ncol;
  const bool live = KS || unit0 + wv < units;
  const long long u = KS ? unit0 : live ? unit0 + wv : units - 1;
  constexpr int STEP = KS ? 64 * RG : 16 * RG;   // rows from one turn of a wave to its next
  const int kw = KS ? 16 * RG * wv : 0;
  const long long a = u / ncol;
  const long long b = (u - a * ncol) * (16 * V) + c * V;
  const long long bc = b < j.Bsz ? b : j.Bsz - V;
  const long long base = a * j.Nin * j.Bsz + bc;
  const TX* X = static_cast<const TX*>(j.X) + base;
  const TX* X0 = j.X0 ? static_cast<const TX*>(j.X0) + base : nullptr;
  typename Acc<S>::v acc[OT][V];
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int v = 0; v < V; ++v) acc[t][v] = (typename Acc<S>::v){0, 0, 0, 0};
  vx x[RG][4], y[RG][4];
  auto load = [&](int k) {
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const long long i = min(k + 16 * g + 4 * s + kg, j.Nin - 1);
        x[g][s] = *reinterpret_cast<const vx*>(X + i * j.Bsz);
        if (X0) y[g][s] = *reinterpret_cast<const vx*>(X0 + i * j.Bsz);
      }
  };
  load(kw);
  constexpr int KC = mrows<T, OT>() & ~(STEP - 1);
  static_assert(KC >= STEP, "a staged chunk holds a turn of every wave");
  for (int k0 = 0; k0 < j.Nin; k0 += KC) {
    const int kc = min(KC, (j.Nin - k0 + 15) & ~15);
    if (k0) __syncthreads();
    stage_m<T, OT>(j, k0, kc, o0, Ml);
    __syncthreads();
    // one turn; tail: rows past the last are its copies, and zeros take their place (a zero of
    // the matrix times an infinity would be NaN)
    auto turn = [&](int k, auto tail) {
      T d[RG][4][V];
#pragma unroll
      for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int v = 0; v < V; ++v) {
            d[g][s][v] = X0 ? (T)x[g][s][v] - (T)y[g][s][v] : (T)x[g][s][v];
            if (tail.value) d[g][s][v] = k0 + k + 16 * g + 4 * s + kg < j.Nin ? d[g][s][v] : (T)0;
          }
      load(k0 + (k + STEP < kc ? k + STEP : kc + kw));
#pragma unroll
      for (int g = 0; g < RG; ++g) {
        if (RG > 1 && k + 16 * g >= kc) break;
        T m[OT][4];
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
          for (int s = 0; s < 4; ++s) m[t][s] = Ml[(((k >> 4) + g) * (OT * 16) + 16 * t + c) * 16 + kg * 4 + s];
        typename Acc<T>::v run[OT][V];
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
          for (int v = 0; v < V; ++v) begin_run<T, S>(acc[t][v], run[t][v]);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int t = 0; t < OT; ++t)
#pragma unroll
            for (int v = 0; v < V; ++v) run[t][v] = Acc<T>::mma(m[t][s], d[g][s][v], run[t][v]);
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
          for (int v = 0; v < V; ++v) end_run<T, S>(run[t][v], acc[t][v]);
      }
    };
    for (int k = kw; k < kc; k += STEP) {
      if (k0 + k + 16 * RG <= j.Nin) turn(k, std::false_type{});
      else turn(k, std::true_type{});
    }
  }
  if constexpr (KS) {
    __syncthreads();
    ks_sum<T, S, OT, V>(reinterpret_cast<S*>(Ml), acc, [&](int o, const S(&val)[V]) {
      if (b < j.Bsz && o0 + o < j.Nout) emit(a, o0 + o, b, (a * j.Nout + o0 + o) * j.Bsz + b, val);
    });
    return;
  }
  if (!live || b >= j.Bsz) return;
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = o0 + 16 * t + Acc<T>::row(kg, i);
      if (o < j.Nout) {
        S val[V];
#pragma unroll
        for (int v = 0; v < V; ++v) val[v] = acc[t][v][i];
        emit(a, o, b, (a * j.Nout + o) * j.Bsz + b, val);
      }
    }
}

// Bsz < 16: the columns of 64 / Bsz slices (at most 64), staged through LDS in chunks
// of TTM_KS contracted rows (each slice's chunk is contiguous in memory), one 16-column
// tile per wave. The slices are padded so that the 16 columns a wave reads at a time fall
// into different banks for Bsz = 1. KS: 16 columns a block, its waves splitting the rows
// of each chunk.
template <typename TX, typename T, typename S, int OT, bool KS, typename Emit>
__device__ __forceinline__ void ttm_rows(const TtmJob& j, long long a0, int o0, T* Ml, T* Xl, Emit emit) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int c = lane & 15, kg = lane >> 4;
  const int B = (int)j.Bsz;
  constexpr int NC = KS ? 16 : 64, NL = KS ? 4 : 16;   // columns a block, values a thread stages
  const int TA = NC / B;
  const int ta = (int)min((long long)TA, j.A - a0);
  const int P = TTM_KS * B + 4;
  const int col = KS ? c : 16 * wv + c;
  const int cc = min(col, ta * B - 1);
  const int al = cc / B, bl = cc - al * B;
  const TX* X = static_cast<const TX*>(j.X);
  const TX* X0 = static_cast<const TX*>(j.X0);
  typename Acc<S>::v acc[OT][1];
#pragma unroll
  for (int t = 0; t < OT; ++t) acc[t][0] = (typename Acc<S>::v){0, 0, 0, 0};
  T buf[NL];
  const int row = j.Nin * B;                       // values of a slice
  auto load = [&](int k0) {
    const int kc = min(TTM_KS, (j.Nin - k0 + 15) & ~15), per = kc * B;
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int t = (int)threadIdx.x + 256 * q;
      const int s = t / per, e = t - s * per;
      T v = (T)0;
      if (s < ta && k0 * B + e < row) {
        const long long at = (a0 + s) * row + (long long)k0 * B + e;
        v = (T)X[at];
        if (X0) v -= (T)X0[at];
      }
      buf[q] = v;
    }
  };
  load(0);
  for (int k0 = 0; k0 < j.Nin; k0 += TTM_KS) {
    const int kc = min(TTM_KS, (j.Nin - k0 + 15) & ~15), per = kc * B;
    if (k0) __syncthreads();
    stage_m<T, OT>(j, k0, kc, o0, Ml);
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      const int t = (int)threadIdx.x + 256 * q;
      const int s = t / per;
      if (s < ta) Xl[s * P + (t - s * per)] = buf[q];
    }
    __syncthreads();
    if (k0 + TTM_KS < j.Nin) load(k0 + TTM_KS);
    const T* xp = Xl + al * P + bl;
    for (int k = KS ? 16 * wv : 0; k < kc; k += KS ? 64 : 16) {
      typename Acc<T>::v run[OT];
#pragma unroll
      for (int t = 0; t < OT; ++t) begin_run<T, S>(acc[t][0], run[t]);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const T d = xp[(k + 4 * s + kg) * B];
#pragma unroll
        for (int t = 0; t < OT; ++t)
          run[t] = Acc<T>::mma(Ml[((k >> 4) * (OT * 16) + 16 * t + c) * 16 + kg * 4 + s], d, run[t]);
      }
#pragma unroll
      for (int t = 0; t < OT; ++t) end_run<T, S>(run[t], acc[t][0]);
    }
  }
  const long long a = a0 + al;
  if constexpr (KS) {
    __syncthreads();
    ks_sum<T, S, OT, 1>(reinterpret_cast<S*>(Ml), acc, [&](int o, const S(&val)[1]) {
      if (col < ta * B && o0 + o < j.Nout) emit(a, o0 + o, (long long)bl, (a * j.Nout + o0 + o) * B + bl, val);
    });
    return;
  }
  if (col >= ta * B) return;
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = o0 + 16 * t + Acc<T>::row(kg, i);
      if (o < j.Nout) {
        S val[1] = {acc[t][0][i]};
        emit(a, o, (long long)bl, (a * j.Nout + o) * j.Bsz + bl, val);
      }
    }
}

// How a job is cut into blocks (host and device).
struct TtmCut {
  long long blocks;   // along the columns
  int oblocks;        // along the outputs
  int vec;            // columns a lane loads at a time (0: Bsz < 16)
  int ks;             // a block's waves split the contracted rows
};

struct TtmLaunch {
  int n;
  long long first;    // blocks of earlier launches of the same products
  long long start[TTM_JOBS + 1];
  TtmCut cut[TTM_JOBS];
  TtmJob j[TTM_JOBS];
};

constexpr int TTM_XBYTES(int elem) { return (64 * TTM_KS + 64 * 4 + 16) * elem; }

template <typename TX, typename T, typename TY, typename S, int OT>
__global__ void __launch_bounds__(256) k_ttm_mm(TtmLaunch g) {
  __shared__ __align__(16) unsigned char raw[TTM_MBYTES + TTM_XBYTES(sizeof(T))];
  T* Ml = reinterpret_cast<T*>(raw);
  T* Xl = reinterpret_cast<T*>(raw + TTM_MBYTES);
  const long long bid = g.first + blockIdx.x;
  int q = 0;
  while (q + 1 < g.n && bid >= g.start[q + 1]) ++q;
  const TtmJob& j = g.j[q];
  const TtmCut& cut = g.cut[q];
  const long long lb = bid - g.start[q];
  const long long cb = lb / cut.oblocks;
  const int o0 = (int)(lb - cb * cut.oblocks) * (OT * 16);
  constexpr int V = vec_of<TX>();
  TY* Y = static_cast<TY*>(j.Y);
  if (cut.vec == V) {
    typedef TY vy __attribute__((ext_vector_type(V)));
    auto put = [&](long long, int, long long, long long at, const S(&val)[V]) {
      vy v;
#pragma unroll
      for (int k = 0; k < V; ++k) v[k] = (TY)val[k];
      *reinterpret_cast<vy*>(Y + at) = v;
    };
    if constexpr (ks_fits<S, OT, V>())
      if (cut.ks) {
        ttm_cols<TX, T, S, V, 1, OT, true>(j, cb, o0, Ml, put);
        return;
      }
    ttm_cols<TX, T, S, V, 1, OT, false>(j, cb * 4, o0, Ml, put);
  } else {
    auto put = [&](long long, int, long long, long long at, const S(&val)[1]) { Y[at] = (TY)val[0]; };
    if (cut.vec == 1) {
      if (cut.ks) ttm_cols<TX, T, S, 1, 1, OT, true>(j, cb, o0, Ml, put);
      else ttm_cols<TX, T, S, 1, 2, OT, false>(j, cb * 4, o0, Ml, put);
    } else {
      if (cut.ks) ttm_rows<TX, T, S, OT, true>(j, cb * (16 / j.Bsz), o0, Ml, Xl, put);
      else ttm_rows<TX, T, S, OT, false>(j, cb * (64 / j.Bsz), o0, Ml, Xl, put);
    }
  }
}

// The last product of a reconstruction, compared with the snapshot instead of stored:
// the reconstruction never reaches memory, and the snapshot is read once.
template <typename TX, typename T, typename TV, int OT>
__global__ void __launch_bounds__(256) k_ttm_err(TtmLaunch g, TtmErr e) {
  __shared__ __align__(16) unsigned char raw[TTM_MBYTES + TTM_XBYTES(sizeof(T))];
  __shared__ double red[16];
  T* Ml = reinterpret_cast<T*>(raw);
  T* Xl = reinterpret_cast<T*>(raw + TTM_MBYTES);
  const TtmJob& j = g.j[0];
  const TtmCut& cut = g.cut[0];
  const long long bid = g.first + blockIdx.x;
  const long long cb = bid / cut.oblocks;
  const int o0 = (int)(bid - cb * cut.oblocks) * (OT * 16);
  constexpr int V = vec_of<TX>();
  const TV* S = static_cast<const TV*>(e.V);
  double se = 0.0, sv = 0.0;
  auto add = [&](double wr, long long b, TV x, T r) {
    const double w = wr * e.wb[b], v = (double)x, d = (double)((T)x - r);
    se += w * d * d;
    sv += w * v * v;
  };
  if (cut.vec == V) {
    typedef TV vv __attribute__((ext_vector_type(V)));
    ttm_cols<TX, T, T, V, 1, OT, false>(j, cb * 4, o0, Ml, [&](long long a, int o, long long b, long long at, const T(&val)[V]) {
      const double wr = e.wa[a] * e.wo[o];
      const vv x = *reinterpret_cast<const vv*>(S + at);
#pragma unroll
      for (int k = 0; k < V; ++k) add(wr, b + k, x[k], val[k]);
    });
  } else if (cut.vec == 1) {
    ttm_cols<TX, T, T, 1, 2, OT, false>(j, cb * 4, o0, Ml, [&](long long a, int o, long long b, long long at, const T(&val)[1]) {
      add(e.wa[a] * e.wo[o], b, S[at], val[0]);
    });
  } else {
    ttm_rows<TX, T, T, OT, false>(j, cb * (64 / j.Bsz), o0, Ml, Xl,
                        [&](long long a, int o, long long b, long long at, const T(&val)[1]) {
                          add(e.wa[a] * e.wo[o], b, S[at], val[0]);
                        });
  }
  se = block_sum(se, red);
  sv = block_sum(sv, red);
  if (threadIdx.x == 0) {
    e.partials[2 * bid] = se;
    e.partials[2 * bid + 1] = sv;
  }
}

// ---------------------------------------------------------------- launchers
// Tiles of 16 outputs a block holds: all of them up to 64.
static int tiles_of(int Nout) { return Nout <= 16 ? 1 : Nout <= 32 ? 2 : Nout <= 48 ? 3 : 4; }

// A grid holds fewer than 2^32 threads; outputs beyond that take several launches.
constexpr long long TTM_GRID = 1 << 23;
static unsigned grid_of(long long blocks) { return (unsigned)(blocks < TTM_GRID ? blocks : TTM_GRID); }

static bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Several columns a lane (one 16-byte load each) where the rows keep that alignment and
// enough waves remain (four per compute unit; below that, more waves of single columns
// were faster: they hide more latency). Y and Y2 (the snapshot of an error pass) are
// accessed V values at a time as well. ks: contractions of 64 rows and more take a block per
// unit, its waves splitting the rows. wide: with a quarter of the waves that the rule asks
// for, 16-byte loads of rows split over a block's waves replace single columns (as many
// blocks, four times the bytes a load: a 192^3 FP32 step at ranks 5 took 184 us, 191 with single
// columns, both with FP32 sums).
static TtmCut cut_of(const TtmJob& j, int OT, int V, size_t xb, size_t yb, const void* Y, bool ks, bool wide) {
  TtmCut c;
  c.oblocks = (j.Nout + OT * 16 - 1) / (OT * 16);
  c.ks = ks && j.Nin >= 64 ? 1 : 0;
  if (j.Bsz < 16) {
    const long long TA = (c.ks ? 16 : 64) / j.Bsz;
    c.vec = 0;
    c.blocks = (j.A + TA - 1) / TA;
    return c;
  }
  const bool al = j.Bsz % V == 0 && aligned(j.X, V * xb) && (!j.X0 || aligned(j.X0, V * xb)) && aligned(Y, V * yb);
  const long long uv = j.A * ((j.Bsz + 16 * V - 1) / (16 * V)) * c.oblocks;
  if (wide && al && !c.ks && uv < 1024 && uv >= 256 && j.Nin >= 64) {
    c.vec = V;
    c.ks = 1;
  } else {
    c.vec = al && uv >= 1024 && !c.ks ? V : 1;
  }
  const long long units = j.A * ((j.Bsz + 16 * c.vec - 1) / (16 * c.vec));
  c.blocks = c.ks ? units : (units + 3) / 4;
  return c;
}

static bool job_ok(const TtmJob& j) {
  return j.A >= 1 && j.Bsz >= 1 && j.Nin >= 1 && j.Nout >= 1 && j.X && j.M;
}

template <typename TX, typename T, typename TY, typename S, int OT>
static hipError_t launch_as(const TtmGroup& g, hipStream_t s) {
  TtmLaunch L{};
  // A launch that leaves compute units without a block splits its contractions: four times
  // the blocks, a quarter of the serial rows each (400 x 200 x 12 at ranks (12, 11, 3), 118
  // blocks: a step 209 -> 173 us). With a block for every unit it does not: each block
  // stages the matrix again (channel, 439 blocks of 48 outputs: 26 -> 50 us). Nor where the
  // caller asks for one chain an output (the core of the HOSVD: see wave_chol_inv).
  for (int ks = 0; ks < 2; ++ks) {
    L.n = 0;
    for (int q = 0; q < g.n; ++q) {
      if (tiles_of(g.j[q].Nout) != OT) continue;
      if (!job_ok(g.j[q]) || !g.j[q].Y) return hipErrorInvalidValue;
      const int n = L.n++;
      L.j[n] = g.j[q];
      L.cut[n] = cut_of(g.j[q], OT, vec_of<TX>(), sizeof(TX), sizeof(TY), g.j[q].Y, ks != 0,
                        !g.chain && ks_fits<S, OT, vec_of<TX>()>());
      L.start[n + 1] = L.start[n] + L.cut[n].blocks * L.cut[n].oblocks;
    }
    if (g.chain || L.start[L.n] >= 256) break;
  }
  if (!L.n) return hipSuccess;
  for (; L.first < L.start[L.n]; L.first += TTM_GRID)
    hipLaunchKernelGGL((k_ttm_mm<TX, T, TY, S, OT>), dim3(grid_of(L.start[L.n] - L.first)), dim3(256), 0, s, L);
  return hipGetLastError();
}

// One output a thread, its sum in order, eight rows' loads at a time: for expansions of a small
// core, where staging M and a wave's tiles cost more than they save. The same sums as
// k_ttm_mm's, bit for bit.
template <typename TX, typename T, typename TY>
__global__ void __launch_bounds__(256) k_ttm_each(TtmJob j, unsigned total) {
  const unsigned t = blockIdx.x * 256 + threadIdx.x;
  if (t >= total) return;
  const unsigned B = (unsigned)j.Bsz, ao = t / B, b = t - ao * B, a = ao / (unsigned)j.Nout, o = ao - a * (unsigned)j.Nout;
  const TX* x = static_cast<const TX*>(j.X) + (size_t)a * j.Nin * B + b;
  const double* m = j.M + (long long)o * j.ms_o;
  T acc = (T)0;
  int i = 0;
  for (; i + 8 <= j.Nin; i += 8) {
    TX xv[8];
    double mv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      xv[u] = x[(size_t)(i + u) * B];
      mv[u] = m[(i + u) * j.ms_i];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = fma((T)mv[u], (T)xv[u], acc);
  }
  for (; i < j.Nin; ++i) acc = fma((T)m[i * j.ms_i], (T)x[(size_t)i * B], acc);
  static_cast<TY*>(j.Y)[t] = (TY)acc;
}
// Up to 10 M multiply-adds: the whole decode of 512 x 500 at ranks 24 takes 13.2 us (16.7 in
// tiles), 50 x 48 x 50 x 4 at (20, 18, 16, 4), 10 M in its last product, 22.9 (28.4); above it
// 160^3 at 24, 15 M in its second product, 55.3 (51.4), 120 x 100 x 90 at 22, 24 M, 38.2 (26.8).
constexpr long long TTM_EACH = 10000000;
static bool each_ok(const TtmGroup& g) {
  if (g.n != 1) return false;
  const TtmJob& j = g.j[0];
  return !j.X0 && !j.mw && job_ok(j) && j.Y && j.Nin <= 64 && j.A * j.Nout * j.Bsz <= TTM_EACH / j.Nin;
}

template <typename TX, typename T, typename TY, typename S>
hipError_t launch_ttm_group(const TtmGroup& g, hipStream_t s) {
  if (g.n < 0 || g.n > TTM_JOBS) return hipErrorInvalidValue;
  if (each_ok(g)) {
    const unsigned total = (unsigned)(g.j[0].A * g.j[0].Nout * g.j[0].Bsz);
    hipLaunchKernelGGL((k_ttm_each<TX, T, TY>), dim3((total + 255) / 256), dim3(256), 0, s, g.j[0], total);
    return hipGetLastError();
  }
  hipError_t e = launch_as<TX, T, TY, S, 4>(g, s);
  if (e == hipSuccess) e = launch_as<TX, T, TY, S, 3>(g, s);
  if (e == hipSuccess) e = launch_as<TX, T, TY, S, 2>(g, s);
  if (e == hipSuccess) e = launch_as<TX, T, TY, S, 1>(g, s);
  return e;
}
template hipError_t launch_ttm_group<float, float, float>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<double, float, float>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<float, float, double>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<float, double, float>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<float, float, float, double>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<double, float, float, double>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<float, double, double>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<double, double, double>(const TtmGroup&, hipStream_t);
template hipError_t launch_ttm_group<double, double, float>(const TtmGroup&, hipStream_t);

long long ttm_err_blocks(long long A, int Nout, long long Bsz) {
  const long long ob = (Nout + 15) / 16;
  if (Bsz < 16) return (A + 64 / Bsz - 1) / (64 / Bsz) * ob;
  return (A * ((Bsz + 15) / 16) + 3) / 4 * ob;
}

template <typename TX, typename T, typename TV>
hipError_t launch_ttm_err(const TtmJob& j, const TtmErr& e, int* blocks, hipStream_t s) {
  if (!job_ok(j) || !e.V || !e.partials) return hipErrorInvalidValue;
  const int OT = tiles_of(j.Nout);
  TtmLaunch L{};
  L.n = 1;
  L.j[0] = j;
  L.cut[0] = cut_of(j, OT, vec_of<TX>(), sizeof(TX), sizeof(TV), e.V, false, false);
  const long long nb = L.cut[0].blocks * L.cut[0].oblocks;
  if (nb > 0x7fffffffLL) return hipErrorInvalidValue;
  *blocks = (int)nb;
  for (; L.first < nb; L.first += TTM_GRID) {
    const dim3 grid(grid_of(nb - L.first)), blk(256);
    switch (OT) {
      case 1: hipLaunchKernelGGL((k_ttm_err<TX, T, TV, 1>), grid, blk, 0, s, L, e); break;
      case 2: hipLaunchKernelGGL((k_ttm_err<TX, T, TV, 2>), grid, blk, 0, s, L, e); break;
      case 3: hipLaunchKernelGGL((k_ttm_err<TX, T, TV, 3>), grid, blk, 0, s, L, e); break;
      default: hipLaunchKernelGGL((k_ttm_err<TX, T, TV, 4>), grid, blk, 0, s, L, e); break;
    }
  }
  return hipGetLastError();
}
template hipError_t launch_ttm_err<float, float, float>(const TtmJob&, const TtmErr&, int*, hipStream_t);
template hipError_t launch_ttm_err<float, float, double>(const TtmJob&, const TtmErr&, int*, hipStream_t);
template hipError_t launch_ttm_err<double, double, float>(const TtmJob&, const TtmErr&, int*, hipStream_t);
template hipError_t launch_ttm_err<double, double, double>(const TtmJob&, const TtmErr&, int*, hipStream_t);

// ---------------------------------------------------------------- third-order expansion
// A block takes 64 columns of the mode-1 unfolding (a run of (i2, i3)) and `rows` rows. It
// forms T3 = C x_3 U_3 for the i3 it meets and E = T3 x_2 U_2 for its columns in LDS (the
// same in every row block: a few hundred multiply-adds a thread), then the rows as a
// matrix product with U_1, four consecutive columns a lane. One launch instead of one a
// mode: bound by the launch and by the stores, where the chain of three products took
// about 24 us for a 256 x 256 x 4 FP32 field at ranks (17, 17, 4), 8.7 now.
constexpr int R3C = 64;

struct Rec3Lds {
  int nd, n2, r1p;              // distinct i3, rows of U_2, r1 rounded up to 4
  int oC, oU3, oU2, oT, oE, oU1, total;   // offsets and size in values of T
};
__host__ __device__ inline Rec3Lds rec3_lds(const Rec3Args& a) {
  Rec3Lds L;
  L.nd = (int)(a.N[2] < R3C ? a.N[2] : R3C);
  L.n2 = (int)((R3C + a.N[2] - 2) / a.N[2]) + 1;
  L.r1p = (a.r[0] + 3) & ~3;
  L.oC = 0;
  L.oU3 = L.oC + a.r[0] * a.r[1] * a.r[2];
  L.oU2 = L.oU3 + L.nd * a.r[2];
  L.oT = L.oU2 + L.n2 * a.r[1];
  L.oE = (L.oT + a.r[0] * a.r[1] * L.nd + 3) & ~3;
  L.oU1 = L.oE + L.r1p * R3C;
  L.total = L.oU1 + 64 * (L.r1p + 1);
  return L;
}

// NL: loads of the core and of U_1 a thread issues at once (2 for mode-1 ranks up to 8).
template <typename T, typename TY, int NL>
__global__ void __launch_bounds__(256) k_rec3(Rec3Args a) {
  extern __shared__ __align__(16) unsigned char raw_r[];
  T* lds = reinterpret_cast<T*>(raw_r);
  const Rec3Lds L = rec3_lds(a);
  T *Cl = lds + L.oC, *U3l = lds + L.oU3, *U2l = lds + L.oU2, *Tl = lds + L.oT, *El = lds + L.oE, *U1l = lds + L.oU1;
  const int r1 = a.r[0], r2 = a.r[1], r3 = a.r[2], tid = threadIdx.x;
  const int N3 = (int)a.N[2];
  const long long M = a.N[1] * a.N[2], col0 = (long long)blockIdx.x * R3C;
  const int i20 = (int)(col0 / N3), i30 = (int)(col0 - (long long)i20 * N3);
  const bool wide = N3 >= R3C;
  const long long row0 = (long long)blockIdx.y * a.rows;
  const int nrows = (int)min((long long)a.rows, a.N[0] - row0);
  // Every factor's loads before any store, NC, NU and so on of them a thread (a loop over
  // loads and stores would wait for each load), then what is left over.
  constexpr int NC = NL, NU1 = NL, NU2 = 1, NU3 = 2;
  const int nC = r1 * r2 * r3, nU3 = L.nd * r3, nU2 = L.n2 * r2, nU1 = 64 * L.r1p;
  const float f1 = 1.0f / (float)L.r1p, f2 = 1.0f / (float)r2, f3 = 1.0f / (float)r3, fd = 1.0f / (float)L.nd;
  auto gC = [&](int t) { return a.C[min(t, nC - 1)]; };
  auto gU3 = [&](int t) {
    t = min(t, nU3 - 1);
    const int d = small_div(t, r3, f3), c = t - d * r3;
    int i3 = wide ? i30 + d : d;   // (d < 64 <= N3 when wide)
    i3 -= i3 >= N3 ? N3 : 0;
    return a.U[2][(long long)i3 * a.ldU[2] + c];
  };
  auto gU2 = [&](int t) {
    t = min(t, nU2 - 1);
    const int q = small_div(t, r2, f2), b = t - q * r2;
    return a.U[1][min((long long)i20 + q, a.N[1] - 1) * a.ldU[1] + b];
  };
  int c0 = 0;
  auto gU1 = [&](int t) {         // rows c0 .. c0 + 63 of the block, zero past r1
    t = min(t, nU1 - 1);
    const int q = small_div(t, L.r1p, f1), k = t - q * L.r1p;
    const double x = a.U[0][(row0 + min(c0 + q, nrows - 1)) * a.ldU[0] + min(k, r1 - 1)];
    return k < r1 ? x : 0.0;
  };
  auto sU1 = [&](int t, double x) {
    if (t < nU1) U1l[t + small_div(t, L.r1p, f1)] = (T)x;   // row stride r1p + 1
  };
  {
    double vC[NC], v1[NU1], v2[NU2], v3[NU3];
#pragma unroll
    for (int u = 0; u < NC; ++u) vC[u] = gC(tid + 256 * u);
#pragma unroll
    for (int u = 0; u < NU3; ++u) v3[u] = gU3(tid + 256 * u);
#pragma unroll
    for (int u = 0; u < NU2; ++u) v2[u] = gU2(tid + 256 * u);
#pragma unroll
    for (int u = 0; u < NU1; ++u) v1[u] = gU1(tid + 256 * u);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NC; ++u)
      if (tid + 256 * u < nC) Cl[tid + 256 * u] = (T)vC[u];
#pragma unroll
    for (int u = 0; u < NU3; ++u)
      if (tid + 256 * u < nU3) U3l[tid + 256 * u] = (T)v3[u];
#pragma unroll
    for (int u = 0; u < NU2; ++u)
      if (tid + 256 * u < nU2) U2l[tid + 256 * u] = (T)v2[u];
#pragma unroll
    for (int u = 0; u < NU1; ++u) sU1(tid + 256 * u, v1[u]);
    for (int t = tid + 256 * NC; t < nC; t += 256) Cl[t] = (T)gC(t);
    for (int t = tid + 256 * NU3; t < nU3; t += 256) U3l[t] = (T)gU3(t);
    for (int t = tid + 256 * NU2; t < nU2; t += 256) U2l[t] = (T)gU2(t);
    for (int t = tid + 256 * NU1; t < nU1; t += 256) sU1(t, gU1(t));
  }
  __syncthreads();
  for (int t = tid; t < r1 * r2 * L.nd; t += 256) {
    const int ab = small_div(t, L.nd, fd), d = t - ab * L.nd;
    T s = (T)0;
#pragma unroll 4
    for (int c = 0; c < r3; ++c) s += Cl[ab * r3 + c] * U3l[d * r3 + c];
    Tl[t] = s;
  }
  __syncthreads();
  {
    // a thread keeps its column
    const int q = tid & 63, i2 = (i30 + q) / N3, d = wide ? q : (i30 + q) % N3;
    for (int x = tid >> 6; x < L.r1p; x += 4) {
      T s = (T)0;
      if (x < r1)
#pragma unroll 8
        for (int b = 0; b < r2; ++b) s += Tl[(x * r2 + b) * L.nd + d] * U2l[i2 * r2 + b];
      El[x * R3C + q] = s;
    }
  }
  const int lane = tid & 63, wv = tid >> 6, c = lane & 15, kg = lane >> 4;
  typedef T tv __attribute__((ext_vector_type(4)));
  typedef TY yv __attribute__((ext_vector_type(4)));
  const long long col = col0 + 4 * c;
  for (; c0 < nrows; c0 += 64) {
    if (c0) {
      __syncthreads();
      double v1[NU1];
#pragma unroll
      for (int u = 0; u < NU1; ++u) v1[u] = gU1(tid + 256 * u);
#pragma unroll
      for (int u = 0; u < NU1; ++u) sU1(tid + 256 * u, v1[u]);
      for (int t = tid + 256 * NU1; t < nU1; t += 256) sU1(t, gU1(t));
    }
    __syncthreads();
    typename Acc<T>::v acc[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = (typename Acc<T>::v){0, 0, 0, 0};
    const T* ur = U1l + (16 * wv + c) * (L.r1p + 1) + kg;
#pragma unroll 4
    for (int k = 0; k < L.r1p; k += 4) {
      const T m = ur[k];
      const tv e = *reinterpret_cast<const tv*>(El + (k + kg) * R3C + 4 * c);
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = Acc<T>::mma(m, e[v], acc[v]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int rl = c0 + 16 * wv + Acc<T>::row(kg, i);
      if (rl >= nrows) continue;
      TY* o = static_cast<TY*>(a.out) + (row0 + rl) * M + col;
      if (a.vec) {
        if (col < M) *reinterpret_cast<yv*>(o) = (yv){(TY)acc[0][i], (TY)acc[1][i], (TY)acc[2][i], (TY)acc[3][i]};
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (col + v < M) o[v] = (TY)acc[v][i];
      }
    }
  }
}

// Up to 64 KB of factors, so that two blocks share a compute unit (and the launch needs no
// attribute set).
template <typename T>
bool rec3_ok(const Rec3Args& a) {
  const long long big = (long long)a.r[0] * a.r[1] * (a.r[2] + R3C);
  // (the grid: fewer than 2^32 threads along the columns, 65 535 row blocks)
  return big < (1 << 20) && a.N[1] * a.N[2] < 64 * TTM_GRID && a.N[0] <= 64 * 65535LL && (size_t)rec3_lds(a).total * sizeof(T) <= 65536;
}
template bool rec3_ok<float>(const Rec3Args&);
template bool rec3_ok<double>(const Rec3Args&);

template <typename T, typename TY>
hipError_t launch_rec3(const Rec3Args& a0, hipStream_t s) {
  Rec3Args a = a0;
  const long long M = a.N[1] * a.N[2], cols = (M + R3C - 1) / R3C;
  a.vec = M % 4 == 0 && aligned(a.out, 4 * sizeof(TY));
  // longer row blocks (less of the common part repeated) once the grid has four blocks for
  // each compute unit
  a.rows = 64;
  while (a.rows < 512 && cols * ((a.N[0] + 2 * a.rows - 1) / (2 * a.rows)) >= 1024) a.rows *= 2;
  const size_t lds = (size_t)rec3_lds(a).total * sizeof(T);
  const dim3 grid((unsigned)cols, (unsigned)((a.N[0] + a.rows - 1) / a.rows));
  // loads a thread of the core and of 64 rows of the first basis
  const Rec3Lds L = rec3_lds(a);
  const int need = std::max((a.r[0] * a.r[1] * a.r[2] + 255) / 256, (64 * L.r1p + 255) / 256);
  if (need <= 2) {
    hipLaunchKernelGGL((k_rec3<T, TY, 2>), grid, dim3(256), lds, s, a);
  } else if (need <= 4) {
    hipLaunchKernelGGL((k_rec3<T, TY, 4>), grid, dim3(256), lds, s, a);
  } else {
    hipLaunchKernelGGL((k_rec3<T, TY, 8>), grid, dim3(256), lds, s, a);
  }
  return hipGetLastError();
}
template hipError_t launch_rec3<float, float>(const Rec3Args&, hipStream_t);
template hipError_t launch_rec3<float, double>(const Rec3Args&, hipStream_t);
template hipError_t launch_rec3<double, float>(const Rec3Args&, hipStream_t);
template hipError_t launch_rec3<double, double>(const Rec3Args&, hipStream_t);

}  // namespace tdb
