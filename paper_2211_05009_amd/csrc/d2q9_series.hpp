// d2q9_series.hpp -- flow state of probe time series (the stable / periodic /
// aperiodic states of Sec. 3.3 and the periods of Table 3).
//
// Definition (the library documents it with lbm_classify_series):
//   amplitude A = max - min; steady if A <= steady_tol;
//   D(T) = mean_{k < n-T} (u[k+T] - u[k])^2 / sigma^2 for T in
//   [min_lag, max_lag]; candidates are interior local minima of D reached
//   after D exceeded 1; the parabola through D at T-1, T, T+1 refines the
//   period (vertex) and gives the mismatch sqrt(max(vertex value, 0));
//   periodic at the first candidate with mismatch <= periodic_tol; a drift
//   if there is no candidate; aperiodic otherwise.
//
// Three launches: k_series_stats (a block per series: the series laid out
// densely, its mean, deviation and range), k_series_lags (a block per series
// and tile of lags: D), k_series_pick (a block per series: the candidates).
// Every D(T) is one sequential sum over k, and the other sums run in a fixed
// order (per-thread sequential sums, then a fixed LDS tree), so the result
// depends neither on scheduling nor on how the lags are tiled.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

namespace lbm {

constexpr int kSeriesThreads = 256;

// Sample k of a series lives at base[((start + k) % cap) * stride]: a ring
// of records (cap = n, start = 0 for a plain strided array).
struct SeriesDesc {
  const double *base;
  long long cap, start, n, stride;
};

// Work memory of one series, series_work_doubles(n) doubles: the n samples,
// the D values of lags min_lag .. max_lag (at most n - 2 of them), and in the
// last eight what k_series_stats found.
__host__ __device__ constexpr long long series_work_doubles(long long n) { return 2 * n + 8; }
enum { kStatMean, kStatStd, kStatAmp, kStatInvVar, kStatActive };
__device__ __forceinline__ double *series_stats(double *work, long long n) { return work + 2 * n; }

// Last lag of a series of n samples.
__host__ __device__ __forceinline__ long long series_max_lag(long long n, int max_lag_req) {
  const long long m = max_lag_req > 0 ? max_lag_req : n / 3;
  return m < n - 2 ? m : n - 2;
}

// Fixed-order block sum / min / max of one value per thread.
__device__ __forceinline__ void series_reduce(double &sum, double &mn, double &mx, double *s0,
                                              double *s1, double *s2) {
  const int t = threadIdx.x;
  s0[t] = sum;
  s1[t] = mn;
  s2[t] = mx;
  __syncthreads();
  for (int h = kSeriesThreads / 2; h > 0; h >>= 1) {
    if (t < h) {
      s0[t] += s0[t + h];
      s1[t] = fmin(s1[t], s1[t + h]);
      s2[t] = fmax(s2[t], s2[t + h]);
    }
    __syncthreads();
  }
  sum = s0[0];
  mn = s1[0];
  mx = s2[0];
  __syncthreads();
}

// The source of series s: a descriptor each, or rows of a plain array.
struct SeriesFromDesc {
  const SeriesDesc *desc;
  __device__ __forceinline__ SeriesDesc operator()(int s) const { return desc[s]; }
};
struct SeriesFromRows {
  const double *base;
  long long ld, n;
  __device__ __forceinline__ SeriesDesc operator()(int s) const {
    return SeriesDesc{base + s * ld, n, 0, n, 1};
  }
};

// Samples into work (dense), then mean, population deviation and range.
// Eight loads in flight per thread: a thread's samples are 256 apart, and
// one load at a time left the block waiting on each.
template <typename Src>
__global__ __launch_bounds__(kSeriesThreads) void k_series_stats(
    Src src, long long n, double steady_tol, double *__restrict__ work, long long work_stride) {
  __shared__ double s0[kSeriesThreads], s1[kSeriesThreads], s2[kSeriesThreads];
  const SeriesDesc d = src(blockIdx.x);
  double *u = work + (long long)blockIdx.x * work_stride;
  double sum = 0.0, mn = INFINITY, mx = -INFINITY;
#pragma unroll 8
  for (long long k = threadIdx.x; k < n; k += kSeriesThreads) {
    long long r = d.start + k;           // start < cap, k < n <= cap
    if (r >= d.cap) r -= d.cap;
    const double v = d.base[r * d.stride];
    u[k] = v;
    sum += v;
    mn = fmin(mn, v);
    mx = fmax(mx, v);
  }
  series_reduce(sum, mn, mx, s0, s1, s2);
  const double mean = sum / (double)n;
  // variance about the mean (two passes, like the population std); each
  // thread reads back its own samples
  double ss = 0.0, dummy0 = 0.0, dummy1 = 0.0;
  const double *v = u;
#pragma unroll 8
  for (long long k = threadIdx.x; k < n; k += kSeriesThreads) {
    const double e = v[k] - mean;
    ss += e * e;
  }
  series_reduce(ss, dummy0, dummy1, s0, s1, s2);
  if (threadIdx.x == 0) {
    const double sd = sqrt(ss / (double)n), amp = mx - mn;
    double *st = series_stats(u, n);
    st[kStatMean] = mean;
    st[kStatStd] = sd;
    st[kStatAmp] = amp;
    st[kStatInvVar] = 1.0 / (sd * sd);
    st[kStatActive] = amp <= steady_tol ? 0.0 : 1.0;
  }
}

// D of lags min_lag + [tile NT L, (tile + 1) NT L) of one series.  A lane
// owns L consecutive lags and slides their L samples u[k + T] through
// registers, so a step of k costs one LDS read of its own and a broadcast of
// u[k] for 2 L FP64 operations; L = 3 keeps the lanes' stride odd (no bank
// conflicts), L = 1 makes three times the wavefronts for small problems
// (series_lags_wide).  The samples come through LDS in chunks of C values
// of k, summed in unrolled groups of U; the last groups of a wavefront, where
// its longer lags run past the end of the series, add zeros for those.
// Bound by LDS reads and the FP64 vector rate together (each sum is one
// dependent chain): 153 series of 10,000 samples, 3333 lags each, in 458 us
// = 28 FP64 TFLOP/s counting subtract, multiply and add; one thread per
// chain of 13 lags, a block per series, took 10.3 ms.  u[k] from a register
// by lane reads instead of the LDS broadcast: 530 us; by scalar loads: 514.
template <int L, int NT, int C, int U>
__global__ __launch_bounds__(NT) void k_series_lags(double *__restrict__ work,
                                                    long long work_stride, long long n,
                                                    int nseries, int min_lag, long long nlags) {
  constexpr int W = NT * L;
  static_assert(C % U == 0 && U % L == 0, "whole groups");
  __shared__ double ua[C], ub[C + W + L];
  const int s = blockIdx.x % nseries;
  const long long tile = blockIdx.x / nseries;
  double *u = work + s * work_stride;
  const double *st = series_stats(u, n);
  if (st[kStatActive] == 0.0) return;      // steady: no lags (the whole block)
  const long long T0 = min_lag + tile * W;              // the block's first lag
  const int own = threadIdx.x * L;                      // the lane's first lag - T0
  // its wavefront's first lag - T0
  const int wave_lo = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63) * L;
  const int wave_hi = wave_lo + 64 * L - 1;             // and its last
  const bool live = tile * W + wave_lo < nlags;         // the wavefront has lags
  double acc[L];
#pragma unroll
  for (int l = 0; l < L; ++l) acc[l] = 0.0;
  for (long long k0 = 0; k0 + T0 < n; k0 += C) {
    __syncthreads();
#pragma unroll
    for (int i = threadIdx.x; i < C; i += NT) ua[i] = k0 + i < n ? u[k0 + i] : 0.0;
#pragma unroll
    for (int i = threadIdx.x; i < C + W; i += NT)
      ub[i] = k0 + T0 + i < n ? u[k0 + T0 + i] : 0.0;
    __syncthreads();
    if (!live) continue;
    // k0 + i + T < n for every lag of the wavefront below `full`, for none from `last` on
    const long long room = n - (k0 + T0);
    const int full = (int)min((long long)C, max(0LL, room - wave_hi));
    const int last = (int)min((long long)C, max(0LL, room - wave_lo));
    const int mine = (int)min((long long)C + W, room) - own;   // i + l < mine: inside
    double w[L];
#pragma unroll
    for (int l = 0; l < L; ++l) w[l] = ub[own + l];
    int i = 0;
    for (; i + U <= full; i += U) {
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const double a = ua[i + j];
#pragma unroll
        for (int l = 0; l < L; ++l) {
          const double e = w[(j + l) % L] - a;
          acc[l] += e * e;
        }
        w[j % L] = ub[own + i + j + L];
      }
    }
    for (; i < last; i += U) {
#pragma unroll
      for (int j = 0; j < U; ++j) {
        const double a = ua[i + j];
#pragma unroll
        for (int l = 0; l < L; ++l) {
          const double d = w[(j + l) % L] - a;
          const double e = i + j + l < mine ? d : 0.0;
          acc[l] += e * e;
        }
        w[j % L] = ub[own + i + j + L];
      }
    }
  }
  double *D = u + n;
  const double inv_var = st[kStatInvVar];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const long long j = tile * W + own + l;
    if (j < nlags) D[j] = acc[l] / (double)(n - (min_lag + j)) * inv_var;
  }
}

// The parabola through D at lags j - 1, j, j + 1: vertex lag and mismatch.
__device__ __forceinline__ double series_vertex(const double *D, long long j, int min_lag,
                                                double &period) {
  const double curv = D[j - 1] - 2.0 * D[j] + D[j + 1];
  period = (double)(min_lag + j);
  double vertex = D[j];
  if (curv > 0.0) {
    period += 0.5 * (D[j - 1] - D[j + 1]) / curv;
    vertex = D[j] - (D[j - 1] - D[j + 1]) * (D[j - 1] - D[j + 1]) / (8.0 * curv);
  }
  return sqrt(fmax(vertex, 0.0));
}

// Fixed-order block minimum of an index.
__device__ __forceinline__ long long series_min(long long v, long long *sm) {
  const int t = threadIdx.x;
  sm[t] = v;
  __syncthreads();
  for (int h = kSeriesThreads / 2; h > 0; h >>= 1) {
    if (t < h) sm[t] = min(sm[t], sm[t + h]);
    __syncthreads();
  }
  v = sm[0];
  __syncthreads();
  return v;
}

// The state of one series from its D values, in the ABI's record layout
// (OutRec: the fields of lbm_flow_state_t).  The threads look at lags in
// parallel: the first D above 1, then the first candidate (the dominant
// cycle), the first periodic one, and the smallest mismatch of all; a walk
// through the lags by one thread waited on one load of D after another.
template <typename OutRec>
__global__ __launch_bounds__(kSeriesThreads) void k_series_pick(
    const double *__restrict__ work, long long work_stride, long long n, int min_lag,
    long long nlags, double periodic_tol, OutRec *__restrict__ out) {
  __shared__ long long sm[kSeriesThreads];
  __shared__ double s0[kSeriesThreads], s1[kSeriesThreads], s2[kSeriesThreads];
  const double *u = work + (long long)blockIdx.x * work_stride;
  const double *st = u + 2 * n, *D = u + n;
  OutRec r;
  r.state = 0;
  r.lag = 0;
  r.period = 0.0;
  r.amplitude = st[kStatAmp];
  r.mean = st[kStatMean];
  r.std = st[kStatStd];
  r.mismatch = 0.0;
  r.cycle = 0.0;
  r.cycle_mismatch = 0.0;
  if (st[kStatActive] != 0.0) {
    const long long none = nlags;
    long long first = none;              // the first lag with D above 1
    for (long long j = threadIdx.x; j < nlags && first == none; j += kSeriesThreads)
      if (D[j] > 1.0) first = j;
    first = series_min(first, sm);
    long long cyc = none, per = none;
    double best = INFINITY, dummy0 = 0.0, dummy1 = 0.0, p;
    for (long long j = 1 + threadIdx.x; j + 1 < nlags; j += kSeriesThreads) {
      if (!(j > first && D[j - 1] > D[j] && D[j] <= D[j + 1])) continue;
      const double mis = series_vertex(D, j, min_lag, p);
      cyc = min(cyc, j);
      best = fmin(best, mis);
      if (mis <= periodic_tol) per = min(per, j);
    }
    cyc = series_min(cyc, sm);
    per = series_min(per, sm);
    series_reduce(dummy0, best, dummy1, s0, s1, s2);
    r.state = per != none ? 1 : cyc != none ? 2 : 3;
    if (cyc != none)
      r.cycle_mismatch = series_vertex(D, cyc, min_lag, r.cycle);
    else
      r.cycle_mismatch = INFINITY;       // no return within the window: a drift
    if (per != none) {
      r.lag = (int)(min_lag + per);
      r.mismatch = series_vertex(D, per, min_lag, r.period);
    } else {
      r.mismatch = best;
    }
  }
  if (threadIdx.x == 0) out[blockIdx.x] = r;
}

}  // namespace lbm
