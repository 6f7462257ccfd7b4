// lbm_series.hip -- flow-state classification of time series on the device
// (d2q9_series.hpp): lbm_classify_series and the shared launcher used by
// the probe-series entry points.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "../../include/lbm.h"
#include "d2q9_series.hpp"
#include "lbm_internal.h"

using namespace lbm;

namespace {

// Threads and chunk of k_series_lags' two forms.
constexpr int kWideThreads = 256, kWideChunk = 960, kWideUnroll = 24;
constexpr int kNarrowThreads = 64, kNarrowChunk = 512, kNarrowUnroll = 16;

// Whether the lags take three lags per lane.  One lag per lane gives three
// times the wavefronts but two LDS reads per sample and lag: it is faster
// until its wavefronts fill the GPU's 1024 SIMDs about three deep.  Narrow
// against wide, whole call: 1 x 10,000 samples (53 narrow wavefronts) 153 /
// 341 us, 97 x 4000 (2037) 122 / 158, 153 x 3000 (2448) 106 / 119, 153 x
// 10,000 (8109) 837 / 451.
bool series_lags_wide(int nseries, long long nlags) {
  return (long long)nseries * ((nlags + 63) / 64) > 3072;
}

// Issue the classification of nseries series of n samples from src on st:
// work holds work_stride doubles per series, out nseries records (device).
template <typename Src>
hipError_t launch_classify(const Src &src, int nseries, long long n, double steady_tol,
                           double periodic_tol, int min_lag, int max_lag, double *work,
                           long long work_stride, lbm_flow_state_t *out, hipStream_t st) {
  const long long nlags = series_max_lag(n, max_lag) - min_lag + 1;
  hipLaunchKernelGGL(k_series_stats<Src>, dim3(nseries), dim3(kSeriesThreads), 0, st, src, n,
                     steady_tol, work, work_stride);
  if (series_lags_wide(nseries, nlags)) {
    constexpr int W = 3 * kWideThreads;
    hipLaunchKernelGGL((k_series_lags<3, kWideThreads, kWideChunk, kWideUnroll>),
                       dim3((unsigned)(nseries * ((nlags + W - 1) / W))), dim3(kWideThreads), 0,
                       st, work, work_stride, n, nseries, min_lag, nlags);
  } else {
    constexpr int W = kNarrowThreads;
    hipLaunchKernelGGL((k_series_lags<1, kNarrowThreads, kNarrowChunk, kNarrowUnroll>),
                       dim3((unsigned)(nseries * ((nlags + W - 1) / W))), dim3(kNarrowThreads),
                       0, st, work, work_stride, n, nseries, min_lag, nlags);
  }
  hipLaunchKernelGGL(k_series_pick<lbm_flow_state_t>, dim3(nseries), dim3(kSeriesThreads), 0, st,
                     work, work_stride, n, min_lag, nlags, periodic_tol, out);
  return hipGetLastError();
}

// Classify into out_host with device scratch of this call: one allocation
// holding the records, the descriptors (descs_host, may be null) and the
// work memory.
template <typename MakeSrc>
int classify_alloc(const MakeSrc &make_src, const SeriesDesc *descs_host, int nseries,
                   long long n, double steady_tol, double periodic_tol, int min_lag, int max_lag,
                   hipStream_t st, lbm_flow_state_t *out_host) {
  const long long stride = series_work_doubles(n);
  const size_t out_bytes = (sizeof(lbm_flow_state_t) * nseries + 255) / 256 * 256;
  const size_t desc_bytes = descs_host ? (sizeof(SeriesDesc) * nseries + 255) / 256 * 256 : 0;
  char *mem = nullptr;
  hipError_t e = hipMalloc(&mem, out_bytes + desc_bytes + sizeof(double) * stride * nseries);
  if (e != hipSuccess)
    return lbm_fail(e == hipErrorOutOfMemory ? LBM_ENOMEM : LBM_EDEVICE, "classify: %s",
                    hipGetErrorString(e));
  lbm_flow_state_t *d_out = reinterpret_cast<lbm_flow_state_t *>(mem);
  SeriesDesc *d_desc = reinterpret_cast<SeriesDesc *>(mem + out_bytes);
  double *d_work = reinterpret_cast<double *>(mem + out_bytes + desc_bytes);
  if (descs_host)
    e = hipMemcpyAsync(d_desc, descs_host, sizeof(SeriesDesc) * nseries, hipMemcpyHostToDevice,
                       st);
  if (e == hipSuccess)
    e = launch_classify(make_src(d_desc), nseries, n, steady_tol, periodic_tol, min_lag, max_lag,
                        d_work, stride, d_out, st);
  if (e == hipSuccess)
    e = hipMemcpyAsync(out_host, d_out, sizeof(lbm_flow_state_t) * nseries,
                       hipMemcpyDeviceToHost, st);
  const hipError_t es = hipStreamSynchronize(st);
  if (e == hipSuccess) e = es;
  (void)hipFree(mem);
  if (e != hipSuccess)
    return lbm_fail(e == hipErrorOutOfMemory ? LBM_ENOMEM : LBM_EDEVICE, "classify: %s",
                    hipGetErrorString(e));
  return LBM_OK;
}

}  // namespace

int classify_series_descs(const SeriesDesc *descs_host, int nseries, long long n,
                          double steady_tol, double periodic_tol, int min_lag, int max_lag,
                          hipStream_t st, lbm_flow_state_t *out_host) {
  if (nseries <= 0) return LBM_OK;
  return classify_alloc([](const SeriesDesc *d) { return SeriesFromDesc{d}; }, descs_host,
                        nseries, n, steady_tol, periodic_tol, min_lag, max_lag, st, out_host);
}

// Lag range check shared by the entry points.
int check_lags(long long n, int min_lag, int max_lag) {
  if (n < 8) return lbm_fail(LBM_EINVAL, "n = %lld < 8 samples", n);
  if (min_lag < 1) return lbm_fail(LBM_EINVAL, "min_lag = %d < 1", min_lag);
  long long hi = max_lag > 0 ? max_lag : n / 3;
  hi = std::min(hi, n - 2);
  if (hi - min_lag + 1 < 3)
    return lbm_fail(LBM_EINVAL, "lag range [%d, %lld] holds fewer than 3 lags", min_lag, hi);
  return LBM_OK;
}

int lbm_classify_series(const double *series_dev, int nseries, int64_t n, int64_t ld,
                        double steady_tol, double periodic_tol, int min_lag, int max_lag,
                        lbm_flow_state_t *out_host, void *hip_stream) {
  if (!series_dev || !out_host) return lbm_fail(LBM_EINVAL, "NULL argument");
  if (nseries < 1) return lbm_fail(LBM_EINVAL, "nseries = %d < 1", nseries);
  if (ld < n) return lbm_fail(LBM_EINVAL, "ld = %lld < n = %lld", (long long)ld, (long long)n);
  if (!(steady_tol >= 0.0) || !(periodic_tol >= 0.0))
    return lbm_fail(LBM_EINVAL, "tolerances must be >= 0 (steady %g, periodic %g)", steady_tol,
                    periodic_tol);
  int rc = check_lags(n, min_lag, max_lag);
  if (rc) return rc;
  return classify_alloc(
      [=](const SeriesDesc *) { return SeriesFromRows{series_dev, (long long)ld, (long long)n}; },
      nullptr, nseries, n, steady_tol, periodic_tol, min_lag, max_lag, (hipStream_t)hip_stream,
      out_host);
}

// ------------------------------------------------ no-allocation classifier
// Work memory of lbm_classify_series_noalloc: one array per device, held
// from the library's load until the process ends.  Host code never uses the
// name `scratch` as an address (in host code it is a stand-in, not device
// memory): each device's address comes from hipGetSymbolAddress, taken once
// per device on that entry point's first call there.
constexpr long long kNoAllocScratchDoubles = 4LL << 20;   // 32 MiB
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static double *g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch array (nullptr and an
// error message on failure).
static double *scratch_for_current_device(int &rc) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    rc = lbm_fail(LBM_EDEVICE, "hipGetDevice: %s", hipGetErrorString(e));
    return nullptr;
  }
  if (dev < 0 || dev >= kMaxDevices) {
    rc = lbm_fail(LBM_EDEVICE, "device %d beyond the %d this entry point supports", dev,
                  kMaxDevices);
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      rc = lbm_fail(LBM_EDEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                    hipGetErrorString(e));
      return nullptr;
    }
    g_scratch_ptr[dev] = static_cast<double *>(p);
  }
  rc = LBM_OK;
  return g_scratch_ptr[dev];
}

int lbm_classify_series_noalloc(const double *series_dev, int nseries, int64_t n, int64_t ld,
                                double steady_tol, double periodic_tol, int min_lag,
                                int max_lag, lbm_flow_state_t *out_dev, void *hip_stream) {
  if (!series_dev || !out_dev) return lbm_fail(LBM_EINVAL, "NULL argument");
  if (nseries < 1) return lbm_fail(LBM_EINVAL, "nseries = %d < 1", nseries);
  if (ld < n) return lbm_fail(LBM_EINVAL, "ld = %lld < n = %lld", (long long)ld, (long long)n);
  if (!(steady_tol >= 0.0) || !(periodic_tol >= 0.0))
    return lbm_fail(LBM_EINVAL, "tolerances must be >= 0 (steady %g, periodic %g)", steady_tol,
                    periodic_tol);
  int rc = check_lags(n, min_lag, max_lag);
  if (rc) return rc;
  // the same work layout as lbm_classify_series: the series, then its lags
  const long long stride = series_work_doubles(n);
  if ((long long)nseries > kNoAllocScratchDoubles / stride)
    return lbm_fail(LBM_EINVAL,
                    "nseries * (2 n + 8) = %d * %lld doubles exceeds the %lld-double (32 MiB) "
                    "work array of the no-allocation classifier; classify fewer or shorter "
                    "series per call",
                    nseries, stride, kNoAllocScratchDoubles);
  double *work = scratch_for_current_device(rc);
  if (!work) return rc;
  hipError_t e = launch_classify(SeriesFromRows{series_dev, (long long)ld, (long long)n}, nseries,
                                 n, steady_tol, periodic_tol, min_lag, max_lag, work, stride,
                                 out_dev, (hipStream_t)hip_stream);
  if (e != hipSuccess) return lbm_fail(LBM_EDEVICE, "classify launch: %s", hipGetErrorString(e));
  return LBM_OK;
}
