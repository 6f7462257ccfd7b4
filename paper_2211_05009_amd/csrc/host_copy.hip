// host_copy.hip -- HostStage (host_copy.h).
#include "host_copy.h"

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace lbm {

namespace {
bool pageable(const void *p) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();   // memory the runtime has not seen
    return true;
  }
  return at.type == hipMemoryTypeUnregistered;
}

// Whether work issued to st runs now and is not recorded into a graph: the
// staged copies and their events would be recorded, with the pinned buffers in
// the caller's graph, and the wait for them would fail without ending the
// capture.
bool runs_now(hipStream_t st) {
  hipStreamCaptureStatus status;
  if (hipStreamIsCapturing(st, &status) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return status == hipStreamCaptureStatusNone;
}
}  // namespace

bool HostStage::ensure() {
  if (pin_) return true;
  if (hipHostMalloc((void **)&pin_, kBufs * kChunkBytes, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    pin_ = nullptr;
    return false;
  }
  for (hipEvent_t &e : ev_)
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      e = nullptr;
      release();
      return false;
    }
  return true;
}

void HostStage::release() {
  for (hipEvent_t &e : ev_) {
    if (e) (void)hipEventDestroy(e);
    e = nullptr;
  }
  if (pin_) (void)hipHostFree(pin_);
  pin_ = nullptr;
}

hipError_t HostStage::copy(const CopyOut *outs, int n, hipStream_t st) {
  size_t total = 0;
  bool staged = true;
  for (int k = 0; k < n; ++k)
    if (outs[k].dst) total += outs[k].bytes;
  staged = total >= kMinBytes && runs_now(st);
  const bool large = total >= kLargeBytes;
  const size_t chunk = large ? kChunkBytes : kSmallChunkBytes;
  for (int k = 0; k < n && staged; ++k)
    if (outs[k].dst) staged = pageable(outs[k].dst);
  std::vector<CopyOut> chunks;
  std::vector<std::thread> threads;
  if (staged) {
    try {
      for (int k = 0; k < n; ++k)
        for (size_t o = 0; outs[k].dst && o < outs[k].bytes; o += chunk)
          chunks.push_back({(char *)outs[k].dst + o, (const char *)outs[k].src + o,
                            std::min(chunk, outs[k].bytes - o)});
      threads.reserve(kThreads);
      staged = ensure();
    } catch (...) {
      staged = false;
    }
  }

  // ready: chunks that have arrived in their buffer; left[b]: slices of buffer
  // b that are still to be moved on
  std::atomic<size_t> ready{0};
  std::atomic<bool> stop{false};
  std::atomic<int> workers{0}, left[kBufs];
  for (auto &l : left) l = 0;
  // The first chunk comes after all that is queued on the stream, so the
  // workers sleep until then; later chunks follow at the link's rate.
  std::mutex mutex;
  std::condition_variable begun;
  bool go = false;
  auto begin = [&]() {
    {
      std::lock_guard<std::mutex> lock(mutex);
      go = true;
    }
    begun.notify_all();
  };
  auto work = [&](int k) {
    {
      std::unique_lock<std::mutex> lock(mutex);
      begun.wait(lock, [&] { return go; });
    }
    for (size_t c = 0; c < chunks.size(); ++c) {
      while (ready.load(std::memory_order_acquire) <= c) {
        if (stop.load(std::memory_order_acquire)) return;
        std::this_thread::yield();
      }
      const int T = workers.load(std::memory_order_relaxed), b = (int)(c % kBufs);
      auto cut = [&](int j) {   // slices of whole pages
        return j == T ? chunks[c].bytes : chunks[c].bytes * j / T / 4096 * 4096;
      };
      std::memcpy((char *)chunks[c].dst + cut(k), pin_ + b * kChunkBytes + cut(k),
                  cut(k + 1) - cut(k));
      left[b].fetch_sub(1, std::memory_order_release);
    }
  };
  if (staged) {
    const unsigned hw = std::thread::hardware_concurrency();
    const int most = large ? kThreads : kThreads / 2;
    const int want = hw ? std::min<int>(most, (int)hw) : most;
    try {
      for (int k = 0; k < want; ++k) threads.emplace_back(work, k);
    } catch (...) {   // as many as there are
    }
    staged = !threads.empty();
  }
  if (!staged) {
    for (int k = 0; k < n; ++k)
      if (outs[k].dst) {
        hipError_t e =
            hipMemcpyAsync(outs[k].dst, outs[k].src, outs[k].bytes, hipMemcpyDeviceToHost, st);
        if (e != hipSuccess) return e;
      }
    return hipStreamSynchronize(st);
  }

  const int T = (int)threads.size();
  workers.store(T, std::memory_order_relaxed);   // published by the first `ready`
  hipError_t e = hipSuccess;
  size_t issued = 0;
  for (size_t c = 0; c < chunks.size() && e == hipSuccess; ++c) {
    while (issued < chunks.size() && issued < c + kBufs && e == hipSuccess) {
      const int b = (int)(issued % kBufs);
      if (left[b].load(std::memory_order_acquire)) {
        if (issued > c) break;   // buffer busy, chunk c is on its way
        std::this_thread::yield();
        continue;
      }
      left[b].store(T, std::memory_order_relaxed);
      e = hipMemcpyAsync(pin_ + b * kChunkBytes, chunks[issued].src, chunks[issued].bytes,
                         hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipEventRecord(ev_[b], st);
      ++issued;
    }
    if (e == hipSuccess) e = hipEventSynchronize(ev_[c % kBufs]);
    if (e == hipSuccess) ready.store(c + 1, std::memory_order_release);
    if (c == 0 && e == hipSuccess) begin();
  }
  if (e != hipSuccess) stop.store(true, std::memory_order_release);
  begin();
  for (std::thread &t : threads) t.join();
  return e;
}

}  // namespace lbm
