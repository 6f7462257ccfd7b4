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

// Whether work issued to st runs now and is not recorded into a graph: a staged
// copy would put the pinned buffers into the caller's graph.
bool runs_now(hipStream_t st) {
  hipStreamCaptureStatus status;
  if (hipStreamIsCapturing(st, &status) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return status == hipStreamCaptureStatusNone;
}

constexpr int kBufs = 3, kMaxRings = 4;
constexpr int kLargeHelpers = 8, kSmallHelpers = 3;
constexpr size_t kLargeChunk = 4u << 20, kSmallChunk = 1u << 20;
constexpr size_t kLargeBytes = 16u << 20, kMinBytes = 4u << 20;

// kBufs buffers of `chunk` bytes, pinned for every device.
struct Ring {
  char *mem = nullptr;
  size_t chunk = 0;
  bool busy = false;
};

class Rings {
 public:
  void join() {
    std::lock_guard<std::mutex> lock(mutex_);
    ++users_;
  }
  void leave() {
    std::lock_guard<std::mutex> lock(mutex_);
    if (--users_ > 0) return;
    Ring *keep = &ring_[0];   // the largest stays
    for (Ring &r : ring_)
      if (r.chunk > keep->chunk) keep = &r;
    for (Ring &r : ring_)
      if (&r != keep && !r.busy) drop(r);
  }
  // An idle ring of at least `chunk` bytes a buffer, marked busy; null if all
  // are in use or there is no memory.
  Ring *take(size_t chunk) {
    std::lock_guard<std::mutex> lock(mutex_);
    Ring *best = nullptr;   // the smallest that serves, else an empty place, else any
    auto rank = [&](const Ring &r) { return r.chunk >= chunk ? 0 : r.mem ? 2 : 1; };
    for (Ring &r : ring_)
      if (!r.busy && (!best || rank(r) < rank(*best) ||
                      (rank(r) == 0 && rank(*best) == 0 && r.chunk < best->chunk)))
        best = &r;
    if (!best) return nullptr;
    if (best->chunk < chunk) {
      drop(*best);
      if (hipHostMalloc((void **)&best->mem, kBufs * chunk, hipHostMallocPortable) !=
          hipSuccess) {
        (void)hipGetLastError();
        best->mem = nullptr;
        return nullptr;
      }
      best->chunk = chunk;
    }
    best->busy = true;
    return best;
  }
  void give(Ring *r) {
    std::lock_guard<std::mutex> lock(mutex_);
    r->busy = false;
  }

 private:
  static void drop(Ring &r) {
    if (r.mem) (void)hipHostFree(r.mem);
    r = Ring{};
  }
  std::mutex mutex_;
  Ring ring_[kMaxRings];
  int users_ = 0;
};
Rings g_rings;

hipError_t copy_plain(const CopyOut *outs, int n, hipStream_t st) {
  for (int k = 0; k < n; ++k)
    if (outs[k].dst) {
      const hipError_t e =
          hipMemcpyAsync(outs[k].dst, outs[k].src, outs[k].bytes, hipMemcpyDeviceToHost, st);
      if (e != hipSuccess) return e;
    }
  return hipStreamSynchronize(st);
}

// Copy the chunks into the buffers at pin (`chunk` bytes each) in turn; up to
// `most` helpers move each one on, a slice each, while the next one comes.
// Started threads go into `helpers`; with none, e is hipErrorNotReady and
// nothing has been issued.
hipError_t copy_staged(const std::vector<CopyOut> &chunks, char *pin, size_t chunk,
                       std::vector<std::thread> &helpers, int most, hipStream_t st) {
  // ready: chunks that have arrived in their buffer; left[b]: slices of buffer
  // b that are still to be moved on; parts: slices of a chunk (set before go)
  std::atomic<size_t> ready{0};
  std::atomic<bool> stop{false};
  std::atomic<int> left[kBufs];
  for (auto &l : left) l = 0;
  int parts = 0;
  // The first chunk comes after all that is queued on the stream, so the
  // helpers sleep until then; later chunks follow at the link's rate.
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
  auto help = [&](int k) {
    {
      std::unique_lock<std::mutex> lock(mutex);
      begun.wait(lock, [&] { return go; });
    }
    for (size_t c = 0; c < chunks.size(); ++c) {
      while (ready.load(std::memory_order_acquire) <= c) {
        if (stop.load(std::memory_order_acquire)) return;
        std::this_thread::yield();
      }
      const int b = (int)(c % kBufs);
      auto cut = [&](int j) {   // slices of whole pages
        return j == parts ? chunks[c].bytes : chunks[c].bytes * j / parts / 4096 * 4096;
      };
      std::memcpy((char *)chunks[c].dst + cut(k), pin + b * chunk + cut(k),
                  cut(k + 1) - cut(k));
      left[b].fetch_sub(1, std::memory_order_release);
    }
  };
  const unsigned hw = std::thread::hardware_concurrency();
  if (hw) most = std::min(most, (int)hw);
  try {
    for (int k = 0; k < most; ++k) helpers.emplace_back(help, k);
  } catch (...) {   // as many as there are
  }
  parts = (int)helpers.size();
  if (parts == 0) return hipErrorNotReady;
  hipError_t e = hipSuccess;
  for (size_t c = 0; c < chunks.size() && e == hipSuccess; ++c) {
    const int b = (int)(c % kBufs);
    while (left[b].load(std::memory_order_acquire)) std::this_thread::yield();
    e = hipMemcpyAsync(pin + b * chunk, chunks[c].src, chunks[c].bytes, hipMemcpyDeviceToHost,
                       st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) break;
    left[b].store(parts, std::memory_order_relaxed);
    ready.store(c + 1, std::memory_order_release);
    if (c == 0) begin();
  }
  if (e != hipSuccess) stop.store(true, std::memory_order_release);
  begin();
  for (std::thread &t : helpers) t.join();
  return e;
}
}  // namespace

void HostStage::release() {
  if (user_) g_rings.leave();
  user_ = false;
}

hipError_t HostStage::copy(const CopyOut *outs, int n, hipStream_t st) {
  size_t total = 0;
  for (int k = 0; k < n; ++k)
    if (outs[k].dst) total += outs[k].bytes;
  bool staged = total >= kMinBytes && runs_now(st);
  for (int k = 0; k < n && staged; ++k)
    if (outs[k].dst) staged = pageable(outs[k].dst);
  if (!staged) return copy_plain(outs, n, st);

  const bool large = total >= kLargeBytes;
  const size_t chunk = large ? kLargeChunk : kSmallChunk;
  const int most = large ? kLargeHelpers : kSmallHelpers;
  std::vector<CopyOut> chunks;
  std::vector<std::thread> helpers;
  Ring *ring = nullptr;
  try {
    for (int k = 0; k < n; ++k)
      for (size_t o = 0; outs[k].dst && o < outs[k].bytes; o += chunk)
        chunks.push_back({(char *)outs[k].dst + o, (const char *)outs[k].src + o,
                          std::min(chunk, outs[k].bytes - o)});
    helpers.reserve(most);
    if (!user_) g_rings.join();
    user_ = true;
    ring = g_rings.take(chunk);
  } catch (...) {   // no host memory
  }
  if (!ring) return copy_plain(outs, n, st);
  const hipError_t e = copy_staged(chunks, ring->mem, chunk, helpers, most, st);
  // after an error the copy into the ring may still be running
  if (e == hipSuccess || e == hipErrorNotReady || hipStreamSynchronize(st) == hipSuccess)
    g_rings.give(ring);
  return e == hipErrorNotReady ? copy_plain(outs, n, st) : e;
}

}  // namespace lbm
