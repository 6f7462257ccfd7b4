// host_copy.h -- large results into the caller's pageable memory.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace lbm {

struct CopyOut {
  void *dst;         // host memory (entries with a null dst are skipped)
  const void *src;   // device memory
  size_t bytes;
};

// A handle's path for device-to-host copies.  hipMemcpy into pageable memory
// runs on one thread, which also takes the page faults of a fresh array:
// 226 MB (the fields of a 192^3 box) take 21 to 62 ms, or 12.5 ms into an array
// that was written before.  The device fills pinned memory at 57 GB/s (4 ms),
// so larger copies go through a ring of pinned buffers and several threads
// move each one on, a slice each: 5 to 14 ms into the same fresh arrays (1, 2, 4
// and 8 threads: 19, 10, 6.3, 5.3 ms with huge pages).  Below kLargeBytes four
// threads and smaller chunks do better than eight: the fields of 500 x 500 FP64
// (6 MB) 1.38 -> 0.54 ms into fresh arrays, 0.35 either way into memory that was
// just freed; of 500 x 1000 2.7 -> 1.0 and 2.3 -> 1.0 ms.  Below kMinBytes
// starting the threads costs what it saves (2.3 MB: 0.53 -> 0.30 ms fresh, 0.14 ->
// 0.20 reused); pinned or device destinations are left to hipMemcpyAsync.
class HostStage {
 public:
  // Copy every entry after the work queued on st; returns once all have arrived.
  hipError_t copy(const CopyOut *outs, int n, hipStream_t st);
  void release();   // give the pinned buffers back (no copy running)

 private:
  static constexpr int kBufs = 4, kThreads = 8;
  static constexpr size_t kChunkBytes = 4u << 20, kSmallChunkBytes = 512u << 10;
  static constexpr size_t kMinBytes = 4u << 20, kLargeBytes = 16u << 20;
  bool ensure();
  char *pin_ = nullptr;
  hipEvent_t ev_[kBufs] = {};
};

}  // namespace lbm
