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
// runs on one thread, which also takes the page faults of a fresh array; the
// device fills pinned memory at 57 GB/s.  So larger copies go through a ring of
// three pinned buffers: the calling thread copies one chunk after another into
// them, and helper threads move each on, a slice each.  Medians of the copy
// alone, ms, plain / staged (fresh: into pages never touched, 4 KB each):
//            4.2 MB       6 MB         16 MB        54 MB        226 MB
//   warm     0.25 / 0.14  0.35 / 0.19  1.02 / 0.44  3.14 / 1.20  12.3 / 4.7
//   fresh    0.98 / 0.51  1.37 / 0.63  4.04 / 0.95  12.9 / 3.0   51.5 / 9.9
// From kLargeBytes on eight helpers and buffers of 4 MB; below that three
// helpers and buffers of 1 MB (16 MB warm in chunks of 512 KB, 1, 2, 4 MB: 0.62,
// 0.47, 0.42, 0.44 ms; with eight helpers 6 MB take 0.26).  A wait for the
// stream after each chunk: with an event per buffer and the next chunks queued
// ahead a chunk took 39 us instead of 26 a MB, and destroying a stream after
// that 0.1 ms longer.  Below kMinBytes, and for pinned or device destinations,
// the copy is hipMemcpyAsync's.
//
// The rings belong to the process, not to a handle: the first touch of newly
// pinned memory costs up to 0.35 ms a MB, so a ring of every handle's own made
// its first read slower than the plain copy (18 MB of populations at 500 x 500:
// 1.3 ms plain, 2.1 staged) and held 16 MB until it was destroyed.  A copy
// takes an idle ring for its length.  There are at most kMaxRings (48 MB in
// all); a copy that finds them in use is hipMemcpyAsync's.  When the last
// handle that has used one is destroyed all but one are given back: with a
// ring pinned again for each of a sequence of handles that are created, read
// once and destroyed, a sequence took 0.67 ms at 500 x 500 (6 MB), with plain
// copies 0.57, now 0.49.
class HostStage {
 public:
  // Copy every entry after the work queued on st; returns once all have arrived.
  hipError_t copy(const CopyOut *outs, int n, hipStream_t st);
  void release();   // the handle reads no more (no copy running)

 private:
  bool user_ = false;   // counted among the rings' users
};

}  // namespace lbm
