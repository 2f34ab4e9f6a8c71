// Device blocks of destroyed plans, kept for the next plans of their context.
//
// A plan is made for every request and its tables are one device allocation.  hipFree waits for
// everything on the GPU and so stalls the requests behind it; a block is parked instead and handed
// out when the work that reads it is known to be done, whether or not it was done when its plan went,
// and in whatever order plans come and go.  A stream of the caller's may be gone by the time a plan
// is destroyed, so its handle is only compared, never used: the next plan that is uploaded on that
// stream looks whether it is idle, or leaves an event there behind the work of the parked blocks.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <utility>

namespace mpic {

inline bool capturing(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// Not a stream that work can be followed on: it is being captured (a graph may run at any time), or
// its handle means another stream in every thread.
inline bool trackable(hipStream_t stream) { return stream != hipStreamPerThread && !capturing(stream); }

// Where the work that reads a plan's tables was enqueued.
struct PlanUse {
  static constexpr int kMaxStreams = 3;  // (the caller's, the library's linking stream, one more)
  hipStream_t streams[kMaxStreams] = {};
  int n = 0;
  bool known = true;  // false: on more streams, or on one that is not trackable

  void add(hipStream_t stream) {
    if (!known) return;
    known = trackable(stream);
    for (int i = 0; i < n; ++i)
      if (streams[i] == stream) return;
    if (n == kMaxStreams)
      known = false;
    else
      streams[n++] = stream;
  }
};

// The pool of one context.  Plans hold it too: one that outlives its context gives its block back
// to the runtime.
class SpareBlocks {
 public:
  static constexpr int kMax = 4;
  static constexpr size_t kMaxBytes = size_t{16} << 20;

  // What to allocate for a plan of `bytes`: 64 KB times 1, 1.5, 2, 3, 4, 6 ..., so that plans of similar or
  // slowly growing requests fit each other's blocks; larger plans, which are not kept, as they are.
  // (Allocations of 2 MB and more cost 60 us more here, so sizes are not rounded up further than that.)
  static size_t size_for(size_t bytes) {
    if (bytes > kMaxBytes) return bytes;
    size_t size = size_t{64} << 10;
    while (size < bytes) size *= 2;
    return size > (size_t{64} << 10) && size / 4 * 3 >= bytes ? size / 4 * 3 : size;
  }
  // A stream of the library's own, which lives as long as the pool is open.
  void own(hipStream_t stream) { own_ = stream; }

  // The smallest kept block of at least `bytes` that no work reads any more, or null.  `stream`: where
  // the plan it is for will be used first.
  void* take(size_t bytes, size_t* have, hipStream_t stream) {
    std::lock_guard<std::mutex> lock(mu_);
    follow(stream);
    Block* best = nullptr;
    for (Block& b : blocks_)
      if (b.ptr && b.bytes >= bytes && (!best || b.bytes < best->bytes) && done(&b)) best = &b;
    if (!best) return nullptr;
    void* const ptr = best->ptr;
    *have = best->bytes;
    best->ptr = nullptr;
    ++n_taken_;
    return ptr;
  }
  // Keep the block of a plan.  False: not kept, the caller frees it.  *replaced: one that had to go for
  // it, to be freed by the caller too (hipFree waits for the work that reads it), or null.
  bool give(void* ptr, size_t bytes, const PlanUse& use, void** replaced) {
    *replaced = nullptr;
    std::lock_guard<std::mutex> lock(mu_);
    if (closed_ || bytes > kMaxBytes || !use.known) return false;
    Block* to = nullptr;
    for (Block& b : blocks_)
      if (!b.ptr || (b.bytes < bytes && (!to || (to->ptr && b.bytes < to->bytes)))) to = &b;
    if (!to)  // all are as large: one whose stream may never be used again, the oldest of them
      for (Block& b : blocks_)
        if (!done(&b) && (!to || b.number < to->number)) to = &b;
    if (!to) return false;
    *replaced = to->ptr;
    to->ptr = nullptr;
    to->n_wait = 0;
    for (int i = 0; i < use.n; ++i) {
      to->wait[i] = Wait{use.streams[i], false};
      to->n_wait = i + 1;
      if (own_ && use.streams[i] == own_ && !(trackable(own_) && mark(to, i, own_))) return false;
    }
    to->ptr = ptr;
    to->bytes = bytes;
    to->number = ++n_given_;
    return true;
  }
  uint64_t handed_out() const { return n_taken_; }
  // Free what is kept (`free` waits for the work that reads it), for an allocation that fails otherwise.
  template <typename Free>
  bool trim(Free&& free) {
    std::lock_guard<std::mutex> lock(mu_);
    bool any = false;
    for (Block& b : blocks_) {
      if (!b.ptr) continue;
      free(b.ptr);
      b.ptr = nullptr;
      any = true;
    }
    return any;
  }
  template <typename Free>
  void close(Free&& free) {
    trim(free);
    std::lock_guard<std::mutex> lock(mu_);
    closed_ = true;
    for (Block& b : blocks_)
      for (hipEvent_t& ev : b.ev) {
        if (ev) (void)hipEventDestroy(ev);
        ev = nullptr;
      }
  }

 private:
  struct Wait {
    hipStream_t stream;
    bool marked;  // the event of the same index is on it, behind the work that reads the block
  };
  struct Block {
    void* ptr = nullptr;
    size_t bytes = 0;
    uint64_t number = 0;
    Wait wait[PlanUse::kMaxStreams] = {};
    hipEvent_t ev[PlanUse::kMaxStreams] = {};
    int n_wait = 0;
  };
  static bool mark(Block* b, int i, hipStream_t stream) {
    hipError_t e = hipSuccess;
    if (!b->ev[i]) e = hipEventCreateWithFlags(&b->ev[i], hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(b->ev[i], stream);
    if (e != hipSuccess) (void)hipGetLastError();
    b->wait[i].marked = e == hipSuccess;
    return b->wait[i].marked;
  }
  // `stream` is there: whatever parked blocks wait for on it can be followed from now on.
  void follow(hipStream_t stream) {
    bool any = false;
    for (Block& b : blocks_)
      for (int i = 0; b.ptr && i < b.n_wait; ++i) any = any || (b.wait[i].stream == stream && !b.wait[i].marked);
    if (!any || !trackable(stream)) return;
    const bool idle = hipStreamQuery(stream) == hipSuccess;
    if (!idle) (void)hipGetLastError();
    for (Block& b : blocks_)
      for (int i = b.n_wait - 1; b.ptr && i >= 0; --i) {
        if (b.wait[i].stream != stream || b.wait[i].marked) continue;
        if (idle)
          drop(&b, i);
        else
          mark(&b, i, stream);
      }
  }
  static void drop(Block* b, int i) {
    const int last = --b->n_wait;
    b->wait[i] = b->wait[last];
    std::swap(b->ev[i], b->ev[last]);
  }
  static bool done(Block* b) {
    for (int i = b->n_wait - 1; i >= 0; --i) {
      if (!b->wait[i].marked) return false;
      if (hipEventQuery(b->ev[i]) != hipSuccess) {
        (void)hipGetLastError();
        return false;
      }
      drop(b, i);
    }
    return true;
  }
  std::mutex mu_;
  Block blocks_[kMax];
  hipStream_t own_ = nullptr;
  bool closed_ = false;
  uint64_t n_given_ = 0, n_taken_ = 0;
};

}  // namespace mpic
