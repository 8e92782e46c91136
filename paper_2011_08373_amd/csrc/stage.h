// Page-locked host memory of a thread's calls.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace rp {

// Page-locked host staging for the descriptor upload, and space for results,
// one per host thread, grown on demand and kept for the life of the thread
// (never freed: a thread-exit free could run after the runtime is gone).  A
// call waits for its stream before it returns; one that fails before that
// leaves an event behind what it enqueued (the upload out of the one buffer,
// kernels and copies that write the other), which the next call waits for
// before it writes or frees either.
struct PinnedStage {
  uint8_t* p = nullptr;
  size_t cap = 0;
  hipEvent_t done = nullptr;
  bool pending = false;
  uint8_t* get(size_t n) {
    if (!settle()) return nullptr;
    return grow(p, cap, n) ? p : nullptr;
  }
  // page-locked space for results read back by this thread's calls (each
  // call waits for its copies before it returns)
  uint8_t* rb = nullptr;
  size_t rb_cap = 0;
  template <class T = uint32_t>
  T* readback(size_t n) {
    if (!settle()) return nullptr;
    return grow(rb, rb_cap, n) ? reinterpret_cast<T*>(rb) : nullptr;
  }
  // a call that has not waited for its stream ends: what it enqueued on s
  void in_flight(hipStream_t s) {
    if (!done && hipEventCreateWithFlags(&done, hipEventDisableTiming) != hipSuccess) done = nullptr;
    if (done && hipEventRecord(done, s) == hipSuccess) pending = true;
    else (void)hipStreamSynchronize(s);
  }

 private:
  bool settle() {
    if (pending && (!done || hipEventSynchronize(done) != hipSuccess)) return false;
    pending = false;
    return true;
  }
  static bool grow(uint8_t*& b, size_t& have, size_t n) {
    if (n <= have) return true;
    if (b) (void)hipHostFree(b);
    b = nullptr;
    have = 0;
    const size_t want = n < 4096 ? 4096 : n;
    if (hipHostMalloc((void**)&b, want, hipHostMallocDefault) != hipSuccess) {
      b = nullptr;
      return false;
    }
    have = want;
    return true;
  }
};

}  // namespace rp
