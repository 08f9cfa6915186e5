// Reading the device's ticket counter: a one-thread kernel stores it to a word
// of pinned memory and the host watches that word.  9 us, against 21 for a
// copy to pageable memory and a stream synchronisation, 13 for one to pinned
// memory.  Like such a copy (a kernel too, for so few bytes) it waits for the
// device: behind a kernel that shares its hardware queue, or for a free
// wavefront.  So the wait has a bound, and no answer is an error, not a count.
#pragma once

#include <errno.h>
#include <immintrin.h>
#include <stdint.h>
#include <time.h>

#include <mutex>

namespace gsys_host {

class CounterRead {
 public:
  enum Stream { kBusy, kIdle, kFailed };

  // launch(): queue the store of the counter to *word on a stream (false: it
  // failed).  stream(): what that stream does.  Gives up at `deadline`
  // (CLOCK_MONOTONIC ns; 0: never), also while another thread reads.
  // 0 and *out, -ETIMEDOUT, or -ENODEV (the launch failed, or the stream ended
  // or failed without storing).
  template <class Launch, class StreamState>
  int read(uint64_t* word, uint64_t deadline, Launch launch, StreamState stream, uint64_t* out) {
    Pause turn;
    while (!mu_.try_lock())
      if (turn.passed(deadline)) return -ETIMEDOUT;
    std::lock_guard<std::mutex> g(mu_, std::adopt_lock);
    // a read that was given up still owes its store: were it to arrive after
    // the word is cleared below, it would pass for this read's, and it may be
    // older than tickets that this read has to see
    if (owed_)
      if (int e = await(word, deadline, stream)) return e;
    __atomic_store_n(word, kUnset, __ATOMIC_RELEASE);
    if (!launch()) return -ENODEV;
    owed_ = true;
    const int e = await(word, deadline, stream);
    if (!e) *out = __atomic_load_n(word, __ATOMIC_ACQUIRE);
    return e;
  }

 private:
  static constexpr uint64_t kUnset = ~0ull;  // no ticket gets that far

  static uint64_t now_ns() {
    timespec ts;
    clock_gettime(CLOCK_MONOTONIC, &ts);
    return (uint64_t)ts.tv_sec * 1000000000ull + (uint64_t)ts.tv_nsec;
  }

  // One turn of a wait: spins for 200 us, then sleeps 20 us at a time.
  struct Pause {
    uint32_t n = 0;
    uint64_t t0 = 0;
    bool slow = false;
    bool passed(uint64_t deadline) {
      _mm_pause();
      if (!slow && (++n & 63)) return false;
      const uint64_t t = now_ns();
      if (!t0) t0 = t;
      slow = t - t0 > 200000;
      if (deadline && t > deadline) return true;
      if (slow) {
        timespec ts{0, 20000};
        nanosleep(&ts, nullptr);
      }
      return false;
    }
  };

  // Until the store that is owed has arrived.
  template <class StreamState>
  int await(uint64_t* word, uint64_t deadline, StreamState stream) {
    auto here = [&] { return __atomic_load_n(word, __ATOMIC_ACQUIRE) != kUnset; };
    Pause p;
    for (uint32_t k = 0; !here();) {
      if (p.passed(deadline)) return -ETIMEDOUT;
      if (!p.slow || (++k & 63)) continue;
      const Stream s = stream();
      if (s == kBusy || here()) continue;
      if (s == kIdle) owed_ = false;  // it ended without storing
      return -ENODEV;
    }
    owed_ = false;
    return 0;
  }

  std::mutex mu_;
  bool owed_ = false;  // under mu_
};

}  // namespace gsys_host
