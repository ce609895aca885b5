// The host's wait for a pinned staging slot that a kernel reads: the kernel's workgroups store the call's number in the slot's
// flags when they have read their part.  No HIP in this file: the tests compile it with the host compiler.
#pragma once

#include <stdint.h>

#include <chrono>
#include <thread>

namespace relaygr {

// What is known of the stream the kernel was put on.  kBusy: it has work left, or cannot be asked (it is under capture).
enum class StreamState { kBusy, kDrained, kFailed };

struct FlagWait {
  int polls = 20000;                                  // looks without a pause (about a millisecond), then one every `nap`
  std::chrono::microseconds nap{20};
  std::chrono::milliseconds ask_every{10};            // a question about the stream takes a lock or two of the runtime's
  // A stream that has run dry has run the kernel.  The wait goes on for this long all the same, because the stream may be
  // another one by now (destroyed by its owner, and its handle given out again).
  std::chrono::milliseconds grace{1000};
};

// Waits until flags[0 .. n-1] all hold seq.  A busy stream is waited for as long as it takes; false if the stream has failed, or has
// had nothing left to run for FlagWait::grace: the kernel is not going to set its flags then.
// (No wait for the device: that would also wait for streams that have nothing to do with the call, and fail while one of them is
// being captured.)
template <class Ask>
inline bool wait_for_flags(const uint32_t* flags, int n, uint32_t seq, Ask ask, const FlagWait& w = FlagWait()) {
  using clock = std::chrono::steady_clock;
  int k = 0;
  auto all_set = [&] {
    while (k < n && __atomic_load_n(flags + k, __ATOMIC_ACQUIRE) == seq) ++k;
    return k == n;
  };
  for (int looks = 0; looks < w.polls; ++looks) {
    if (all_set()) return true;
    __builtin_ia32_pause();
  }
  clock::time_point next_ask = clock::now(), drained{};
  bool dry = false;                                   // the last answers all were: drained, since `drained`
  for (;;) {
    if (all_set()) return true;
    const clock::time_point now = clock::now();
    if (now >= next_ask) {
      const StreamState s = ask();
      if (s != StreamState::kBusy && all_set()) return true;
      if (s == StreamState::kFailed) return false;
      if (s == StreamState::kDrained && dry && now - drained >= w.grace) return false;
      if (s == StreamState::kDrained && !dry) drained = now;
      dry = s == StreamState::kDrained;
      next_ask = now + w.ask_every;
    }
    std::this_thread::sleep_for(w.nap);
  }
}

}  // namespace relaygr
