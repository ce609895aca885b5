// Host build of the staging wait (csrc/staging.h) for tests/test_staging_wait.py.
#include "../paper_2601_01712_amd/csrc/staging.h"

using namespace relaygr;

extern "C" int wait_flags(const uint32_t* flags, int n, uint32_t seq, int grace_ms, int (*ask)()) {
  FlagWait w;
  w.polls = 100;
  w.ask_every = std::chrono::milliseconds(2);
  w.grace = std::chrono::milliseconds(grace_ms);
  return wait_for_flags(flags, n, seq, [&] { return static_cast<StreamState>(ask()); }, w) ? 1 : 0;
}
