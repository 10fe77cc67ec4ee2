// The host's wait for a run that the device drives.
#pragma once
#include <thread>

namespace mmsd {

enum class Wait { kOutcome, kBatch, kTimeout, kError };

// Waits until outcome() holds (the run's result is in host memory), the batch of
// launches whose end query() watches is done (1; 0: not yet, < 0: error), or
// late() says that the run's time is up, which a batch that never ends must
// not keep from being seen.  Polls without a pause for about the time of a
// short evaluation, then lets other threads have the core in between.
template <typename Outcome, typename Query, typename Late>
Wait wait_batch(Outcome&& outcome, Query&& query, Late&& late) {
  constexpr int kSpins = 1024;
  for (int spins = 0;; ++spins) {
    if (outcome()) return Wait::kOutcome;
    if (late()) return Wait::kTimeout;
    const int q = query();
    if (q != 0) return q > 0 ? Wait::kBatch : Wait::kError;
    if (spins < kSpins) {
      for (int k = 0; k < 16; ++k) __builtin_ia32_pause();
    } else {
      std::this_thread::yield();
    }
  }
}

}  // namespace mmsd
