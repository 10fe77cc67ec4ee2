// Host check of the wait for a device-driven run, with stand-ins for the event
// and the clock; argument 1 names the case.  Prints how the wait ended (0 outcome,
// 1 batch, 2 time limit, 3 error) and how often the event was asked.
#include <cstdio>
#include <string>

#include "wait.h"

int main(int argc, char** argv) {
  if (argc < 2) return 2;
  const std::string what = argv[1];
  int polls = 0;
  const mmsd::Wait w = mmsd::wait_batch(
      [&] { return what == "outcome" && polls >= 5; },
      [&] {
        ++polls;
        return what == "batch" && polls == 7 ? 1 : what == "error" && polls == 3 ? -1 : 0;
      },
      [&] { return what == "hung" ? polls >= 5000 : what == "late" ? true : polls >= 100000; });
  std::printf("wait %d polls %d\n", (int)w, polls);
  return 0;
}
