// Host check of parallel_for where no thread can be started: the address
// space is closed to new thread stacks, then every index of a range has to be
// visited exactly once.  Prints the number of indices visited once and of the
// calls that covered them.
#include <sys/resource.h>

#include <atomic>
#include <cstdio>
#include <vector>

#include "amg.h"

int main() {
  const int64_t n = 1 << 20;
  std::vector<int> seen(n, 0);
  std::atomic<int> calls{0};
  auto f = [&](int64_t a, int64_t b) {
    ++calls;
    for (int64_t i = a; i < b; ++i) ++seen[i];
  };
  long pages = 0;
  FILE* s = std::fopen("/proc/self/statm", "r");
  if (!s || std::fscanf(s, "%ld", &pages) != 1) return 2;
  std::fclose(s);
  rlimit lim{};
  lim.rlim_cur = lim.rlim_max = (rlim_t)pages * 4096 + (1 << 20);   // a stack takes 8 MB
  if (setrlimit(RLIMIT_AS, &lim) != 0) return 2;
  mmsd::parallel_for(n, f);
  int64_t once = 0;
  for (int v : seen) once += v == 1;
  std::printf("once %lld calls %d\n", (long long)once, calls.load());
  return 0;
}
