// Host check of the slices' offsets near their 32-bit limit, from row lengths
// alone (`rows` rows of `len` entries, the first of `first`, W lanes per row):
// prints the number of offsets and the last one.
#include <cstdio>
#include <cstdlib>

#include "slices.h"

int main(int argc, char** argv) {
  if (argc < 5) return 2;
  const int rows = std::atoi(argv[1]), len = std::atoi(argv[2]), first = std::atoi(argv[3]), W = std::atoi(argv[4]);
  std::vector<int> rp(rows + 1, 0);
  for (int i = 0; i < rows; ++i) rp[i + 1] = rp[i] + (i ? len : first);
  const std::vector<int> so = mmsd::slice_offsets(rp, W);
  std::printf("offsets %zu last %d\n", so.size(), so.empty() ? -1 : so.back());
  return 0;
}
