// Prints, for each "Hk blocks" line of its input, whether a short context's compaction goes into the launch that selects, by the
// library's own header.  Built and run by tests/test_split.py.
#include <cstdio>

#include "short_plan.h"

int main() {
  int Hk, blocks;
  while (scanf("%d %d", &Hk, &blocks) == 2) printf("%d\n", asl::short_whole(Hk, blocks) ? 1 : 0);
  return 0;
}
