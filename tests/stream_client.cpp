// Prints, for each "bytes reads shared" line of its input, whether such keys are loaded past the last-level cache, by the library's
// own header.  Built and run by tests/test_split.py.
#include <cstdio>

#include "score_split.h"

int main() {
  long long bytes;
  int reads, shared;
  while (scanf("%lld %d %d", &bytes, &reads, &shared) == 3) printf("%d\n", asl::stream_keys(bytes, reads, shared != 0) ? 1 : 0);
  return 0;
}
