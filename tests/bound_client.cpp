// Prints, for each "T k runs" line of its input, the top-k bound's sample size, rank and slack and the sizes of the
// candidate buffers, from the library's own header.  Built and run by tests/test_bound.py.
#include <cstdio>

#include "select_bound.h"

int main() {
  int T, k, runs;
  while (scanf("%d %d %d", &T, &k, &runs) == 3) {
    const int run = runs ? asl::kSelSampleRun : 1;
    const int n_s = asl::sel_sample_size(T) / run * run;
    const int m = asl::sel_sample_rank(T, k, n_s, run);
    printf("%d %d %d %d %d %d %d\n", n_s, run, m, m < n_s ? asl::sel_bound_slack(T, m, n_s, run) : 0, asl::kSelCandCap,
           asl::kSelTile, asl::kSelSegment);
  }
  return 0;
}
