// Prints, for each "T k S" line of its input, what a layer step's top-k of scores pooled over S tokens makes room for: sample
// size, rank, slack, sampled keys alike, candidates, from the library's own header.  Built and run by tests/test_bound.py.
#include <cstdio>

#include "select_bound.h"

int main() {
  int T, k, S;
  while (scanf("%d %d %d", &T, &k, &S) == 3) {
    const int n_s = asl::sel_sample_size(T), m = asl::sel_sample_rank(T, k, n_s, 1);
    const int slack = asl::sel_bound_slack(T, m, n_s, 1), alike = asl::sel_sample_alike(T, S);
    printf("%d %d %d %d %d\n", n_s, m, slack, alike, asl::sel_cand_cap(T, m, slack, n_s, alike));
  }
  return 0;
}
