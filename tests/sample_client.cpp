// Prints, for each T of its input, the stride of the sample that rankings and top-k take of T scores and the sampled
// positions, from the library's own header.  Built and run by tests/test_bound.py.
#include <cstdio>

#include "select_bound.h"

int main() {
  int T;
  while (scanf("%d", &T) == 1) {
    const int stride = asl::sel_sample_stride(T), n_s = asl::sel_sample_size(T);
    printf("%d", stride);
    for (int j = 0; j < n_s; ++j) printf(" %u", asl::sel_sample_position((uint32_t)j, stride));
    printf("\n");
  }
  return 0;
}
