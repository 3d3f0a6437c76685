// Prints, for each "Hk n_chunks n_tiles n_cu two_blocks" line of its input, how the library's own header shares a KV head's key
// tiles out: whether every tile is taken once, forwards and backwards alike, the longest share and the weight behind the
// shares.  Built and run by tests/test_split.py.
#include <cstdio>
#include <vector>

#include "score_split.h"

int main() {
  int Hk, n_chunks, n_tiles, n_cu, two;
  while (scanf("%d %d %d %d %d", &Hk, &n_chunks, &n_tiles, &n_cu, &two) == 5) {
    const asl::TileSplit s = asl::split_tiles(Hk, n_chunks, n_tiles, n_cu, two != 0);
    std::vector<int> seen(n_tiles, 0);
    bool ok = true;
    int longest = 0;
    for (int c = 0; c < n_chunks; ++c) {
      const int n = s.count(c);
      longest = n > longest ? n : longest;
      int t = s.tile(c, 0);
      for (int i = 0; i < n; ++i) {
        if (t != s.tile(c, i) || t < 0 || t >= n_tiles) ok = false;
        else ++seen[t];
        t += s.step(i);
      }
      for (int i = n - 1; i > 0; --i) ok = ok && s.tile(c, i) - s.step(i - 1) == s.tile(c, i - 1);
    }
    for (int x : seen) ok = ok && x == 1;
    printf("%d %d %d\n", ok ? 1 : 0, longest, asl::first_placed_weight(two != 0));
  }
  return 0;
}
