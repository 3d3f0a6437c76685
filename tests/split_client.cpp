// Prints, for each "Hk n_chunks n_tiles n_cu two_blocks" line of its input, how the library's own header shares a KV head's key
// tiles out, in turn and in contiguous shares: whether every tile is taken once, forwards and backwards alike, the longest share
// and the weight behind the shares.  Built and run by tests/test_split.py.
#include <cstdio>
#include <vector>

#include "score_split.h"

static int longest;

template <bool IN_TURN>
static bool whole(int Hk, int n_chunks, int n_tiles, int n_cu, bool two) {
  const asl::TileSplit<IN_TURN> s = asl::split_tiles<IN_TURN>(Hk, n_chunks, n_tiles, n_cu, two);
  std::vector<int> seen(n_tiles, 0);
  bool ok = true;
  longest = 0;
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
  return ok;
}

int main() {
  int Hk, n_chunks, n_tiles, n_cu, two;
  while (scanf("%d %d %d %d %d", &Hk, &n_chunks, &n_tiles, &n_cu, &two) == 5) {
    const bool own = whole<false>(Hk, n_chunks, n_tiles, n_cu, two != 0), turn = whole<true>(Hk, n_chunks, n_tiles, n_cu, two != 0);
    printf("%d %d %d\n", own && turn ? 1 : 0, longest, asl::first_placed_weight(two != 0));
  }
  return 0;
}
