// Whether a short context's compaction goes into the launch that selects.  Host code.
#pragma once

namespace asl {

constexpr int kTailUnits = 256;                       // compute units of an MI355X ...
constexpr int kDies = 8;                              // ... on so many dies

// Its workgroups (`blocks` a KV head) all run on the die of the head's selecting one, so few heads use few dies, which copy 0.5 MB/us
// each: in the launch where the fullest die's workgroups are at most one for each of its units, or where it has at most 8/5 of the heads'
// average.  A layer step, us, with statistic and compaction in a launch of their own and so; d = 128, T about 6000, evaluated (below
// L_min): 1 head, 1000 tokens 26.5, 25.0 (24.6, 24.2), 2200 26.5, 26.6 (25.0, 26.8), 4000 27.1, 28.3 (25.8, 28.4); 4 heads, 1000 27.0,
// 25.3 (25.7, 24.7), 2200 27.7, 27.5 (26.6, 27.5), 4000 29.1, 29.2 (28.1, 29.1); T about 10500, 4080 tokens: 5 heads 31.6, 31.3 (30.6,
// 31.3), 7 34.5, 33.3 (34.1, 33.3), 9 38.7, 39.4 (38.5, 39.5), 12 44.8, 43.0 (44.1, 43.0); 8 heads, 4000 38.1, 36.2.
inline bool short_whole(int Hk, int blocks) {
  const int most = (Hk + kDies - 1) / kDies;
  return 5 * most <= Hk || most * blocks <= kTailUnits / kDies;
}

}  // namespace asl
