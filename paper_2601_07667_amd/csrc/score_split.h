// How a scoring launch shares a KV head's key tiles out among its workgroups, and which loads it takes them with.  Host code
// but for TileSplit, which the kernels get as an argument.
#pragma once
#include <stdint.h>

#ifndef ASL_HOST_DEVICE
#ifdef __HIPCC__
#define ASL_HOST_DEVICE __host__ __device__
#else
#define ASL_HOST_DEVICE
#endif
#endif

namespace asl {

// The key tiles of a workgroup.  IN_TURN: the n_chunks workgroups of a KV head take the tiles in turn: the k-th of them tiles k,
// k + n_chunks, ..., so that a head's workgroups, which advance together, read one stretch of memory at a time.  (Each with a
// contiguous share they read at as many places, a power of two apart: a bare ring of this shape streams 268 MB in 44.9 us so,
// in turn in 41.6; 8B shape, 128K, `lse` supplied, pass 2 61.2 and 58.8 us; 32K, both passes, 33.4 and 31.5.)  Not IN_TURN:
// contiguous shares; for workgroups of one wavefront (kInTurn), which wait for every tile: theirs are then neighbours in memory
// (8B shape, W = 8, both passes, in turn and so: 16K 19.8, 18.9; 32K 31.6, 30.0; 64K 54.7, 52.8; two heads of d = 64, 8K 13.5, 13.0).
// All workgroups of a pass are resident at once (one round), block b being the (b / n_cu)-th placed on its compute unit.  A
// unit's older wavefronts go first, so with two workgroups per unit the second ends up alone on it for the last part of the
// kernel: after `all` rounds of everybody only the first placed take turns (1250 : 798 of a unit's tiles, with two row blocks a
// wavefront 1350 : 698, the more unequal the more the arithmetic bounds the kernel; pass 1 + pass 2 at 256K, W = 64, equal shares
// 152 + 158 us, 1250 : 798 147 + 153, 1350 : 698 145 + 150).  Up to four tiles per chunk that come out even to 1/16 stay
// equal: weighted, rounding makes some chunks a tile longer (8 KV heads, whole call, weighted and equal: one tile, W = 64
// 27.3 and 25.1 us; two tiles, W = 32 20.4 and 19.9; but 2.45, W = 64 31.1 and 31.7, 5.9 28.5 and 28.9).
template <bool IN_TURN>
struct TileSplit {
  int n_chunks;
  int all;                       // rounds that every chunk takes part in
  int first;                     // chunks that go on after them
  int more, longer;              // their further tiles: `more` each, and one for the first `longer` of them
  ASL_HOST_DEVICE int count(int chunk) const { return all + (chunk < first ? more + (chunk < longer ? 1 : 0) : 0); }
  ASL_HOST_DEVICE int tile(int chunk, int i) const {                  // i-th tile of a chunk, i < count(chunk)
    if (!IN_TURN) return chunk * all + (chunk < first ? chunk : first) * more + (chunk < longer ? chunk : longer) + i;
    return chunk + (i < all ? i * n_chunks : all * n_chunks + (i - all) * first);
  }
  // from the i-th to the next; backwards from the i-th to the one before: step(i - 1)
  ASL_HOST_DEVICE int step(int i) const { return !IN_TURN ? 1 : i < all ? n_chunks : first; }
};
template <int NW> constexpr bool kInTurn = NW > 1;     // NW wavefronts a workgroup

// Tiles of a unit's first-placed workgroup of every 2048 of the unit's.
inline int first_placed_weight(bool two_blocks) { return two_blocks ? 1350 : 1250; }

// two_blocks: two row blocks a wavefront.  n_chunks <= n_tiles.
template <bool IN_TURN>
TileSplit<IN_TURN> split_tiles(int Hk, int n_chunks, int n_tiles, int n_cu, bool two_blocks) {
  const int first_w = first_placed_weight(two_blocks), second_w = 2048 - first_w;
  const int grid = n_chunks * Hk;
  const int slots = n_chunks * (1 + (n_tiles > n_chunks) + (n_tiles > 2 * n_chunks) + (n_tiles > 3 * n_chunks));
  const bool even = n_tiles <= slots && 16 * (slots - n_tiles) <= slots;
  TileSplit<IN_TURN> s = {n_chunks, 0, n_chunks, 0, 0};
  if (grid > n_cu && grid <= 2 * n_cu && !even) {
    const int first = n_cu / Hk < 1 ? 1 : n_cu / Hk;   // block c * Hk + g is the first of its unit iff it is below n_cu
    const int64_t weight = (int64_t)first_w * first + (int64_t)second_w * (n_chunks - first);
    // No workgroup gets more than the first placed's weighted share rounded up: what is left by rounding the second placed's
    // down can be a tile for one or two of the first more, and they are the last to end (8B shape, `lse` supplied, us, so and with the
    // second's share rounded down throughout: W = 5, 12K 12.7, 13.3; W = 32, 24K 17.6, 18.3; 28 heads, W = 16, 60K 19.3, 20.0; two
    // heads of d = 64, 128K 15.2, 15.8).  Where only equal shares keep to that, they are equal.
    const int most = (int)(((int64_t)n_tiles * first_w + weight - 1) / weight);
    int all = (int)((int64_t)n_tiles * second_w / weight);
    if (all < 1) all = 1;                              // n_chunks <= n_tiles
    auto longest = [&] { return all + (n_tiles - all * n_chunks + first - 1) / first; };
    while (all < n_tiles / n_chunks && longest() > most) ++all;
    if (longest() <= most) {
      s.all = all;
      s.first = first;
    }
  }
  const int left = n_tiles - s.all * n_chunks;
  s.more = left / s.first;
  s.longer = left % s.first;
  return s;
}

// Whether the keys, so many bytes of them, are loaded with the non-temporal bit, past the last-level cache (256 MB).  `reads`: how
// often the call goes through them, once a pass and row group.  shared: several heads read the same keys (a head stride of 0).
// Lines where it gains in a layer step, whose other tensors leave little of the keys in the cache, and loses next to nothing in
// calls of asl_score_layer alone on a few sets of keys in turn, which find them there; us, without and with, of the 8B shape:
//  read once: 64 MB, step 42.3, 42.4, alone 21.5, 22.2; 80 MB 46.6, 45.3 and 24.1, 25.3; 96 MB 51.5, 48.0 and 27.7, 28.3; 200 MB
//    76.7, 68.2 and 50.4, 45.7; four heads of d = 256, step, 80 MB 45.4, 44.1; 96 MB 50.3, 46.9;
//  read by both passes: 96 MB, step 71.3, 70.7, alone 46.2, 51.3; 112 MB 79.2, 75.6 and 52.9, 56.6; 128 MB 85.3, 81.0 and 60.4, 60.7;
//    200 MB 114, 107 and 87.7, 85.2; d = 256, step, 128 MB 86.1, 80.5;
//  two row groups, `lse` supplied, four heads of d = 256 alone: 96 MB 56.0, 56.5; 200 MB 98.1, 97.6; 400 MB 191, 179.
// Shared keys are in the cache for the other heads: 8 of 4 query heads on one set, `lse` supplied, 32K 20.8, 22.5; 128K 54.3, 57.2.
inline bool stream_keys(int64_t bytes, int reads, bool shared) {
  return !shared && bytes >= int64_t(reads == 1 ? 80 : 112) << 20;
}

}  // namespace asl
