// The arithmetic behind the top-k's bound (see select.hip): the strided sample it is taken from, its rank in the
// sample, and the candidate buffers it has to respect.  Host code: the kernels get the numbers as arguments (worked
// out by every workgroup of the bound kernel they cost it 0.5 us).
#pragma once
#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define ASL_HOST_DEVICE __host__ __device__
#else
#define ASL_HOST_DEVICE
#endif

#ifndef ASL_SEL_TILE
#define ASL_SEL_TILE 4096
#endif

namespace asl {

constexpr int kSelTile = ASL_SEL_TILE;     // elements per select workgroup tile (a multiple of 256)
constexpr int kSelSegment = kSelTile / 2;   // candidate slots per select tile
constexpr int kSelCandCap = 16384;     // candidates of one row the finishing workgroup holds in LDS

constexpr int kShortT = 12288;           // longest score vector that is ranked and selected from in one launch, every
                                         // workgroup with all of it
// The top-k on its own takes longer ones so too, up to what fits a workgroup's LDS: kSelMidT scores always, kSelShortT from
// kSelShortRows rows on (a call, us, with bound, filter and finish, and so: 8 rows of 16000 16.1, 11.9; 130 rows of 20000
// 20.2, 15.5; 256 of 30000 27.8, 20.7; 64 of 30000 18.6, 17.0; with fewer rows of that length there is nothing left to gain).
constexpr int kSelMidT = 16384, kSelShortT = 32768, kSelShortRows = 64;
// The sample of a row of T scores: n_s = sel_sample_size(T) keys, one of every sel_sample_stride(T) tokens (all but the
// row's last few: the stride is rounded up), for T > kShortT.
constexpr int kSelMaxSample = 8192;    // sampled keys per row
inline int sel_sample_stride(int T) {
  int n = T / 32;
  n = n < 1024 ? 1024 : n;
  const int most = T <= 262144 ? kSelMaxSample / 2 : kSelMaxSample;   // the whole is for the ranking's 1024 buckets
  n = n > most ? most : n;
  return (T + n - 1) / n;
}
inline int sel_sample_size(int T) { return T / sel_sample_stride(T); }
// Sampled keys, one per stride, that a pooling of width S makes alike.
inline int sel_sample_alike(int T, int S) { return (S + sel_sample_stride(T) - 1) / sel_sample_stride(T); }
// Position of sampled key j among the tokens j * stride .. (j + 1) * stride - 1 that it stands for: a scattered one, so
// that scores with a period (rows of a grid, repeated text) do not meet a sample of the same period.  With positions
// j * stride a layer step of 131072 tokens whose scores repeat every 32 had one bucket of 124 K tokens: 4.7 ms.
ASL_HOST_DEVICE inline uint32_t sel_sample_position(uint32_t j, int stride) {
  return j * (uint32_t)stride + (((j * 2654435761u >> 16) * (uint32_t)stride) >> 16);
}
// Rank m of the sample key taken as the bound: f = n_s / T of the row is sampled, the top-k members
// among the sample are ~Binomial(n_s, k / T) with mean k f; m = k f + 5 sqrt(c k f) + 4 leaves the
// bound too low with probability < 1e-6.  c = 1 for single sampled keys; c = `run` when the sample
// consists of runs of `run` neighbouring keys, which may be as correlated as identical (pooled
// scores are): the count's variance is then at most `run` times the binomial one.
inline int sel_sample_rank(int T, int k, int n_s, int run) {
  const float kf = (float)k * (float)n_s / (float)T;
  const int m = (int)(kf + 5.0f * sqrtf((float)run * kf) + 4.0f);
  return m;                                            // >= n_s means: no usable bound, admit everything
}
// Rank of a sample key that is behind the row's k-th with probability < 1e-6, by the same estimate; at least 1.
inline int sel_sample_rank_low(int T, int k, int n_s, int run) {
  const float kf = (float)k * (float)n_s / (float)T;
  const int m = (int)(kf - 5.0f * sqrtf((float)run * kf) - 4.0f);
  return m < 1 ? 1 : m;
}
// How many sample keys beyond the m-th the bound may let pass: m / 8, and no more than the candidate buffers
// hold.  The m-th sample key admits m T / n_s tokens with standard deviation T / n_s sqrt(c m), c as above; a row's
// buffer must keep 3 of those free.  A tile's segment holds kSelTile / n_s keys per sample key, with the bound's
// deviation and that of the tile itself (kSelTile / 4 tokens in independent groups of 8, wider than pooling
// couples them); it must keep 4 free, since any of a row's tiles may overflow.  A row with more than its buffer
// holds costs ~10 us, one with a full tile is selected from global memory (~200 us); where the m-th key alone overflows them by
// a deviation, nothing is left to lose.
inline int sel_bound_slack(int T, int m, int n_s, int run) {
  const float per_key = (float)T / (float)n_s, per_key_tile = (float)kSelTile / (float)n_s, var = (float)run * (float)m;
  const float row_room = (float)kSelCandCap - (float)m * per_key, row_dev = per_key * sqrtf(var);
  const float tile_room = (float)kSelSegment - (float)m * per_key_tile, tile_dev = sqrtf(per_key_tile * per_key_tile * var + 2.0f * (float)kSelTile);
  const int s = m / 8;
  if (row_room < -row_dev || tile_room < -tile_dev) return s;
  const float row = (row_room - 3.0f * row_dev) / per_key, tile = (tile_room - 4.0f * tile_dev) / per_key_tile;
  const float cap = row < tile ? row : tile;
  return cap <= 0.f ? 0 : ((float)s < cap ? s : (int)cap);
}
// Candidates of a row that the finishing workgroup makes room for: half of kSelCandCap where the bound admits more than
// that once in 10^6 rows at most, since two workgroups then share a compute unit (a row with more takes ~10 us more).  alike: sampled keys that may be as correlated as identical, `run` as above or, for scores pooled over
// more tokens than the sample's stride, as many strides as the pooling covers.
inline int sel_cand_cap(int T, int m, int slack, int n_s, int alike) {
  const float per_key = (float)T / (float)n_s;
  return (float)(m + slack) * per_key + 5.0f * per_key * sqrtf((float)alike * (float)m) <= (float)(kSelCandCap / 2) ? kSelCandCap / 2 : kSelCandCap;
}
// Without a prepared sample the bound kernel reads runs of kSelSampleRun neighbouring keys, one run
// per kSelSampleRun sample strides: the same number of keys from a quarter of the cache lines.
constexpr int kSelSampleRun = 4;
static_assert(kShortT / 1024 >= kSelSampleRun && 32 >= kSelSampleRun, "a run fits the stride of any row that is sampled");

}  // namespace asl
