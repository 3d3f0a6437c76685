// Device code of a short vector's ranking with the statistic in the same launch.
#pragma once
#include "rank_body.h"
#include "rankvar_body.h"

namespace asl {

// The workgroup that has a token's rank adds up its part of the statistic: the token's older ranks are the only thing still to be
// read, and no launch stands between (a launch of its own takes 5 us on the device and 3 on the host; us, with it and so: a call
// of asl_rank_stat of 2000 scores 13.6, 11.0; of 12000 13.5, 11.2).
struct RankStatShared {
  ShortRankShared rank;
  KeptRanks kept;
  RankvarShared<kSortThreads> var;
};
static_assert(kShortT / kShortPlaces <= kVarMaxBlocks && kCountT / kCountTokens <= kVarMaxBlocks, "the statistic's table");
static_assert(kShortKept % 64 == 0 && kShortKept <= kSortThreads, "a thread per token that is kept");

// Workgroup b of n_blocks = short_rank_blocks(T).  Workgroup 0 waits for the others' sums; they wait for nobody.
__device__ __forceinline__ void rank_stat_short_body(RankStatShared& sh, const float* __restrict__ s, int32_t* __restrict__ rank_row,
                                                     const RankvarArgs& a, int b, int n_blocks) {
  const int tid = threadIdx.x;
  if (tid < kShortKept) sh.kept.tok[tid] = 0xffffffffu;
  if (tid == 0) sh.var.gave_up = 0;
  const bool counts = a.T <= kCountT;
  const uint32_t first = (uint32_t)(b * (counts ? kCountTokens : kShortPlaces));
  rank_short_body(sh.rank, s, a.T, PutAndKeepRank{rank_row, &sh.kept, first, counts}, b);
  if (a.skip != 0) {                                    // uniform
    if (b == 0 && tid == 0) stat_skip_body(a.out, a.state, a.layer_idx, a.l_obs, a.push);
    return;
  }
  const unsigned long long tag = *a.epoch + 1ull;
  const int n = rows_in_use(a.state, a.layer_idx, a.l_obs, a.push);
  __syncthreads();
  if (tid < kShortKept) {                               // whole wavefronts
    unsigned long long num = 0;
    uint32_t cnt = 0;
    const uint32_t t = sh.kept.tok[tid], r = sh.kept.rank[tid];
    if (n >= 2 && t < (uint32_t)a.T) {
      unsigned long long s1 = r, s2 = (unsigned long long)r * r;
      uint32_t least = r;
      int row0 = (a.layer_idx - (n - 1)) % a.l_obs;      // oldest row in use
      if (row0 < 0) row0 += a.l_obs;
      for (int j0 = 0; j0 < n - 1; j0 += kVarRowBatch) {
        uint32_t v[kVarRowBatch];
#pragma unroll
        for (int u = 0; u < kVarRowBatch; ++u) {          // issued together; beyond the last row the oldest once more, left out below
          int row = row0 + (j0 + u < n - 1 ? j0 + u : 0);
          row = row >= a.l_obs ? row - a.l_obs : row;
          v[u] = (uint32_t)a.ring[(int64_t)row * a.T + t];
        }
#pragma unroll
        for (int u = 0; u < kVarRowBatch; ++u)
          if (j0 + u < n - 1) {                           // uniform
            s1 += v[u];
            s2 += (unsigned long long)v[u] * v[u];
            least = min(least, v[u]);
          }
      }
      if (least < (uint32_t)a.k) {
        num = (unsigned long long)n * s2 - s1 * s1;
        cnt = 1;
      }
    }
    num = wave_sum(num);
    cnt = wave_sum(cnt);
    if ((tid & 63) == 0) {
      sh.var.red_num[tid >> 6] = num;
      sh.var.red_cnt[tid >> 6] = cnt;
    }
  }
  __syncthreads();
  if (tid == 0) {
    unsigned long long num = 0;
    uint32_t cnt = 0;
    for (int w = 0; w < kShortKept / 64; ++w) {
      num += sh.var.red_num[w];
      cnt += sh.var.red_cnt[w];
    }
    rankvar_publish(a, b, tag, num, cnt);
  }
  if (b != 0) return;
  __syncthreads();                                      // red_* are reused
  rankvar_collect(sh.var, a, n_blocks, tag, n);
}

}  // namespace asl
