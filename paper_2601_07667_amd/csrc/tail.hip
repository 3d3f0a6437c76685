// The part of a layer step that follows the scoring, in three launches on one stream (one or two for short contexts).
//
// After the scores are pooled two independent chains remain: the ranking (partition, buckets: Alg. 1 step 11) with the
// statistic (Alg. 2 steps 4-10), and the top-k + KV compaction (bound, filter, finish, gather: Alg. 1
// steps 9-10 and 12; Alg. 2 steps 11-12).  Run as separate launches they either serialise (one
// stream) or pay two cross-queue synchronisations per layer (two streams).  Here the stages share launches:
// the two jobs of a launch are independent, and every stage depends only on earlier launches, which the launch
// boundary orders (short contexts' compaction and statistic apart, which wait for words of other workgroups).  The bodies are the same device functions the single-call kernels use.
#include <type_traits>

#include "gather_body.h"
#include "rank_stat_body.h"
#include "select_body.h"
#include "short_plan.h"

namespace asl {

static_assert(kSortThreads == kFinThreads, "both jobs of a launch use the same workgroup size");
constexpr int kTailThreads = kSortThreads;

union PartFilterShared {
  PartShared part;
  FilterShared<true> filter;
};

// Short contexts (T <= kShortT) take one launch for all of it: the top-k of every row, the ranking with the statistic, and the compaction
// (up to kPickMost tokens of kPickMaxRows heads, where short_whole says so; else tail_short_kernel).  The selecting workgroups, the longer
// ones, come first; workgroup r < Hk leaves row r's tokens in words that carry the launch's tag, and the compacting
// workgroups of head r wait for theirs.  Those come last, 8 * i + x for heads r with r % 8 == x: on the die of the workgroup they
// wait for, behind it in the order in which a die starts them, so that waiting workgroups cannot keep the waited-for ones from
// starting, whatever else runs on the device.  gx: blocks per (head, tensor) slab, 0 for no compaction here.  A layer step, us, with
// statistic and compaction in a launch of their own and so: 8 KV heads 1K 23.6, 20.3; 8K 37.4, 33.7; 12K 35.2, 33.4; two heads of
// d = 64, 4K 21.7, 19.7; 11K 26.4, 24.5; 10K below L_min 25.2, 24.4.  WAVES: wavefronts of a SIMD that the scalar registers
// allow: 8 for two workgroups a unit where ranking and top-k have more than one for each (8K 37.3, 34.4); else 4, whose code is 0.6
// to 1 us faster.  Dynamic LDS: kTailShortLds.
constexpr size_t kTailShortLds = sizeof(ShortSelectShared<kShortPer>) > sizeof(RankStatShared) ? sizeof(ShortSelectShared<kShortPer>) : sizeof(RankStatShared);
__host__ __device__ constexpr int short_gather_from(int rows, int n_rank) { return (rows + n_rank + kDies - 1) / kDies * kDies; }
template <bool POW2, int WAVES>
__global__ void __launch_bounds__(kTailThreads, WAVES) tail_whole_kernel(const float* s_all, int32_t* rank_row, SelectArgs se, int rows, int n_rank,
                                                                     RankvarArgs ra, GatherArgs ga, int gx, int Hk) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  const int b = (int)blockIdx.x;
  if (b < rows) {
    select_short_body<kShortPer, true>(*reinterpret_cast<ShortSelectShared<kShortPer>*>(lds_dyn), se, b);
  } else if (b < rows + n_rank) {
    rank_stat_short_body(*reinterpret_cast<RankStatShared*>(lds_dyn), s_all, rank_row, ra, b - rows, n_rank);
  } else {
    const int j = b - short_gather_from(rows, n_rank);
    if (j < 0) return;
    const int i = j / kDies, slabs = gx * ga.n_tensors, h = j % kDies + kDies * (i / slabs), slab = i % slabs;
    if (h >= Hk) return;
    if (!gather_picked_body<POW2, kTailThreads>(ga, slab % gx, h, slab / gx, se.T, se.k, se.picks + (int64_t)h * se.k, *se.pick_tag))
      *ra.fault = 1u;
  }
}

// The top-k and the ranking alone, where statistic and compaction follow in a launch of their own, side by side (28 heads, 6592 tokens, of
// which 6366 are kept: 36.1 us the layer step, with the statistic in this launch 36.9).  Dynamic LDS: kTailShortLds.
__global__ void __launch_bounds__(kTailThreads) tail_short_kernel(const float* s_all, int32_t* rank_row, SelectArgs se, int rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  const int b = (int)blockIdx.x;
  if (b < rows)
    select_short_body<kShortPer>(*reinterpret_cast<ShortSelectShared<kShortPer>*>(lds_dyn), se, b);
  else
    rank_short_body(*reinterpret_cast<ShortRankShared*>(lds_dyn), s_all, se.T, PutRank{rank_row}, b - rows);
}

// launch 0: the ranking's partition | top-k bound and filter (TILES tiles of a score row per workgroup).  64 registers, for two
// workgroups a unit where the grid has more than one for each.
template <int R, int TILES>
__global__ void __launch_bounds__(kTailThreads, 8) tail0_kernel(RankArgs ra, SelectArgs se) {
  __shared__ PartFilterShared sh;
  const int b = (int)blockIdx.x;
  if (b < ra.n_tiles) {
    partition_body<R>(sh.part, ra, b);
  } else {
    const int j = b - ra.n_tiles, per_row = (se.n_tiles + TILES - 1) / TILES;
    select_filter_body<kTailThreads, true, TILES>(sh.filter, se, j / per_row, (j % per_row) * TILES);
  }
}

// launch 1: top-k finish (one workgroup per score row, the longer ones, first) | the ranking's buckets;
// dynamic LDS for the larger of the two
__global__ void __launch_bounds__(kTailThreads, 8) tail1_kernel(RankArgs ra, SelectArgs se, int rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  const int b = (int)blockIdx.x;
  if (b < rows)
    select_finish_body(lds_dyn, se, b);
  else
    bucket_body(*reinterpret_cast<BucketShared*>(lds_dyn), ra, b - rows);
}

// launch 2: rank-variance statistic over the ring that now holds this layer's ranks (its first
// n_stat workgroups; workgroup 0 waits for the others) | KV compaction with the per-head indices of
// launch 1 (gx blocks per (head, tensor) slab)
template <bool POW2>
__global__ void __launch_bounds__(kVarThreads) tail2_kernel(RankvarArgs ra, int n_stat, GatherArgs ga, int gx, int Hk) {
  __shared__ RankvarShared<> sh;
  const int b = (int)blockIdx.x;
  if (b < n_stat) {
    if (ra.skip != 0) {
      if (threadIdx.x == 0) stat_skip_body(ra.out, ra.state, ra.layer_idx, ra.l_obs, ra.push);   // n_stat = 1
    } else {
      rankvar_body(sh, ra, b, n_stat);
    }
  } else {
    const int j = b - n_stat;
    const int bx = j % gx, hw = j / gx;
    gather_body<POW2, kVarThreads>(ga, bx, hw % Hk, hw / Hk, 0);
  }
}

// Launches 0 and 1.
static hipError_t launch_rank_select(const Workspace& ws, const SelectArgs& se, const RankArgs& ra, int rows, hipStream_t st) {
  constexpr size_t kMost = finish_lds_bytes(kSelCandCap) > sizeof(BucketShared) ? finish_lds_bytes(kSelCandCap) : sizeof(BucketShared);
  static OncePerDevice once;
  const hipError_t attr = allow_lds(once, reinterpret_cast<const void*>(tail1_kernel), kMost);
  if (attr != hipSuccess) return attr;
  const dim3 block(kTailThreads), grid1(rows + ra.n_buckets);
  // Tiles per filtering workgroup: as few as leave launch 0 one workgroup per compute unit; two on a unit slow down each
  // other's barriers and scans (launch 0 of the 8B shape: 128K 12.0 us with one tile each and 352 workgroups, 10.0 with
  // 208; 256K 18.6 us with 704, 15.0 with 208).
  auto grid0 = [&](int tiles) { return ra.n_tiles + rows * ((se.n_tiles + tiles - 1) / tiles); };
  const int tiles = grid0(1) <= kTailUnits ? 1 : grid0(2) <= kTailUnits ? 2 : kFilterMostTiles;
  auto launch0 = [&](auto r) {
    constexpr int R = decltype(r)::value;
    if constexpr (R < 8) {                              // the 8192-token tiles come with more than a unit's share of the filter's
      if (tiles == 1) {
        ASL_LAUNCH(ws.prof, kKernTail, st, (tail0_kernel<R, 1>), dim3(grid0(1)), block, 0, st, ra, se);
        return;
      }
      if (tiles == 2) {
        ASL_LAUNCH(ws.prof, kKernTail, st, (tail0_kernel<R, 2>), dim3(grid0(2)), block, 0, st, ra, se);
        return;
      }
    }
    ASL_LAUNCH(ws.prof, kKernTail, st, (tail0_kernel<R, 4>), dim3(grid0(4)), block, 0, st, ra, se);
  };
  if (ra.tile_log == 11)
    launch0(std::integral_constant<int, 2>());
  else if (ra.tile_log == 12)
    launch0(std::integral_constant<int, 4>());
  else
    launch0(std::integral_constant<int, 8>());
  const size_t fin = finish_lds_bytes(se.cand_cap), lds = fin > sizeof(BucketShared) ? fin : sizeof(BucketShared);
  ASL_LAUNCH(ws.prof, kKernTail, st, tail1_kernel, grid1, block, lds, st, ra, se, rows);
  return hipGetLastError();
}

// The last launch: statistic (or the note that it is not evaluated yet) beside the compaction, which may be
// absent (no output tensors).
static hipError_t launch_stat_gather(const Workspace& ws, const GatherArgs* gather, int Hk, const RankvarArgs& stat, hipStream_t st) {
  if (gather != nullptr) {
    GatherArgs ga = *gather;
    const bool pow2 = gather_prepare(ga);
    const int64_t total = (int64_t)ga.n_idx * ga.cpr;
    const int per_block = kVarThreads * kGatherUnroll;
    const int gx = (int)((total + per_block - 1) / per_block);
    const int n_stat = stat.skip != 0 ? 1 : rankvar_blocks(stat.T);
    const dim3 grid4(n_stat + gx * Hk * ga.n_tensors);
    if (gx == 0)
      ASL_LAUNCH(ws.prof, kKernRankvar, st, (tail2_kernel<true>), dim3(n_stat), dim3(kVarThreads), 0, st, stat, n_stat, ga, 1, Hk);
    else if (pow2)
      ASL_LAUNCH(ws.prof, kKernTail, st, (tail2_kernel<true>), grid4, dim3(kVarThreads), 0, st, stat, n_stat, ga, gx, Hk);
    else
      ASL_LAUNCH(ws.prof, kKernTail, st, (tail2_kernel<false>), grid4, dim3(kVarThreads), 0, st, stat, n_stat, ga, gx, Hk);
    return hipGetLastError();
  }
  if (stat.skip != 0) return launch_stat_skip(ws.prof, stat.out, stat.state, stat.layer_idx, stat.l_obs, stat.push, st);
  return launch_rankvar(ws, stat.ring, stat.l_obs, stat.T, stat.layer_idx, stat.k, stat.tau, stat.push, stat.state, stat.out, st);
}

bool tail_takes(const Workspace& ws, int rows, int T) { return rows <= ws.sel_rows && T <= kRankMaxT; }

hipError_t launch_tail(const Workspace& ws, const float* scores, int rows, int T, int k, int W, int32_t* rank_row,
                       int32_t* idx_out, const GatherArgs* gather, int Hk, bool have_sample, int S,
                       const RankvarArgs& stat, hipStream_t st, bool* taken) {
  *taken = false;
  if (!tail_takes(ws, rows, T)) return hipSuccess;
  if (gather != nullptr && ((int64_t)gather->n_idx * gather->cpr >= (int64_t(1) << 31))) return hipSuccess;
  *taken = true;
  const float* s_all = scores + (int64_t)(rows - 1) * T;       // the all-head row is the last one
  const SelectArgs se = select_args(ws, scores, T, k, W, idx_out, have_sample, S);
  hipError_t e;
  if (T <= kShortT) {
    const int n_rank = short_rank_blocks(T);
    GatherArgs ga = {};
    SelectArgs sp = se;
    int gx = 0, grid = rows + n_rank;
    bool pow2 = true, whole = true;
    if (gather != nullptr) {
      ga = *gather;
      pow2 = gather_prepare(ga);
      gx = (int)(((int64_t)ga.n_idx * ga.cpr + kTailThreads * kPickedUnroll - 1) / (kTailThreads * kPickedUnroll));
      whole = Hk <= ws.pick_rows && k <= kPickMost && short_whole(Hk, gx * ga.n_tensors);
      grid = short_gather_from(rows, n_rank) + kDies * ((Hk + kDies - 1) / kDies) * gx * ga.n_tensors;
      sp.picks = ws.sel_picks;
      sp.pick_tag = ws.pick_tag;
      sp.pick_rows = Hk;
    }
    if (whole) {
      const bool two = rows + n_rank > kTailUnits;      // two workgroups a unit
      auto* const kernel = two ? (pow2 ? tail_whole_kernel<true, 8> : tail_whole_kernel<false, 8>)
                               : (pow2 ? tail_whole_kernel<true, 4> : tail_whole_kernel<false, 4>);
      static OncePerDevice once[4];
      const hipError_t attr = allow_lds(once[2 * two + pow2], reinterpret_cast<const void*>(kernel), kTailShortLds);
      if (attr != hipSuccess) return attr;
      ASL_LAUNCH(ws.prof, kKernTail, st, kernel, dim3(grid), dim3(kTailThreads), kTailShortLds, st, s_all, rank_row, sp, rows, n_rank, stat, ga, gx, Hk);
      return hipGetLastError();
    }
    static OncePerDevice once;
    const hipError_t attr = allow_lds(once, reinterpret_cast<const void*>(tail_short_kernel), kTailShortLds);
    if (attr != hipSuccess) return attr;
    ASL_LAUNCH(ws.prof, kKernTail, st, tail_short_kernel, dim3(rows + n_rank), dim3(kTailThreads), kTailShortLds, st, s_all, rank_row, se, rows);
    e = hipGetLastError();
  } else {
    const uint32_t* sample = have_sample ? ws.sel_sample + (int64_t)(rows - 1) * kSelMaxSample : nullptr;
    const RankArgs ra = rank_args(ws, s_all, T, sample, rank_row);
    e = launch_rank_select(ws, se, ra, rows, st);
  }
  return e != hipSuccess ? e : launch_stat_gather(ws, gather, Hk, stat, st);
}

}  // namespace asl
