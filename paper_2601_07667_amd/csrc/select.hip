// asl_select: the k highest-scoring past tokens of each row, ties to the lower index, written in
// ascending token order and followed by the window tokens (Alg. 1 steps 9-10 per KV head;
// Alg. 2 steps 11-12 on the all-head scores).
//
// Exact selection in three small launches that read the scores once and never wait for each other:
//  1. guess    one workgroup per row looks at a strided sample of the row
//              and takes the sample's m-th smallest key (keys are an order-preserving transform of the scores,
//              ascending key = descending score) as a bound that, with m a few standard deviations
//              above the expected number of top-k members in the sample, admits at least k keys
//              of the row and not many more; the key as far on the other side says where the row's k-th is likely;
//  2. filter   one workgroup per tile of 4096 tokens keeps the tile's keys <= the bound, in token
//              order, in the tile's own segment of a candidate buffer (no offsets to agree on).  Where the pooling
//              kernel left the sample behind in compact form (layer steps), and for a few rows, the filter's workgroups
//              take the bound themselves and there is no launch 1;
//  3. finish   one workgroup per row loads the row's candidates (a few thousand) into LDS, finds
//              the k-th smallest key among them (finish_threshold), and writes the kept tokens in order.
// (With four radix passes for the bound and for the threshold instead of one histogram each, 256 rows of 131040 scores
// took 57.2 us, now 48.7; a layer step's tail with the bound in a launch of its own and the finish in another 37 us,
// now 26.)
// The bound is only a guess: if more candidates passed it than step 3 has room for, it tightens the bound by a histogram of them; if
// fewer than k keys passed it, or a tile's candidates do not fit their segment, it runs the same selection over the whole row
// straight from the scores instead (slower, same result).  The result therefore never depends on the sample.
// Rows of at most kSelMidT scores (many rows: kSelShortT; in a layer step: kShortT) need no bound: one launch, one workgroup per row, all tokens in LDS.
// Integer work throughout: nothing depends on scheduling.
#include "select_body.h"

namespace asl {

__global__ void __launch_bounds__(kFinThreads) select_guess_kernel(SelectArgs a) {
  __shared__ GuessShared sh;
  select_guess_body(sh, a, (int)blockIdx.x);
}

// grid: x = tile, y = row.  Small workgroups: one lives ~5 us whatever its size, and more of them in flight stream faster (us, with
// 1024 threads and so: 32 rows of 200001 scores 22.9, 21.5; 64 of 100001 20.7, 19.3; 130 of 40000 22.2, 20.8).
__global__ void __launch_bounds__(kFilterThreads) select_filter_kernel(SelectArgs a) {
  __shared__ FilterShared<false> sh;
  select_filter_body<kFilterThreads, false>(sh, a, (int)blockIdx.y, (int)blockIdx.x);
}

// Steps 1 and 2 of a few rows, with one workgroup or less for each compute unit: every workgroup takes its row's bound itself, beside
// the loads of its TILES tiles, which saves a launch (us, so and with it: one row of 131040 scores 12.5, 13.9; 8 rows of 20000 14.3,
// 16.0; 8 of 262080 17.3, 18.2; but four tiles a workgroup, 32 rows of 131040, 22.6, 19.6, and two workgroups a unit, 9 rows, 16.8, 16.1).
constexpr long kOwnBoundMost = 256;
template <int TILES>
__global__ void __launch_bounds__(kFinThreads) select_bound_filter_kernel(SelectArgs a) {
  __shared__ FilterShared<true> sh;
  select_filter_body<kFinThreads, true, TILES, false>(sh, a, (int)blockIdx.y, (int)blockIdx.x * TILES);
}

// dynamic LDS: finish_lds_bytes(a.cand_cap)
__global__ void __launch_bounds__(kFinThreads, 8) select_finish_kernel(SelectArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  select_finish_body(lds_dyn, a, (int)blockIdx.x);
}

// dynamic LDS: sizeof(ShortSelectShared<PER>)
template <int PER>
__global__ void __launch_bounds__(kFinThreads) select_short_kernel(SelectArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  select_short_body<PER>(*reinterpret_cast<ShortSelectShared<PER>*>(lds_dyn), a, (int)blockIdx.x);
}
template <int PER>
static hipError_t launch_select_short(Prof* prof, const SelectArgs& a, int rows, hipStream_t st) {
  constexpr size_t lds = sizeof(ShortSelectShared<PER>);
  static OncePerDevice once;
  const hipError_t attr = allow_lds(once, reinterpret_cast<const void*>(select_short_kernel<PER>), lds);
  if (attr != hipSuccess) return attr;
  ASL_LAUNCH(prof, kKernSelWrite, st, select_short_kernel<PER>, dim3(rows), dim3(kFinThreads), lds, st, a);
  return hipGetLastError();
}

SelectArgs select_args(const Workspace& ws, const float* scores, int T, int k, int W, int32_t* idx_out,
                       bool have_sample, int S) {
  SelectArgs a = {};
  a.scores = scores;
  a.sample = have_sample ? ws.sel_sample : nullptr;
  a.T = T;
  a.n_tiles = (T + kSelTile - 1) / kSelTile;
  a.k = k;
  a.W = W;
  const int run = have_sample ? 1 : kSelSampleRun;
  a.stride = sel_sample_stride(T);
  a.n_s = sel_sample_size(T) / run * run;
  a.m = sel_sample_rank(T, k, a.n_s, run);
  a.slack = sel_bound_slack(T, a.m, a.n_s, run);
  a.m_low = sel_sample_rank_low(T, k, a.n_s, run);
  a.cand_cap = sel_cand_cap(T, a.m, a.slack, a.n_s, have_sample ? sel_sample_alike(T, S) : run);
  a.bound = ws.sel_bound;
  a.cand = ws.sel_cand;
  a.seg_count = ws.sel_seg_count;
  a.idx_out = idx_out;
  return a;
}

hipError_t launch_select(const Workspace& ws, const float* scores, int rows, int T, int k, int W,
                         int32_t* idx_out, hipStream_t st) {
  static OncePerDevice once;
  const hipError_t attr = allow_lds(once, reinterpret_cast<const void*>(select_finish_kernel), finish_lds_bytes(kSelCandCap));
  if (attr != hipSuccess) return attr;
  // rows beyond what the candidate buffers hold at once take further rounds of the three launches
  const int rows_per_round = ws.sel_rows;
  for (int row0 = 0; row0 < rows; row0 += rows_per_round) {
    const int nr = rows - row0 < rows_per_round ? rows - row0 : rows_per_round;
    const SelectArgs a = select_args(ws, scores + (int64_t)row0 * T, T, k, W, idx_out + (int64_t)row0 * (k + W), false, 1);
    if (T <= kSelMidT || (T <= kSelShortT && rows >= kSelShortRows)) {
      const hipError_t e = T <= kShortT ? launch_select_short<kShortT / kFinThreads>(ws.prof, a, nr, st)
                                        : launch_select_short<kSelShortT / kFinThreads>(ws.prof, a, nr, st);
      if (e != hipSuccess) return e;
      continue;
    }
    const dim3 fgrid(a.n_tiles, nr), two((a.n_tiles + 1) / 2, nr);
    if ((long)a.n_tiles * nr <= kOwnBoundMost) {
      ASL_LAUNCH(ws.prof, kKernSelHist, st, select_bound_filter_kernel<1>, fgrid, dim3(kFinThreads), 0, st, a);
    } else if ((long)two.x * nr <= kOwnBoundMost) {
      ASL_LAUNCH(ws.prof, kKernSelHist, st, select_bound_filter_kernel<2>, two, dim3(kFinThreads), 0, st, a);
    } else {
      ASL_LAUNCH(ws.prof, kKernSelHist, st, select_guess_kernel, dim3(nr), dim3(kFinThreads), 0, st, a);
      ASL_LAUNCH(ws.prof, kKernSelHist, st, select_filter_kernel, fgrid, dim3(kFilterThreads), 0, st, a);
    }
    ASL_LAUNCH(ws.prof, kKernSelWrite, st, select_finish_kernel, dim3(nr), dim3(kFinThreads), finish_lds_bytes(a.cand_cap), st, a);
  }
  return hipGetLastError();
}

}  // namespace asl
