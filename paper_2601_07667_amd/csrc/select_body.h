// Device code of asl_select's three kernels (see select.hip for the method), written as functions
// over explicit shared-state structs so that another kernel can host them beside a second body.
#pragma once
#include "sample_body.h"

namespace asl {

constexpr int kFinThreads = kRowThreads;               // workgroup of the other kernels
constexpr int kFinWaves = kFinThreads / 64;
constexpr int kFilterThreads = 256;                    // filter workgroup of its own launch
constexpr int kFilterMostTiles = 4;                    // most tiles of one workgroup that takes the bound itself
constexpr uint32_t kSegOverflow = 0xffffffffu;         // a tile's count when its segment was too small
static_assert(kSelTile % kFinThreads == 0 && kSelTile % kFilterThreads == 0, "filter tile geometry");

static_assert(kSelMaxSample % kFinThreads == 0, "the bound kernel's threads share the sample evenly");

// Radix select over n keys read through `key_at(i)`: returns the k-th smallest key (1 <= k <= n)
// and how many of the keys equal to it belong to the k smallest (k_rem >= 1).  All kFinThreads
// threads take part.  The keys' common leading bits are skipped: digits are taken from
// key - min over the bits in which min and max differ, so the first digit already spreads the keys
// over the bins (scores of one row share their sign and most of their exponent).
// h: kHistWords-word LDS histogram (bank-staggered copies), sm: >= 2 * kFinWaves + 2 words.
constexpr int kSelBatch = 4;                           // keys a thread reads together in the selection loops
template <typename KeyAt>
__device__ __forceinline__ void radix_select_block(int n, uint32_t k, KeyAt key_at, uint32_t* h, uint32_t* sm,
                                                   uint32_t& thr_out, uint32_t& k_rem_out) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // The loops over the keys take kSelBatch of a thread's keys at a time (positions past the end
  // re-read the thread's first key of the batch), so that their reads are in flight together.
  uint32_t lo = 0xffffffffu, hi = 0u;
  for (int i0 = tid; i0 < n; i0 += kSelBatch * kFinThreads) {
    uint32_t key[kSelBatch];
#pragma unroll
    for (int u = 0; u < kSelBatch; ++u) key[u] = key_at(i0 + u * kFinThreads < n ? i0 + u * kFinThreads : i0);
#pragma unroll
    for (int u = 0; u < kSelBatch; ++u) {
      lo = key[u] < lo ? key[u] : lo;
      hi = key[u] > hi ? key[u] : hi;
    }
  }
  lo = wave_min(lo);
  hi = wave_max(hi);
  __syncthreads();                                     // sm may still be in use
  if (lane == 0) {
    sm[wave] = lo;
    sm[kFinWaves + wave] = hi;
  }
  __syncthreads();
  for (int w = 0; w < kFinWaves; ++w) {
    const uint32_t l2 = sm[w], h2 = sm[kFinWaves + w];
    lo = l2 < lo ? l2 : lo;
    hi = h2 > hi ? h2 : hi;
  }
  const uint32_t span = hi - lo;
  const int bits = span == 0 ? 0 : 32 - __clz((int)span);
  const int n_pass = (bits + 7) / 8;                   // uniform; 0 when all keys are equal
  uint32_t prefix = 0, k_rem = k;
  for (int pass = 0; pass < n_pass; ++pass) {
    const int shift = 8 * (n_pass - 1 - pass);
    __syncthreads();                                   // h and sm of the previous pass are consumed
    hist_clear(h, tid, kFinThreads);
    __syncthreads();
    for (int i0 = tid; i0 < n; i0 += kSelBatch * kFinThreads) {
      uint32_t v[kSelBatch];
#pragma unroll
      for (int u = 0; u < kSelBatch; ++u) v[u] = key_at(i0 + u * kFinThreads < n ? i0 + u * kFinThreads : i0) - lo;
#pragma unroll
      for (int u = 0; u < kSelBatch; ++u)
        if (i0 + u * kFinThreads < n && (pass == 0 || (v[u] >> (shift + 8)) == prefix)) hist_add(h, tid, (v[u] >> shift) & 255u);
    }
    __syncthreads();
    // exclusive scan of the 256 counts by the first four wavefronts; the digit d with
    // excl < k_rem <= excl + count holds the k-th key
    uint32_t cnt = 0, incl = 0;
    if (tid < 256) {
      cnt = hist_total(h, tid);
      incl = wave_prefix_sum(cnt);
      if (lane == 63) sm[wave] = incl;
    }
    if (tid == 0) {
      sm[4] = 0;                                       // defined even if no digit qualifies
      sm[5] = 1;                                       // (cannot happen while 1 <= k <= n)
    }
    __syncthreads();
    if (tid < 256) {
      uint32_t excl = incl - cnt;
      for (int w = 0; w < wave; ++w) excl += sm[w];
      if (excl < k_rem && excl + cnt >= k_rem) {       // exactly one digit satisfies this
        sm[4] = (uint32_t)tid;
        sm[5] = k_rem - excl;
      }
    }
    __syncthreads();
    prefix = (prefix << 8) | sm[4];
    k_rem = sm[5];
  }
  thr_out = lo + prefix;
  k_rem_out = k_rem;
}

struct SelectArgs {
  const float* scores;           // [rows][T]
  const uint32_t* sample;        // [rows][kSelMaxSample] keys at the sample positions, or null
  int T, n_tiles, k, W;
  int n_s, stride;               // the sample: keys and the stride between their positions
  int m, slack;                  // rank of the bound in the sample, sample keys it may let pass beyond (see select_bound.h)
  int m_low;                     // rank of a sample key that is hardly behind the row's k-th
  int cand_cap;                  // candidates of one row that step 3 holds in LDS
  uint32_t* bound;               // [rows][2] the bound, and a key that the k-th is hardly below
  uint2* cand;                   // [rows][n_tiles][kSelSegment] (key, token)
  uint32_t* seg_count;           // [rows][n_tiles]
  int32_t* idx_out;              // [rows][k + W]
  // where a launch compacts the rows' keys and values too (gather_picked_body): the first pick_rows rows' tokens for its
  // other workgroups, each in a word with the launch's tag
  unsigned long long* picks;     // [pick_rows][k]
  const uint32_t* pick_tag;
  int pick_rows;                 // 0: none
};

struct GuessShared {
  SampleShared s;
};

// The row's bound and the key the threshold is looked for from, from the sample keys v.
__device__ __forceinline__ void select_bound(SampleShared& sh, const SelectArgs& a, const uint32_t (&v)[kSamplePer], uint32_t& bound,
                                             uint32_t& below) {
  bound = 0xffffffffu;
  below = 0u;
  if (a.m < a.n_s) sample_bound(sh, v, a.n_s, (uint32_t)a.m, (uint32_t)a.m_low, (uint32_t)a.slack, bound, below);   // uniform
}

// The sample of a row that nobody left one of: runs of kSelSampleRun neighbouring keys.
__device__ __forceinline__ void load_runs(const float* sr, int n_s, int stride, uint32_t (&v)[kSamplePer]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < kSamplePer; ++u) {               // key j = member j % run of run j / run, whose place is scattered
    const uint32_t j = (uint32_t)min(tid + u * kFinThreads, n_s - 1);
    v[u] = order_key(sr[kSelSampleRun * sel_sample_position(j / kSelSampleRun, stride) + j % kSelSampleRun]);
  }
}

// Step 1 on its own.
__device__ __forceinline__ void select_guess_body(GuessShared& sh, const SelectArgs& a, int row) {
  const int tid = threadIdx.x;
  uint32_t v[kSamplePer];
  load_runs(a.scores + (int64_t)row * a.T, a.n_s, a.stride, v);
  uint32_t bound, below;
  select_bound(sh.s, a, v, bound, below);
  if (tid == 0) {
    a.bound[2 * row] = bound;
    a.bound[2 * row + 1] = below;
  }
}

// key(score) <= bound, decided on the score's bits without forming the key: non-negative scores
// (bits u < 2^31) have key 2^31 - 1 - u, negative ones key u, and -0 counts as +0.  So for a bound
// below 2^31 - 1 exactly the bits in [2^31 - 1 - bound, 2^31 - 1] pass, and for any other bound the
// bits in [0, max(bound, 2^31)] (every non-negative score, -0, and the negative ones up to the
// bound): one subtraction and one unsigned comparison per score.
struct KeepTest {
  uint32_t lo, span;
};
__device__ __forceinline__ KeepTest keep_test(uint32_t bound) {
  KeepTest t;
  if (bound >= 0x7fffffffu) {
    t.lo = 0u;
    t.span = bound > 0x80000000u ? bound : 0x80000000u;
  } else {
    t.lo = 0x7fffffffu - bound;
    t.span = bound;
  }
  return t;
}
__device__ __forceinline__ bool keeps(const KeepTest& t, float score) { return (__float_as_uint(score) - t.lo) <= t.span; }

template <bool INSIDE> struct FilterShared {
  uint32_t wave_tot[1][kFinWaves];
};
template <> struct FilterShared<true> {
  uint32_t wave_tot[kFilterMostTiles][kFinWaves];
  SampleShared s;
};

// Step 2: the tile's keys <= bound, in token order, to the tile's segment of the candidate buffer.
// NT threads per workgroup: each wavefront takes kSelTile / (NT / 64) consecutive tokens.
// On its own a lane reads one score per load: what a ballot says of 64 neighbours is their order, and a kept token is what its
// lane holds.  Four at a time took a loop over each lane's kept ones, as often as the busiest lane has any, with a choice among four
// registers in it: 256 rows of 131040 scores 49.9 us, so 44.4; 64 rows 25.2, 21.8; 256 of 40000 29.6, 26.3 (counts of four
// rounds packed into two prefix sums, the kept scores read again: 53.9).  Inside a layer step, one round a tile, four with one 16-byte load, on
// whatever 4-byte boundary the row starts (8 heads, 32K 59.9, one per load 60.3).
// INSIDE (NT = kFinThreads): the workgroup takes the bound (step 1) beside its own loads, from a sample that is there in compact
// form (SAMPLED) or from the row; the row's first one stores it for step 3.  TILES: consecutive tiles of a workgroup,
// from `tile` on: a bound costs as much as two of them.
template <int NT, bool INSIDE, int TILES = 1, bool SAMPLED = true>
__device__ __forceinline__ void select_filter_body(FilterShared<INSIDE>& sh, const SelectArgs& a, int row, int tile) {
  constexpr int kWaves = NT / 64, kSelPerWave = kSelTile / kWaves;
  constexpr int kPer = INSIDE && SAMPLED ? 4 : 1;                  // neighbouring tokens per lane and round
  typedef float Four __attribute__((ext_vector_type(4), aligned(4)));
  constexpr int kSelRounds = kSelPerWave / (64 * kPer);
  static_assert(kSelRounds >= 1 && (TILES == 1 || INSIDE) && TILES <= kFilterMostTiles, "filter tile geometry");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, T = a.T;
  const float* sr = a.scores + (int64_t)row * T;
  const int base = tile * kSelTile + wave * kSelPerWave;     // of the first tile
  float sc[TILES][kSelRounds][kPer];
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
#pragma unroll
    for (int r = 0; r < kSelRounds; ++r) {             // all loads in flight before the first use
      const int e = base + i * kSelTile + (r * 64 + lane) * kPer;
      if constexpr (kPer == 4) {
        Four v = {0.f, 0.f, 0.f, 0.f};
        if (e + 3 < T) {
          v = *reinterpret_cast<const Four*>(sr + e);
        } else {                                        // the row's last, partial piece
          if (e < T) v.x = sr[e];
          if (e + 1 < T) v.y = sr[e + 1];
          if (e + 2 < T) v.z = sr[e + 2];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) sc[i][r][j] = v[j];
      } else {
        sc[i][r][0] = (e < T) ? sr[e] : 0.f;
      }
    }
  }
  uint32_t bound, below;
  if constexpr (INSIDE) {
    static_assert(NT == kFinThreads, "the sample is shared out among kFinThreads threads");
    uint32_t v[kSamplePer];
    if constexpr (SAMPLED)
      load_sample(nullptr, a.sample + (int64_t)row * kSelMaxSample, a.n_s, a.stride, v);
    else
      load_runs(sr, a.n_s, a.stride, v);
    select_bound(sh.s, a, v, bound, below);
    if (tile == 0 && tid == 0) {
      a.bound[2 * row] = bound;
      a.bound[2 * row + 1] = below;
    }
  } else {
    bound = a.bound[2 * row];
  }
  const KeepTest kt = keep_test(bound);
  // per round: which of the lane's tokens are kept (bit j), how many lower lanes keep, the round's total
  uint32_t kept[TILES][kSelRounds], before[TILES][kSelRounds], round_tot[TILES][kSelRounds];
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    uint32_t w_cnt = 0;
#pragma unroll
    for (int r = 0; r < kSelRounds; ++r) {
      const int e0 = base + i * kSelTile + (r * 64 + lane) * kPer;
      kept[i][r] = 0;
      before[i][r] = 0;
      round_tot[i][r] = 0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        const bool keep = (e0 + j < T) && keeps(kt, sc[i][r][j]);
        const uint64_t bal = __ballot(keep);
        kept[i][r] |= keep ? (1u << j) : 0u;
        before[i][r] += lanes_below(bal);
        round_tot[i][r] += (uint32_t)__popcll(bal);
      }
      w_cnt += round_tot[i][r];
    }
    if (lane == 0) sh.wave_tot[i][wave] = w_cnt;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    if (tile + i >= a.n_tiles) break;                   // uniform
    uint32_t run = 0, total = 0;
    for (int w = 0; w < kWaves; ++w) {
      run += (w < wave) ? sh.wave_tot[i][w] : 0u;
      total += sh.wave_tot[i][w];
    }
    const int64_t seg = ((int64_t)row * a.n_tiles + tile + i);
    if (tid == 0) a.seg_count[seg] = (total > (uint32_t)kSelSegment) ? kSegOverflow : total;
    if (total > (uint32_t)kSelSegment) continue;        // uniform: the finish step takes the whole row instead
    uint2* cand = a.cand + seg * kSelSegment;
#pragma unroll
    for (int r = 0; r < kSelRounds; ++r) {
      // token order inside a round: lane by lane, a lane's kPer tokens in a row.  Few tokens are kept:
      // the loop runs as often as the busiest lane has kept tokens.
      const int e0 = base + i * kSelTile + (r * 64 + lane) * kPer;
      uint32_t pos = run + before[i][r], m = kept[i][r];
      while (m != 0u) {
        const int j = __ffs((int)m) - 1;
        const float f = (j == 0) ? sc[i][r][0] : (j == 1) ? sc[i][r][1 % kPer] : (j == 2) ? sc[i][r][2 % kPer] : sc[i][r][3 % kPer];
        cand[pos] = make_uint2(order_key(f), (uint32_t)(e0 + j));
        ++pos;
        m &= m - 1u;
      }
      run += round_tot[i][r];
    }
  }
}

// Ordered write of the kept elements of a sequence of n (key, token) pairs given in token order:
// kept = key < thr, or key == thr and fewer than k_rem equal keys precede it.
// PER consecutive elements per thread and round.
// load(i0, key): the keys of elements i0 .. i0 + PER - 1; those from n on may be anything.  put(pos, token).
template <int PER, typename Load, typename TokAt, typename Put>
__device__ __forceinline__ void ordered_write(int n, uint32_t thr, uint32_t k_rem, int k, Load load, TokAt tok_at,
                                              uint32_t* red, Put put) {
  const int tid = threadIdx.x;
  static_assert(kFinThreads * PER < 65536, "a round's two counts share a word");
  uint32_t lt_base = 0, eq_base = 0;
  for (int c0 = 0; c0 < n; c0 += kFinThreads * PER) {
    const int i0 = c0 + tid * PER;
    uint32_t key[PER];
    uint32_t cnt = 0;                                  // keys below the threshold | keys equal to it << 16
    if (i0 < n) load(i0, key);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      cnt += (i0 + j < n && key[j] < thr) ? 1u : 0u;
      cnt += (i0 + j < n && key[j] == thr) ? 65536u : 0u;
    }
    uint32_t excl, total, none;
    block_scan<true>(red, cnt, 0u, excl, total, none);
    uint32_t lt_run = lt_base + (excl & 0xffffu), eq_run = eq_base + (excl >> 16);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (i0 + j < n) {
        const bool is_lt = key[j] < thr, is_eq = key[j] == thr;
        if (is_lt || (is_eq && eq_run < k_rem)) {
          const uint32_t pos = lt_run + (eq_run < k_rem ? eq_run : k_rem);
          if (pos < (uint32_t)k) put(pos, (uint32_t)tok_at(i0 + j));      // always true for consistent counts
        }
        lt_run += is_lt ? 1u : 0u;
        eq_run += is_eq ? 1u : 0u;
      }
    }
    lt_base += total & 0xffffu;
    eq_base += total >> 16;
  }
}

// Shared state of step 3; a.cand_cap candidate keys, then as many candidate tokens, follow it in
// the workgroup's dynamic LDS.
constexpr int kFinBins = 2 * kFinThreads;               // two per thread
constexpr int kFinBinBits = 11;
constexpr uint32_t kFinListMax = 64;
static_assert(kFinBins == 1 << kFinBinBits && kFinBins <= kHistWords, "the bins share the histogram's memory");
// Shared words of a search by bins.
struct BinPick {
  uint32_t list[kFinListMax];
  uint32_t pick[4];                                    // the bin that holds the key looked for, its place there, keys in the bin; keys listed
};
struct FinishShared {
  uint32_t h[kHistWords];
  uint32_t sm[2 * kFinWaves + 2];
  BinPick bins;
  uint32_t seg_off[kSelMaxRowTiles + 1];
  int whole_row;                                       // 1: select from the scores; kTooMany: the candidates do not fit
};
constexpr int kTooMany = 2;
constexpr size_t finish_lds_bytes(int cand_cap) { return (sizeof(FinishShared) + 15) / 16 * 16 + 2 * (size_t)cand_cap * sizeof(uint32_t); }
__device__ __forceinline__ uint32_t* finish_cand(void* lds) {
  return reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(lds) + (sizeof(FinishShared) + 15) / 16 * 16);
}

// Step 3 begins with the offsets of the tiles' candidates in the row's candidate sequence and, unless the
// whole row has to be taken instead (sh.whole_row), the candidates copied into LDS.  Returns the
// number of candidates.
__device__ __forceinline__ int finish_load(FinishShared& sh, uint32_t* lds_cand, const SelectArgs& a, int row) {
  const int tid = threadIdx.x, n_tiles = a.n_tiles, k = a.k, wave = uniform_wave(), lane = tid & 63;
  uint32_t c = 0;                                       // thread t takes tile t's count
  if (tid < n_tiles && n_tiles <= kSelMaxRowTiles) c = a.seg_count[(int64_t)row * n_tiles + tid];
  sh.h[2 * tid] = 0;                                    // finish_threshold's bins
  sh.h[2 * tid + 1] = 0;
  if (tid == 0) sh.bins.pick[3] = 0;
  {
    const uint32_t over = (c == kSegOverflow) ? 1u : 0u;
    c = over ? 0u : c;
    uint32_t c_excl, c_tot, any_over;
    block_scan<true>(sh.sm, c, over, c_excl, c_tot, any_over);
    if (tid < n_tiles && n_tiles <= kSelMaxRowTiles) sh.seg_off[tid] = c_excl;
    if (tid == 0) {
      if (n_tiles <= kSelMaxRowTiles) sh.seg_off[n_tiles] = c_tot;
      sh.whole_row = (n_tiles > kSelMaxRowTiles || any_over != 0 || c_tot < (uint32_t)k) ? 1 : c_tot > (uint32_t)a.cand_cap ? kTooMany : 0;
    }
  }
  __syncthreads();
  if (sh.whole_row) return 0;                          // uniform
  uint32_t* lk = lds_cand;
  uint32_t* li = lds_cand + a.cand_cap;
  // Wavefront w copies tiles w, w + kFinWaves, ..., two tiles and kBatch candidates of each at a time, whose loads
  // are in flight together (a tile holds ~100 candidates at the usual budgets, ~400 at the largest).
  constexpr int kDeep = 4, kBatch = 64 * kDeep;
  const uint2* row_cand = a.cand + (int64_t)row * n_tiles * kSelSegment;
  for (int t0 = wave; t0 < n_tiles; t0 += 2 * kFinWaves) {
    uint32_t o[2], n[2];
    const uint2* seg[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int t = t0 + q * kFinWaves;
      const bool in = t < n_tiles;
      o[q] = in ? sh.seg_off[t] : 0u;
      n[q] = in ? sh.seg_off[t + 1] - o[q] : 0u;
      seg[q] = row_cand + (int64_t)(in ? t : 0) * kSelSegment;
    }
    const uint32_t n_max = n[0] > n[1] ? n[0] : n[1];
    for (uint32_t j0 = 0; j0 < n_max; j0 += kBatch) {
      uint2 x[2][kDeep];
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
          const uint32_t j = j0 + u * 64 + lane;
          x[q][u] = make_uint2(0u, 0u);
          if (j < n[q]) x[q][u] = seg[q][j];
        }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
          const uint32_t j = j0 + u * 64 + lane;
          if (j < n[q]) {
            lk[o[q] + j] = x[q][u].x;
            li[o[q] + j] = x[q][u].y;
          }
        }
    }
  }
  __syncthreads();
  return (int)sh.seg_off[n_tiles];
}

// The k_rem-th smallest of the c <= kFinListMax listed keys, and (k_rem) how many of those equal to it are kept.  Every
// wavefront for itself.
__device__ __forceinline__ void pick_listed(const uint32_t* list, uint32_t c, uint32_t& thr, uint32_t& k_rem) {
  const int lane = threadIdx.x & 63;
  const uint32_t key = list[min((uint32_t)lane, c - 1u)];
  uint32_t less = 0, same = 0;
  for (uint32_t j = 0; j < c; ++j) {
    const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)key, (int)j);
    less += x < key ? 1u : 0u;
    same += x == key ? 1u : 0u;
  }
  const uint64_t hit = __ballot((uint32_t)lane < c && less < k_rem && k_rem <= less + same);
  const int who = hit != 0ull ? __ffsll((unsigned long long)hit) - 1 : 0;    // never zero
  thr = (uint32_t)__builtin_amdgcn_readlane((int)key, who);
  k_rem -= (uint32_t)__builtin_amdgcn_readlane((int)less, who);
}

// PER bins per thread (their counts: c) with `excl` keys before the thread's: which holds the kk-th key?
template <int PER>
__device__ __forceinline__ void pick_bin(BinPick& sh, const uint32_t (&c)[PER], uint32_t excl, uint32_t kk) {
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (excl < kk && kk <= excl + c[q]) {               // one bin of the workgroup, if any
      sh.pick[0] = (uint32_t)(PER * (int)threadIdx.x + q);
      sh.pick[1] = kk - excl;
      sh.pick[2] = c[q];
    }
    excl += c[q];
  }
  __syncthreads();
}

// More candidates than fit: they are counted in the bins between `below` and the bound, where they lie, and those up to the end of the
// bin that holds the k-th, which is the bound from here on, are collected.  Returns how many; sh.whole_row 1 where that does not help.
// (By the radix select over all scores such a row took 220 us; k = 8160, where the bound has to be wide, 9 rows of 200001 243.5 us,
// so 32.3; 32 of 262080 320, 39; 256 of 131040, a few of which have too many, 167, 64.)
__device__ __forceinline__ int finish_tighten(FinishShared& sh, uint32_t* lds_cand, const SelectArgs& a, int row, uint32_t& bound, uint32_t below) {
  const int tid = threadIdx.x, n_tiles = a.n_tiles, wave = uniform_wave(), lane = tid & 63;
  const uint32_t kk = (uint32_t)a.k;
  const uint2* row_cand = a.cand + (int64_t)row * n_tiles * kSelSegment;
  const uint32_t* counts = a.seg_count + (int64_t)row * n_tiles;
  const int shift = bin_shift(below, bound, kFinBinBits);
  uint32_t lower = 0;
  for (int t = wave; t < n_tiles; t += kFinWaves) {
    const uint32_t n = counts[t];
    const uint2* seg = row_cand + (int64_t)t * kSelSegment;
    for (uint32_t j0 = 0; j0 < n; j0 += 256) {
      uint32_t key[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) key[u] = seg[min(j0 + 64 * u + lane, n - 1)].x;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (j0 + 64 * u + lane < n) {
          if (key[u] < below)
            ++lower;
          else
            atomicAdd(&sh.h[clamped_bin(key[u], below, bound, shift)], 1u);
        }
    }
  }
  __syncthreads();
  const uint32_t c[2] = {sh.h[2 * tid], sh.h[2 * tid + 1]};
  uint32_t excl, total;
  block_scan<false>(sh.sm, c[0] + c[1], lower, excl, total, lower);
  if (tid == 0) sh.bins.pick[2] = 0;
  __syncthreads();
  pick_bin<2>(sh.bins, c, lower + excl, kk);
  const uint32_t d = sh.bins.pick[0], n_new = kk - sh.bins.pick[1] + sh.bins.pick[2];
  const bool fits = lower < kk && sh.bins.pick[2] != 0 && n_new <= (uint32_t)a.cand_cap;
  if (!fits) {                                          // uniform
    __syncthreads();
    if (tid == 0) sh.whole_row = 1;
    __syncthreads();
    return 0;
  }
  const uint32_t from = below + (d << shift), width = (1u << shift) - 1u;
  bound = bound - from < width ? bound : from + width;
  // the tiles' candidates up to the new bound: how many, then where
  for (int t = wave; t < n_tiles; t += kFinWaves) {
    const uint32_t n = counts[t];
    const uint2* seg = row_cand + (int64_t)t * kSelSegment;
    uint32_t held = 0;
    for (uint32_t j0 = 0; j0 < n; j0 += 256) {
      uint32_t key[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) key[u] = seg[min(j0 + 64 * u + lane, n - 1)].x;
#pragma unroll
      for (int u = 0; u < 4; ++u) held += (uint32_t)__popcll(__ballot(j0 + 64 * u + lane < n && key[u] <= bound));
    }
    if (lane == 0) sh.seg_off[t] = held;
  }
  __syncthreads();
  uint32_t c_excl, c_tot, none;
  block_scan<false>(sh.sm, tid < n_tiles ? sh.seg_off[tid] : 0u, 0u, c_excl, c_tot, none);
  if (tid < n_tiles) sh.seg_off[tid] = c_excl;
  if (tid == 0) {
    sh.seg_off[n_tiles] = c_tot;
    sh.whole_row = 0;
    sh.bins.pick[3] = 0;
  }
  sh.h[2 * tid] = 0;                                    // the bins again
  sh.h[2 * tid + 1] = 0;
  __syncthreads();
  uint32_t* lk = lds_cand;
  uint32_t* li = lds_cand + a.cand_cap;
  for (int t = wave; t < n_tiles; t += kFinWaves) {
    const uint32_t n = counts[t];
    const uint2* seg = row_cand + (int64_t)t * kSelSegment;
    uint32_t at = sh.seg_off[t];
    for (uint32_t j0 = 0; j0 < n; j0 += 256) {
      uint2 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = seg[min(j0 + 64 * u + lane, n - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool keep = j0 + 64 * u + lane < n && x[u].x <= bound;
        const uint64_t bal = __ballot(keep);
        const uint32_t i = min(at + lanes_below(bal), (uint32_t)a.cand_cap - 1u);   // smaller by itself
        if (keep) {
          lk[i] = x[u].x;
          li[i] = x[u].y;
        }
        at += (uint32_t)__popcll(bal);
      }
    }
  }
  __syncthreads();
  return (int)min(sh.seg_off[n_tiles], (uint32_t)a.cand_cap);
}

// f(key, valid) for the thread's of n keys in LDS, four reads at a time, as often for every thread of a wavefront.
template <typename F>
__device__ __forceinline__ void each_key(const uint32_t* keys, int n, F f) {
  for (int i0 = (int)threadIdx.x; __builtin_amdgcn_readfirstlane(i0) < n; i0 += 4 * kFinThreads) {
    uint32_t k[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) k[q] = keys[min(i0 + q * kFinThreads, n - 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) f(k[q], i0 + q * kFinThreads < n);
  }
}
// Counts the keys in [lo, hi] in bins of width 2^shift from lo, where many want the same.
__device__ __forceinline__ void count_repeated(const uint32_t* keys, int n, uint32_t lo, uint32_t hi, int shift, const Repeated& rep, uint32_t* bin) {
  each_key(keys, n, [&](uint32_t k, bool valid) {
    const uint32_t add = add_for(rep, (k - lo) >> shift, valid && k - lo <= hi - lo);
    if (add != 0u) atomicAdd(&bin[(k - lo) >> shift], add);
  });
}

// The k_rem-th smallest of the keys in [from, to], of which there are more than kFinListMax, and (k_rem) how many of those equal
// to it are kept.  keys: all n in LDS; bin: PER * kFinThreads words.  The range is cut into bins between the smallest and
// the largest key in it, then the bin that holds the key looked for, until that is one key or has few enough
// to compare: at most three times, ~2 us each.
template <int PER>
__device__ __forceinline__ void zoom_threshold(BinPick& sh, uint32_t* red, uint32_t* bin, const uint32_t* keys, int n, uint32_t from, uint32_t to,
                                               uint32_t& thr, uint32_t& k_rem) {
  constexpr int kBits = PER == 4 ? 12 : 11;
  static_assert(PER * kFinThreads == 1 << kBits, "bins");
  const int tid = threadIdx.x;
  auto each = [&](auto f) { each_key(keys, n, f); };
  for (;;) {
    uint32_t lo = 0xffffffffu, hi = 0u;
    each([&](uint32_t k, bool) {
      const bool in = k - from <= to - from;
      lo = min(lo, in ? k : 0xffffffffu);
      hi = max(hi, in ? k : 0u);
    });
#pragma unroll
    for (int q = 0; q < PER; ++q) bin[q * kFinThreads + tid] = 0u;
    block_min_max(red, lo, hi);
    thr = lo;
    if (lo >= hi) return;                               // uniform: one key
    const int shift = bin_shift(lo, hi, kBits);
    const uint32_t one = keys[min(tid, n - 1)];
    const Repeated rep = find_repeated((one - lo) >> shift, tid < n && one - lo <= hi - lo);
    if (rep.none())                                     // uniform
      each([&](uint32_t k, bool valid) {
        if (valid && k - lo <= hi - lo) atomicAdd(&bin[(k - lo) >> shift], 1u);
      });
    else
      count_repeated(keys, n, lo, hi, shift, rep, bin);
    __syncthreads();
    uint32_t c[PER], sum = 0, excl, total;
#pragma unroll
    for (int q = 0; q < PER; ++q) sum += c[q] = bin[PER * tid + q];
    block_prefix(red, sum, excl, total);
    pick_bin<PER>(sh, c, excl, k_rem);
    const uint32_t d = sh.pick[0], held = sh.pick[2], width = (1u << shift) - 1u;
    k_rem = sh.pick[1];
    from = lo + (d << shift);
    to = hi - from < width ? hi : from + width;
    if (held <= kFinListMax) {                          // uniform
      if (tid == 0) sh.pick[3] = 0;
      __syncthreads();
      each([&](uint32_t k, bool valid) {
        if (valid && k - from <= to - from) sh.list[atomicAdd(&sh.pick[3], 1u)] = k;      // `held` of them
      });
      __syncthreads();
      pick_listed(sh.list, held, thr, k_rem);
      return;
    }
  }
}

// The k-th smallest of the row's keys and how many keys equal to it are kept.  n: finish_load's result.
// The k-th key is hardly outside [below, bound] (both from the sample): 2048 bins of equal width there, and the few keys
// of the bin that holds the k-th compared with each other.  Where its bin holds more than kFinListMax, that is cut in turn; where
// it is before them, all keys before them are.  Whole rows take the radix select.
__device__ __forceinline__ void finish_threshold(FinishShared& sh, const uint32_t* lds_cand, const SelectArgs& a, int row,
                                                 int n, uint32_t bound, uint32_t below, uint32_t& thr, uint32_t& k_rem) {
  const int tid = threadIdx.x;
  if (sh.whole_row) {                                  // uniform
    const float* sr = a.scores + (int64_t)row * a.T;
    radix_select_block(a.T, (uint32_t)a.k, [&](int i) { return order_key(sr[i]); }, sh.h, sh.sm, thr, k_rem);
    return;
  }
  const int shift = bin_shift(below, bound, kFinBinBits);
  uint32_t lower = 0;                                   // keys before `below`: most of the k, so not by atomics on one word
  for (int i = tid; i < n; i += kFinThreads) {
    const uint32_t key = lds_cand[i];
    if (key < below)
      ++lower;
    else
      atomicAdd(&sh.h[clamped_bin(key, below, bound, shift)], 1u);
  }
  __syncthreads();
  const uint32_t c[2] = {sh.h[2 * tid], sh.h[2 * tid + 1]}, kk = (uint32_t)a.k;
  uint32_t excl, total;
  block_scan<false>(sh.sm, c[0] + c[1], lower, excl, total, lower);
  if (__builtin_expect(lower >= kk, 0)) {               // uniform: the k-th is before `below`
    k_rem = kk;
    zoom_threshold<2>(sh.bins, sh.sm, sh.h, lds_cand, n, 0u, below - 1u, thr, k_rem);
    return;
  }
  pick_bin<2>(sh.bins, c, lower + excl, kk);            // n >= k
  const uint32_t d = sh.bins.pick[0], held = sh.bins.pick[2];
  k_rem = sh.bins.pick[1];
  if (__builtin_expect(held > kFinListMax, 0)) {        // uniform
    const uint32_t from = below + (d << shift), width = (1u << shift) - 1u;
    zoom_threshold<2>(sh.bins, sh.sm, sh.h, lds_cand, n, from, bound - from < width ? bound : from + width, thr, k_rem);
    return;
  }
  for (int i = tid; i < n; i += kFinThreads) {
    const uint32_t key = lds_cand[i];
    if (key >= below && clamped_bin(key, below, bound, shift) == d) sh.bins.list[atomicAdd(&sh.bins.pick[3], 1u)] = key;   // `held` of them
  }
  __syncthreads();
  pick_listed(sh.bins.list, held, thr, k_rem);
}

// The kept tokens in ascending order, then the window tokens.
__device__ __forceinline__ void finish_write(FinishShared& sh, const uint32_t* lds_cand, const SelectArgs& a, int row,
                                             int n, uint32_t thr, uint32_t k_rem) {
  const int tid = threadIdx.x, T = a.T, k = a.k, W = a.W;
  int32_t* out = a.idx_out + (int64_t)row * (k + W);
  auto put = [&](uint32_t pos, uint32_t tok) { out[pos] = (int32_t)tok; };
  const uint32_t* li = lds_cand + a.cand_cap;
  if (sh.whole_row) {                                  // uniform
    const float* sr = a.scores + (int64_t)row * T;
    ordered_write<8>(T, thr, k_rem, k, [&](int i0, uint32_t* key) {
      for (int j = 0; j < 8; ++j) key[j] = order_key(sr[min(i0 + j, T - 1)]);
    }, [&](int i) { return (uint32_t)i; }, sh.sm, put);
  } else {
    // four keys per LDS read: cand_cap is a multiple of eight
    const uint4* lk = reinterpret_cast<const uint4*>(lds_cand);
    auto four = [&](int i0, uint32_t* key) {
      const uint4 x = lk[i0 / 4];
      key[0] = x.x;
      key[1] = x.y;
      key[2] = x.z;
      key[3] = x.w;
    };
    auto tok = [&](int i) { return li[i]; };
    if (n <= 4 * kFinThreads)
      ordered_write<4>(n, thr, k_rem, k, four, tok, sh.sm, put);
    else
      ordered_write<8>(n, thr, k_rem, k, [&](int i0, uint32_t* key) {
        four(i0, key);
        four(i0 + 4, key + 4);
      }, tok, sh.sm, put);
  }
  // window tokens T .. T+W-1 (Alg. 1 step 10: Concat with I_w)
  for (int i = tid; i < W; i += kFinThreads) out[k + i] = T + i;
}

// Step 3: one workgroup per row.
__device__ __forceinline__ void select_finish_body(void* lds, const SelectArgs& a, int row) {
  FinishShared& sh = *static_cast<FinishShared*>(lds);
  uint32_t* lds_cand = finish_cand(lds);
  const uint32_t below = a.bound[2 * row + 1];
  uint32_t bound = a.bound[2 * row];
  int n = finish_load(sh, lds_cand, a, row);
  if (__builtin_expect(sh.whole_row == kTooMany, 0)) n = finish_tighten(sh, lds_cand, a, row, bound, below);   // uniform
  uint32_t thr, k_rem;
  finish_threshold(sh, lds_cand, a, row, n, bound, below, thr, k_rem);
  finish_write(sh, lds_cand, a, row, n, thr, k_rem);
}

// All three steps for a row of at most PER * kFinThreads scores, one workgroup per row: every token is a candidate.  The
// threshold as in the finish step, in 4096 bins between the row's smallest and largest key.  Bound by latency.  8 rows, us, with
// the radix select and so: 2000 scores 7.4, 5.7; 8000 10.4, 7.1; 12000 12.9, 7.9; 12000
// of a few values 15.0, 11.2; within 2 % beside outliers 15.5, 12.2; 16000 so (then in three launches) 21.5, 16.9.
// PER keys a thread.
constexpr int kPickMost = kPickWords;                   // most tokens of a row that go to SelectArgs.picks
static_assert(kPickMost == 4 * kFinThreads, "they are staged in the bins");
template <int PER>
struct ShortSelectShared {
  uint4 keys[PER * kFinThreads / 4];
  uint4 bin[kFinThreads];
  uint32_t sm[2 * kFinWaves + 2];
  BinPick bins;
};
// PICKS: the launch has a place for the tokens (SelectArgs).
template <int PER, bool PICKS = false>
__device__ __forceinline__ void select_short_body(ShortSelectShared<PER>& sh, const SelectArgs& a, int row) {
  const int tid = threadIdx.x, T = a.T;
  constexpr int kPer = PER, kMost = PER * kFinThreads, kWrite = PER <= 16 ? PER : 16;      // keys a thread writes together
  static_assert(PER % 4 == 0 && PER % kWrite == 0, "four keys per read");
  const float* sr = a.scores + (int64_t)row * a.T;
  uint32_t* keys = &sh.keys[0].x;
  uint32_t key[kPer], lo = 0xffffffffu, hi = 0u, thr, k_rem;
  {
    float f[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) f[u] = u * kFinThreads < T ? sr[min(tid + u * kFinThreads, T - 1)] : 0.f;   // one round trip
#pragma unroll
    for (int u = 0; u < kPer; ++u) key[u] = order_key(f[u]);
  }
  sh.bin[tid] = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) sh.bins.pick[3] = 0;
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    if (u * kFinThreads < T) {                          // uniform; positions past the end repeat the last key
      if (tid + u * kFinThreads < T) keys[tid + u * kFinThreads] = key[u];
      lo = min(lo, key[u]);
      hi = max(hi, key[u]);
    }
  block_min_max(sh.sm, lo, hi);
  thr = lo;
  k_rem = (uint32_t)a.k;
  if (lo != hi) {                                       // uniform; else all scores are equal
    const int shift = bin_shift(lo, hi, kSampleBinBits);
    uint32_t* bin = &sh.bin[0].x;
    const Repeated rep = find_repeated((key[0] - lo) >> shift, tid < T);
    if (rep.none()) {             // uniform
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if (tid + u * kFinThreads < T) atomicAdd(&bin[(key[u] - lo) >> shift], 1u);
    } else {
      count_repeated(keys, T, lo, hi, shift, rep, bin);  // (in registers, like the others, it cost rows without any 0.2 to 0.8 us)
    }
    __syncthreads();
    const uint4 c4 = sh.bin[tid];
    const uint32_t cs[4] = {c4.x, c4.y, c4.z, c4.w};
    uint32_t excl, total;
    block_prefix(sh.sm, c4.x + c4.y + c4.z + c4.w, excl, total);
    pick_bin<4>(sh.bins, cs, excl, k_rem);              // 1 <= k <= T
    const uint32_t d = sh.bins.pick[0], held = sh.bins.pick[2];
    k_rem = sh.bins.pick[1];
    if (__builtin_expect(held > kFinListMax, 0)) {      // uniform
      const uint32_t from = lo + (d << shift), width = (1u << shift) - 1u;
      zoom_threshold<4>(sh.bins, sh.sm, bin, keys, T, from, hi - from < width ? hi : from + width, thr, k_rem);
    } else {
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if (tid + u * kFinThreads < T && (key[u] - lo) >> shift == d) sh.bins.list[atomicAdd(&sh.bins.pick[3], 1u)] = key[u];   // `held` of them
      __syncthreads();
      pick_listed(sh.bins.list, held, thr, k_rem);
    }
  } else {
    __syncthreads();                                    // the keys are there
  }
  int32_t* out = a.idx_out + (int64_t)row * (a.k + a.W);
  auto four = [&](int i0, uint32_t* x) {
    const uint4 v = sh.keys[i0 / 4];                    // i0 + 3 < kMost
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
  };
  auto tok = [&](int i) { return (uint32_t)i; };
  const bool picks = PICKS && row < a.pick_rows;
  uint32_t* staged = &sh.bin[0].x;                      // kPickMost words
  auto put = [&](uint32_t pos, uint32_t token) {
    out[pos] = (int32_t)token;
    if (picks) staged[pos] = token;                     // pos < k <= kPickMost
  };
  if (picks) __syncthreads();                           // the bins are done with
  if (T <= 4 * kFinThreads)
    ordered_write<4>(T, thr, k_rem, a.k, four, tok, sh.sm, put);
  else
    ordered_write<kWrite>(T, thr, k_rem, a.k, [&](int i0, uint32_t* x) {
#pragma unroll
      for (int j = 0; j < kWrite; j += 4) four(min(i0 + j, kMost - 4), x + j);
    }, tok, sh.sm, put);
  if (picks) {                                          // 64 words a store: written where they are found, a few at a time, 6 us more
    const unsigned long long tag = (unsigned long long)*a.pick_tag << 32;
    unsigned long long* pick = a.picks + (int64_t)row * a.k;
    __syncthreads();
    for (int i = tid; i < a.k; i += kFinThreads) __hip_atomic_store(pick + i, tag | staged[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  for (int i = tid; i < a.W; i += kFinThreads) out[a.k + i] = T + i;   // window tokens (Alg. 1 step 10)
}

// Arguments of a select over `rows` rows of scores (buffers from the workspace; rows <= ws.sel_rows).  have_sample: the pooling
// kernel left one behind, of scores it pooled over S tokens.
SelectArgs select_args(const Workspace& ws, const float* scores, int T, int k, int W, int32_t* idx_out,
                       bool have_sample, int S);

}  // namespace asl
