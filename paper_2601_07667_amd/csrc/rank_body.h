// Device code of asl_rank's kernels (see rank.hip for the method), written as functions over explicit
// shared-state structs so that another kernel can host them beside a second body.
#pragma once
#include "sample_body.h"

namespace asl {

constexpr int kSortThreads = kRowThreads;
constexpr int kSortWaves = kSortThreads / 64;

struct DigitShared {
  alignas(8) uint16_t cnt[kSortWaves][256];             // pairs per wavefront and digit
  alignas(8) uint16_t start[kSortWaves][256];           // their first places
};

// Sorts n <= PER * kSortThreads pairs in LDS by key, equal keys in the order they are in: LSD radix passes of 8 bits over the
// bits in which the keys differ, equal digits of a wavefront ranked by ballots.  For what equal-width bins cannot
// tell apart: repeated or nearly equal keys.  Two barriers a pass: a wavefront clears and fills its own row of counts,
// and every wavefront works out its own first places from all rows.
template <int PER, typename Tok>
__device__ __forceinline__ void sort_by_digits(uint32_t* key, Tok* tok, DigitShared& sh, uint32_t* red, int n) {
  const int tid = threadIdx.x, wave = uniform_wave(), lane = tid & 63;
  const int rounds = (n + kSortThreads - 1) / kSortThreads;                  // of 64 pairs per wavefront
  uint32_t lo = 0xffffffffu, hi = 0u;
  for (int i = tid; i < n; i += kSortThreads) {
    lo = min(lo, key[i]);
    hi = max(hi, key[i]);
  }
  block_min_max(red, lo, hi);
  const int bits = hi == lo ? 0 : 32 - __clz((int)(hi - lo)), n_pass = (bits + 7) / 8;
  for (int pass = 0; pass < n_pass; ++pass) {           // uniform
    const int shift = 8 * pass;
    int e = wave * 64 * rounds + lane;                  // this thread's pair r: e + 64 r
    asm volatile("" : "+v"(e));                         // addresses are worked out per pass, not held through it
    uint32_t k[PER], t[PER], off[PER];
    // digits 4 lane .. 4 lane + 3.  Lanes read what others of their wavefront wrote without a workgroup barrier between (LDS
    // operations of a wavefront are in order): by bytes, since words of another type might be taken not to be the same
    __builtin_memset(&sh.cnt[wave][4 * lane], 0, 8);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      k[r] = lo;
      t[r] = 0;
      off[r] = 0;
      if (r < rounds) {                                 // uniform
        const bool valid = e + 64 * r < n;
        if (valid) {
          k[r] = key[e + 64 * r];
          t[r] = tok[e + 64 * r];
        }
        const uint32_t d = ((k[r] - lo) >> shift) & 255u;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
          const bool bit = (d >> b) & 1u;
          const uint64_t bal = __ballot(bit);
          peers &= bit ? bal : ~bal;
        }
        const uint32_t before = lanes_below(peers);
        uint32_t old = 0;
        if (valid) old = sh.cnt[wave][d];
        if (valid && before == 0) sh.cnt[wave][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
        off[r] = old + before;
      }
    }
    __syncthreads();                                    // all counts are there, all pairs are read
    // two digits a word: sums stay below 2^16
    uint2 tot = make_uint2(0u, 0u), prev = tot;
#pragma unroll 8
    for (int w = 0; w < kSortWaves; ++w) {
      if (w == wave) prev = tot;
      uint2 c;
      __builtin_memcpy(&c, &sh.cnt[w][4 * lane], 8);
      tot.x += c.x;
      tot.y += c.y;
    }
    const uint32_t t0 = tot.x & 0xffffu, t1 = tot.x >> 16, t2 = tot.y & 0xffffu, t3 = tot.y >> 16, sum = t0 + t1 + t2 + t3;
    const uint32_t s0 = wave_prefix_sum(sum) - sum, s1 = s0 + t0, s2 = s1 + t1;
    const uint2 starts = make_uint2(prev.x + (s0 | (s1 << 16)), prev.y + (s2 | ((s2 + t2) << 16)));
    __builtin_memcpy(&sh.start[wave][4 * lane], &starts, 8);
    __builtin_amdgcn_wave_barrier();                    // a lane reads what others of its wavefront wrote
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      if (r < rounds && e + 64 * r < n) {
        const uint32_t dest = sh.start[wave][((k[r] - lo) >> shift) & 255u] + off[r];   // < n
        key[dest] = k[r];
        tok[dest] = (Tok)t[r];
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
constexpr uint32_t kBinMax = 64;                        // longest bin that is ordered by comparing its keys

// Short vectors (T <= kShortT), in one launch and with nothing exchanged between workgroups: every workgroup reads all
// keys.  Two ways:
//  - by counting: a token's 32 lanes compare its key with every other one, rank = keys before it in the order (key
//    ascending, index ascending), 32 tokens a workgroup.  T^2 comparisons of two vector instructions.
//  - by bins: the workgroup counts all keys in 4096 bins of equal width between the smallest and the largest; of those bins
//    that reach into its 64 places of the order it groups the keys in LDS, and a thread per key compares it with the others
//    of its bin.  A bin longer than kBinMax that reaches into its places (at most two do) is cut into 4096 in turn, between the
//    keys it holds, or is one key, whose tokens are counted in order.  Bound by latency (eight barriers, and as many per
//    such bin).
// Counting takes the sizes up to kCountT, where its time does not depend on the scores and the bins' would (one call, us, counting and
// bins: 8000 tokens 8.4, 6.4 to 17; 9000 13.4, 6.5; 12000 17.0, 7.1; 12000 of which a third are equal 17, 16.8; of a few values 17,
// 16.3; within 2 % beside outliers 17, 15.2; of 84 values and one far away 17, 21).
constexpr int kCountTokens = kSortThreads / 32;
constexpr int kCountT = 8192;
constexpr int kShortPlaces = 2 * kCountTokens;
constexpr int kShortPer = kShortT / kSortThreads;
static_assert(kShortT % kSortThreads == 0 && kCountTokens == 32, "the keys of a workgroup's tokens are one group of 32");
// Where a short vector's ranks go: put(token, rank).
struct PutRank {
  int32_t* out;
  __device__ __forceinline__ void operator()(uint32_t t, uint32_t rank) const { out[t] = (int32_t)rank; }
};
// ... and are kept for the statistic: a workgroup ranks tokens from `first` on by counting, or the tokens of places from `first`
// on by bins, each once.
constexpr int kShortKept = kShortPlaces + (int)kBinMax;
struct KeptRanks {
  uint32_t tok[kShortKept], rank[kShortKept];           // tok ~0: none
};
struct PutAndKeepRank {
  int32_t* out;
  KeptRanks* kept;
  uint32_t first;
  bool by_token;
  __device__ __forceinline__ void operator()(uint32_t t, uint32_t rank) const {
    out[t] = (int32_t)rank;
    const uint32_t i = min((by_token ? t : rank) - first, (uint32_t)kShortKept - 1u);   // smaller by itself
    kept->tok[i] = t;
    kept->rank[i] = rank;
  }
};
struct ShortRankShared {
  uint32_t keys[kShortT];                               // by counting, and where long bins are cut
  union {
    uint4 bin4[kSampleBins / 4 + 1];                    // four bins a thread: their counts, then their first places and the last one's end
    uint32_t bin[kSampleBins + 4];
  };
  uint32_t key[kShortPlaces + 2 * kBinMax];             // by bins: keys of bins that reach into the workgroup's places ...
  uint32_t tok[kShortPlaces + 2 * kBinMax];             // ... and tokens, from their bin's first place on; ~0: nothing there
  uint32_t held[kShortPlaces + kBinMax];                // keys there from a bin's first place on
  uint32_t todo[8][3];                                  // long bins yet to be cut: first and last key, first place
  uint32_t n_todo;
  uint32_t red[2 * kSortWaves];
};
inline int short_rank_blocks(int T) { return T <= kCountT ? (T + kCountTokens - 1) / kCountTokens : (T + kShortPlaces - 1) / kShortPlaces; }

// Ranks of tokens 32 group .. 32 group + 31 by counting.  keys: all T of them; up to the next multiple of 32 the largest
// key, which precedes nothing.
template <typename Put>
__device__ __forceinline__ void count_ranks(const uint32_t* keys, int T, int group, const Put& put) {
  const int tid = threadIdx.x, lane = tid & 31, n_groups = (T + 31) / 32;
  const int i0 = group * kCountTokens, i = i0 + (tid >> 5);
  const uint32_t ki = keys[i];                          // i < kShortT
  uint32_t before = 0;
#pragma unroll 8
  for (int g = 0; g < group; ++g) before += (keys[g * 32 + lane] <= ki) ? 1u : 0u;              // lower indices: ties precede
#pragma unroll 8
  for (int g = group + 1; g < n_groups; ++g) before += (keys[g * 32 + lane] < ki) ? 1u : 0u;    // higher indices: ties follow
  {
    const uint32_t kj = keys[i0 + lane];
    before += (kj < ki || (kj == ki && i0 + lane < i)) ? 1u : 0u;
  }
#pragma unroll
  for (int d = 16; d > 0; d >>= 1) before += (uint32_t)__shfl_xor((int)before, d);
  if (lane == 0 && i < T) put((uint32_t)i, before);
}

// The rest of a way by bins, once the keys in [lo, hi] are counted: the bins' first places (`begin`: that of lo's) to sh.bin, and
// those longer than kBinMax that reach into places [p0, p1) to sh.todo.
__device__ __forceinline__ void short_bins(ShortRankShared& sh, uint32_t lo, uint32_t hi, int shift, uint32_t begin, uint32_t p0, uint32_t p1) {
  const int tid = threadIdx.x;
  const uint4 c = sh.bin4[tid];
  uint32_t at, total;
  block_prefix(sh.red, c.x + c.y + c.z + c.w, at, total);
  const uint32_t cs[4] = {c.x, c.y, c.z, c.w};
  uint32_t at4[4];
  at += begin;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    at4[q] = at;
    at += cs[q];
    if (cs[q] > kBinMax && at4[q] < p1 && at > p0) {    // at most two of the workgroup's
      const uint32_t i = min(atomicAdd(&sh.n_todo, 1u), 7u), from = lo + ((uint32_t)(4 * tid + q) << shift), width = (1u << shift) - 1u;
      sh.todo[i][0] = from;
      sh.todo[i][1] = hi - from < width ? hi : from + width;
      sh.todo[i][2] = at4[q];
    }
  }
  sh.bin4[tid] = make_uint4(at4[0], at4[1], at4[2], at4[3]);       // own counts only were read
  if (tid == 0) sh.bin[kSampleBins] = begin + total;
  __syncthreads();
}
// Ranks of the keys grouped in sh.key / sh.tok from place p0 - kBinMax on, of those with a place in [from, to).
template <typename Put>
__device__ __forceinline__ void short_places(const ShortRankShared& sh, uint32_t lo, int shift, uint32_t p0, uint32_t from, uint32_t to,
                                             const Put& put) {
  // four threads per place: few keys are this workgroup's, and a wavefront that went through its own again would run the
  // comparison once for each (12000 tokens: 28 us the ranking and its statistic, so 18)
  const int tid = threadIdx.x, i = tid >> 2, part = tid & 3;
  static_assert(4 * (kShortPlaces + 2 * kBinMax) <= kSortThreads, "four threads per place");
  if (i >= kShortPlaces + 2 * (int)kBinMax) return;
  const uint32_t k = sh.key[i], t = sh.tok[i];
  uint32_t before = 0, i0 = 0;
  if (t != 0xffffffffu) {
    const uint32_t d = (k - lo) >> shift, i1 = sh.bin[d + 1u] + kBinMax - p0;
    i0 = sh.bin[d] + kBinMax - p0;
    if (i1 - i0 > 1u)
      for (uint32_t j0 = i0 + part; j0 < i1; j0 += 16u) {
#pragma unroll
        for (uint32_t q = 0; q < 16u; q += 4u) {
          const uint32_t j = min(j0 + q, i1 - 1u), kj = sh.key[j], tj = sh.tok[j];
          before += (j0 + q < i1 && (kj < k || (kj == k && tj < t))) ? 1u : 0u;
        }
      }
  }
  before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0xb1, 0xf, 0xf, false);   // quad_perm [1, 0, 3, 2]
  before += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)before, 0x4e, 0xf, 0xf, false);   // quad_perm [2, 3, 0, 1]
  const uint32_t place = p0 + i0 + before - kBinMax;
  if (part == 0 && t != 0xffffffffu && place >= from && place < to) put(t, place);
}

// f(key, token, valid) for the thread's keys in sh.keys, read four at a time.
template <typename F>
__device__ __forceinline__ void four_at_a_time(const ShortRankShared& sh, int T, F f) {
  for (int t0 = threadIdx.x; t0 < kShortT; t0 += 4 * kSortThreads) {
    if (__builtin_amdgcn_readfirstlane(t0) >= T) break;
    uint32_t k[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) k[q] = sh.keys[min(t0 + q * kSortThreads, T - 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) f(k[q], t0 + q * kSortThreads, t0 + q * kSortThreads < T);
  }
}

// A wavefront's stretch of tokens for the loops over all keys: token(g), g < groups.
struct Stretch {
  int t0, groups;
};
__device__ __forceinline__ Stretch short_stretch(int T) {
  const int groups = (T + kSortThreads - 1) / kSortThreads;
  return {uniform_wave() * 64 * groups + (int)(threadIdx.x & 63), groups};
}
// Ranks of the tokens with this key, which has the places from `first` on, that belong to places [p0, p1); n: those in the
// wavefront's stretch.  The one or two wavefronts whose stretches hold such places go through theirs.
template <typename Put>
__device__ __forceinline__ void rank_equal(ShortRankShared& sh, int T, uint32_t value, uint32_t n, uint32_t first, uint32_t p0, uint32_t p1,
                                           const Put& put) {
  const int wave = uniform_wave(), lane = threadIdx.x & 63;
  const Stretch s = short_stretch(T);
  __syncthreads();                                      // red may still be in use
  if (lane == 0) sh.red[wave] = n;
  __syncthreads();
  const uint32_t before = row_prefix_sum(sh.red[lane & (kSortWaves - 1)]);
  uint32_t place = first + (uint32_t)__builtin_amdgcn_readlane((int)before, wave) - n;
  if (place >= p1 || place + n <= p0) return;           // uniform in the wavefront: no barrier follows
  for (int g = 0; g < s.groups; ++g) {
    const int t = s.t0 + 64 * g;
    const bool in = t < T && sh.keys[min(t, T - 1)] == value;
    const uint64_t m = __ballot(in);
    const uint32_t at = place + lanes_below(m);
    if (in && at >= p0 && at < p1) put((uint32_t)t, at);
    place += (uint32_t)__popcll(m);
  }
}

template <typename Put>
__device__ __forceinline__ void rank_short_body(ShortRankShared& sh, const float* __restrict__ s, int T, const Put& put, int b) {
  const int tid = threadIdx.x;
  uint32_t key[kShortPer];
  {
    float f[kShortPer];
#pragma unroll
    for (int u = 0; u < kShortPer; ++u) f[u] = u * kSortThreads < T ? s[min(tid + u * kSortThreads, T - 1)] : 0.f;   // one round trip
#pragma unroll
    for (int u = 0; u < kShortPer; ++u) key[u] = order_key(f[u]);
  }
  auto all_keys = [&] {
#pragma unroll
    for (int u = 0; u < kShortPer; ++u)
      if (u * kSortThreads < T) sh.keys[tid + u * kSortThreads] = tid + u * kSortThreads < T ? key[u] : 0xffffffffu;
    __syncthreads();
  };
  if (T <= kCountT) {                                   // uniform
    all_keys();
    count_ranks(sh.keys, T, b, put);
    return;
  }
  const uint32_t p0 = (uint32_t)(b * kShortPlaces), p1 = min(p0 + (uint32_t)kShortPlaces, (uint32_t)T);
  sh.bin4[tid] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < kShortPlaces + 2 * (int)kBinMax) sh.tok[tid] = 0xffffffffu;
  if (tid == 0) sh.n_todo = 0;
  uint32_t lo = key[0], hi = key[0];                    // positions past the end repeat the last key
#pragma unroll
  for (int u = 1; u < kShortPer; ++u)
    if (u * kSortThreads < T) {                         // uniform
      lo = min(lo, key[u]);
      hi = max(hi, key[u]);
    }
  block_min_max(sh.red, lo, hi);
  if (lo == hi) {                                       // uniform: all scores are equal
    if (tid < kShortPlaces && p0 + tid < p1) put(p0 + (uint32_t)tid, p0 + (uint32_t)tid);
    return;
  }
  int shift = bin_shift(lo, hi, kSampleBinBits);
  const Repeated rep = find_repeated((key[0] - lo) >> shift, tid < T);
  uint32_t slot[kShortPer];
  if (rep.none()) {                 // uniform
#pragma unroll
    for (int u = 0; u < kShortPer; ++u) {
      slot[u] = 0;
      if (tid + u * kSortThreads < T) slot[u] = atomicAdd(&sh.bin[(key[u] - lo) >> shift], 1u);
    }
  } else {
#pragma unroll
    for (int u = 0; u < kShortPer; ++u) {
      slot[u] = 0;
      if (u * kSortThreads < T) slot[u] = slot_for(rep, sh.bin, (key[u] - lo) >> shift, tid + u * kSortThreads < T);    // uniform
    }
  }
  __syncthreads();
  short_bins(sh, lo, hi, shift, 0u, p0, p1);
  // bins that begin at the workgroup's places are all its own
#pragma unroll
  for (int u = 0; u < kShortPer; ++u) {
    if (tid + u * kSortThreads < T) {
      const uint32_t d = (key[u] - lo) >> shift, first = sh.bin[d];
      if (first >= p0 && first < p1 && sh.bin[d + 1u] - first <= kBinMax) {
        const uint32_t i = min(first + kBinMax - p0 + slot[u], (uint32_t)kShortPlaces + 2u * kBinMax - 1u);   // smaller by itself
        sh.key[i] = key[u];
        sh.tok[i] = (uint32_t)(tid + u * kSortThreads);
      }
    }
  }
  __syncthreads();
  short_places(sh, lo, shift, p0, p0, 0xffffffffu, put);
  if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)sh.n_todo) == 0, 1)) return;           // uniform
  all_keys();
  const Stretch s_t = short_stretch(T);
  for (;;) {
    const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.n_todo);
    if (n == 0u) return;                                // uniform; every trip takes a bin off and adds parts of it
    // the last two of the list: smallest and largest keys, and how many the wavefront's stretch holds
    const bool two = n > 1u;
    uint32_t from[2], to[2], at[2], held[2] = {0u, 0u}, lo2[2], hi2[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t* r = sh.todo[min(n, 8u) - (two ? 1u + (uint32_t)i : 1u)];
      from[i] = r[0];
      to[i] = r[1];
      at[i] = r[2];
      lo2[i] = 0xffffffffu;
      hi2[i] = 0u;
    }
#pragma unroll
    for (int g = 0; g < kShortPer; ++g)
      if (g < s_t.groups) {                             // uniform
        const int t = s_t.t0 + 64 * g;
        const uint32_t k = sh.keys[min(t, T - 1)];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bool in = t < T && k - from[i] <= to[i] - from[i];
          lo2[i] = min(lo2[i], in ? k : 0xffffffffu);
          hi2[i] = max(hi2[i], in ? k : 0u);
          held[i] += (uint32_t)__popcll(__ballot(in));
        }
      }
    block_min_max(sh.red, lo2[0], hi2[0]);              // its barriers: everybody has read the list, the bins and the places
    if (two) block_min_max(sh.red, lo2[1], hi2[1]);     // uniform
    const bool one0 = lo2[0] == hi2[0], one1 = !two || lo2[1] == hi2[1];       // of a single key, or not there
    if (one0) rank_equal(sh, T, lo2[0], held[0], at[0], p0, p1, put);
    if (two && one1) rank_equal(sh, T, lo2[1], held[1], at[1], p0, p1, put);
    // both at once if at most 16 bins apart
    const bool both = !one0 && !one1 && max(to[0], to[1]) - min(from[0], from[1]) <= 16u * (to[0] - from[0]);
    if (tid == 0) sh.n_todo = n - (two && (both || one0 || one1) ? 2u : 1u);
    if (!one0 || !one1) {                               // uniform
      const int i = one0 ? 1 : 0;
      const uint32_t begin = both ? min(at[0], at[1]) : at[i];
      lo = both ? min(lo2[0], lo2[1]) : lo2[i];
      hi = both ? max(hi2[0], hi2[1]) : hi2[i];
      // as above, but by the places themselves: the bins are the workgroup's own choice
      shift = bin_shift(lo, hi, kSampleBinBits);
      sh.bin4[tid] = make_uint4(0u, 0u, 0u, 0u);
      if (tid < kShortPlaces + 2 * (int)kBinMax) sh.tok[tid] = 0xffffffffu;
      if (tid < kShortPlaces + (int)kBinMax) sh.held[tid] = 0u;
      __syncthreads();
      auto in = [&](uint32_t k, bool valid) { return valid && k - lo <= hi - lo; };
      const Repeated again = find_repeated((sh.keys[tid] - lo) >> shift, in(sh.keys[tid], true));
      if (again.none())         // uniform
        four_at_a_time(sh, T, [&](uint32_t k, int, bool valid) {
          if (in(k, valid)) atomicAdd(&sh.bin[(k - lo) >> shift], 1u);
        });
      else
        four_at_a_time(sh, T, [&](uint32_t k, int, bool valid) {
          const uint32_t add = add_for(again, (k - lo) >> shift, in(k, valid));
          if (add != 0u) atomicAdd(&sh.bin[(k - lo) >> shift], add);
        });
      __syncthreads();
      short_bins(sh, lo, hi, shift, begin, p0, p1);
      four_at_a_time(sh, T, [&](uint32_t k, int t, bool valid) {
        if (in(k, valid)) {
          const uint32_t d = (k - lo) >> shift, first = sh.bin[d], end = sh.bin[d + 1u], at = first + kBinMax - p0;
          if (first < p1 && end > p0 && end - first <= kBinMax) {              // then at < kShortPlaces + kBinMax
            const uint32_t i = min(at + atomicAdd(&sh.held[at], 1u), (uint32_t)kShortPlaces + 2u * kBinMax - 1u);   // smaller by itself
            sh.key[i] = k;
            sh.tok[i] = (uint32_t)t;
          }
        }
      });
      __syncthreads();
      short_places(sh, lo, shift, p0, p0, p1, put);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
struct RankArgs {
  const float* s;                // scores
  const uint32_t* sample;        // n_s keys of s left behind by its producer, or null: taken from s
  int n_s, stride;               // the sample: keys and the stride between their positions
  int T, n_tiles, tile_log;      // tiles of 2^tile_log tokens
  int tile_step;                 // a power of two, at least half of n_tiles
  int n_buckets;
  int heavy;                     // sampled keys of a bin beyond which it is not one bucket's or part of one
  float per_key, per_key_deep;   // buckets per sampled key; where the sample has heavy bins (the last bucket is left to what
                                 // comes after all sampled keys)
  uint2* pairs;                  // [T] (key, token), grouped by bucket inside each tile
  uint32_t* count;               // [n_tiles][n_buckets] a tile's first place of the bucket | its tokens of the bucket << 16
  uint32_t* edge;                // [n_buckets + 1] first key of each bucket; the last one's last key; then 1: there are but the first and the last
  int32_t* rank_out;
};

// Bucket of what has `place` sampled keys before it, where the sample has heavy bins.
__device__ __forceinline__ uint32_t bucket_of_place(const RankArgs& a, uint32_t place) {
  return min((uint32_t)((float)place * a.per_key_deep), (uint32_t)a.n_buckets - 1u);     // monotone whatever the rounding
}

constexpr uint32_t kHeavyBin = 0x80000000u;
constexpr int kMaxHeavyBins = kRankMaxBuckets / 2 + 1;  // of one level: each holds more than two buckets' worth of the sample
constexpr int kSortedSample = 4096;                     // most keys of a sample that is sorted
struct PartShared {
  SampleShared s;                                       // bin: the sample's counts, then the bucket of each bin, or kHeavyBin | its number;
                                                        // of a sorted sample its numbers, then the buckets' first pairs
  union {
    uint16_t cnt[kSortWaves][kRankMaxBuckets];          // tokens per wavefront and bucket, then their first places
    struct {                                            // a sample to be sorted (sort_sample)
      uint32_t key[kSortedSample];
      DigitShared digit;
    };
    struct {                                            // of heavy bins (heavy_bins), until every token has its bucket
      union {
        uint32_t words[4 * kMaxHeavyBins + kSampleBins];
        struct {
          uint32_t here[4 * kMaxHeavyBins];             // of a single key: sampled in earlier tiles, in this one
          uint4 sub4[kSampleBins / 4];                  // sub-bins: their counts, then sampled keys before | number + 1 of a heavy one << 16
        };
      };
      uint32_t lo[2 * kMaxHeavyBins], hi[2 * kMaxHeavyBins];   // smallest and largest sampled key
      uint32_t place[2 * kMaxHeavyBins];                // sampled keys before (a sub-bin: before it, from all bins' first sub-bin on) | in it << 16
      uint32_t cut[kMaxHeavyBins];                      // a bin's first sub-bin | log2 of their number << 16
    };
  };
};
static_assert(sizeof(PartShared) <= 65536, "static LDS");
static_assert(sizeof(uint16_t) * kSortedSample <= sizeof(SampleShared::bin) && kSortedSample >= 4 * kRankMaxBuckets &&
                  sizeof(uint2) * kRankMaxBuckets <= sizeof(SampleShared::bin), "a sorted sample's numbers, then its borders, are held in bin");

// Sub-bin of a key of heavy bin h, or the bin's nearest one.
__device__ __forceinline__ uint32_t sub_bin(const PartShared& sh, uint32_t h, uint32_t key) {
  const uint32_t cut = sh.cut[h], lo = sh.lo[h], hi = sh.hi[h];
  return (cut & 0xffffu) + clamped_bin(key, lo, hi, bin_shift(lo, hi, (int)(cut >> 16)));
}

// Bins with more than a.heavy sampled keys: scores that repeat, or that lie close together beside outliers that
// spread the bins.  (c, first, h: the thread's four bins, the sampled keys and the heavy bins before them.)
//  - A heavy bin of one sampled key gets the buckets strictly between those of its neighbours; the tokens with that key are
//    shared out among them in token order, by how many of the sampled ones come before, so that such a bucket
//    holds equal keys only.
//  - Any other is cut into sub-bins between its smallest and largest sampled key: of 4096 in all as many as its share of the
//    sample.  Sub-bins that are still heavy and hold one sampled key are treated as above.
// Returns whether there are any that hold several: the bins' buckets are then of no use (half of 131040 scores within 100 of
// the next representable ones, all others spread: one bucket of 65 K, 490 us; with three such scores 1550).
// A wavefront's instruction takes 16 cycles of the unit here, so it is their number that counts: ~4.5 us for four sampled keys
// a thread.  (Sorting the sample instead took 18 us in every tile.  Ranking alone, us, so and sorted: 131040 scores, a third zeros
// 20.4, 42.5; rounded to whole numbers 26.2, 41.6; with a period of 32 19.6, 39.7; a million equal ones 30, 102.)
__device__ __forceinline__ bool heavy_bins(PartShared& sh, const RankArgs& a, const uint32_t (&v)[kSamplePer], uint32_t lo, int shift,
                                           const uint4& c, uint32_t first, uint32_t h, uint32_t n_heavy, int me) {
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t n_s = (uint32_t)a.n_s, most = (uint32_t)a.heavy;
  uint32_t* lut = &sh.s.bin[0].x;
  uint32_t* sub = &sh.sub4[0].x;
  auto each = [&](auto f) {                             // the thread's sampled keys; uniform, `valid` is not
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u)
      if (u * kRowThreads < (int)n_s) f(u, (uint32_t)(tid + u * kRowThreads) < n_s);
  };
  int in[kSamplePer];                                   // heavy bin of each key, -1: none
  auto ranges = [&] {                                   // lo and hi of these bins
    each([&](int u, bool) {
      if (in[u] >= 0) {                                 // any of the bin's keys
        __hip_atomic_store(&sh.lo[in[u]], v[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&sh.hi[in[u]], v[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    });
    __syncthreads();
    // equal keys take no part, and the wavefront's keys of one bin are put together first: atomics on one word come one
    // after the other
    auto widen = [&](int b, uint32_t k0, uint32_t k1) {
      if (k0 < __hip_atomic_load(&sh.lo[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) atomicMin(&sh.lo[b], k0);
      if (k1 > __hip_atomic_load(&sh.hi[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) atomicMax(&sh.hi[b], k1);
    };
    const uint64_t some = __ballot(in[0] >= 0);
    const int one = some == 0ull ? -2 : __builtin_amdgcn_readlane(in[0], __ffsll((unsigned long long)some) - 1);
    uint32_t k0 = 0xffffffffu, k1 = 0u;
    each([&](int u, bool) {
      if (in[u] == one) {
        k0 = min(k0, v[u]);
        k1 = max(k1, v[u]);
      } else if (in[u] >= 0) {
        widen(in[u], v[u], v[u]);
      }
    });
    k0 = wave_min(k0);
    k1 = wave_max(k1);
    if (some != 0ull && lane == 0) widen(one, k0, k1);
    __syncthreads();
  };
  // counts in[u]'s keys: those of a single key in sh.here (earlier tiles', this one's), others in their sub-bins
  auto count = [&](bool sub_bins) {
    const int last = (me + 1) << a.tile_log, first_here = me << a.tile_log;
    Repeated rep = {};
    each([&](int u, bool) {
      uint32_t word = 0u;
      bool valid = in[u] >= 0;
      if (valid) {
        const uint32_t b = (uint32_t)in[u];
        if (sh.lo[b] == sh.hi[b]) {
          const int t = (int)sel_sample_position((uint32_t)(tid + u * kRowThreads), a.stride);
          word = 2u * b + (t >= first_here ? 1u : 0u);
          valid = t < last;
        } else {
          valid = sub_bins;
          if (sub_bins) word = 4u * kMaxHeavyBins + sub_bin(sh, b, v[u]);
        }
      }
      if (u == 0) rep = find_repeated(word, valid);
      const uint32_t n = add_for(rep, word, valid);
      if (n != 0u) atomicAdd(&sh.words[word], n);
    });
    __syncthreads();
  };

  const uint32_t cs[4] = {c.x, c.y, c.z, c.w};
  uint32_t entry[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    entry[i] = bucket_of_place(a, first);
    if (cs[i] > most) {
      entry[i] = kHeavyBin | h;
      sh.place[h] = first | (cs[i] << 16);
      // shares rounded down: [kSampleBins first / n_s, kSampleBins (first + cs) / n_s) are disjoint and hold 2^log
      sh.cut[h++] = first * (uint32_t)kSampleBins / n_s | (uint32_t)(31 - __clz((int)(cs[i] * (uint32_t)kSampleBins / n_s))) << 16;
    }
    first += cs[i];
  }
  sh.s.bin[tid] = make_uint4(entry[0], entry[1], entry[2], entry[3]);         // own counts only were read
  sh.sub4[tid] = make_uint4(0u, 0u, 0u, 0u);
  for (int i = tid; i < 4 * kMaxHeavyBins; i += kRowThreads) sh.here[i] = 0u;
  __syncthreads();
  each([&](int u, bool valid) {
    const uint32_t e = valid ? lut[(v[u] - lo) >> shift] : 0u;
    in[u] = (e & kHeavyBin) != 0u ? (int)(e & 0xffffu) : -1;
  });
  ranges();
  count(true);
  const uint4 c2 = sh.sub4[tid];
  const uint32_t cs2[4] = {c2.x, c2.y, c2.z, c2.w};
  uint32_t x = c2.x + c2.y + c2.z + c2.w, total;
#pragma unroll
  for (int i = 0; i < 4; ++i) x += cs2[i] > most ? 65536u : 0u;
  block_prefix(sh.s.red, x, x, total);
  if (total == 0u) return false;                        // uniform: single keys only
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t before = x & 0xffffu, number = n_heavy + (x >> 16);         // < 2 kMaxHeavyBins
    entry[i] = before;
    if (cs2[i] > most) {
      entry[i] |= (number + 1u) << 16;
      sh.place[number] = before | (cs2[i] << 16);
      x += 65536u;
    }
    x += cs2[i];
  }
  sh.sub4[tid] = make_uint4(entry[0], entry[1], entry[2], entry[3]);
  __syncthreads();
  if (total >> 16 == 0u) return false;                  // uniform
  each([&](int u, bool) {
    const int b = in[u];
    if (b >= 0) in[u] = sh.lo[b] == sh.hi[b] ? -1 : (int)(sub[sub_bin(sh, (uint32_t)b, v[u])] >> 16) - 1;
  });
  ranges();
  const uint32_t number = n_heavy + min((uint32_t)tid, (total >> 16) - 1u);
  if (__syncthreads_or(sh.lo[number] != sh.hi[number]) != 0) return true;      // uniform
  count(false);
  return false;
}

// For a sample that bins and sub-bins do not tell apart: sorted, every n_s / B-th pair (key, token) of it is the first of a
// bucket, so that equal scores are shared out by token whatever the scores are.  Leaves border[b], b > 0, in sh.s.bin.
// One of every 2^thin keys: four a bucket are enough here, and sorting costs what it sorts (1024 keys ~18 us in every tile).
__device__ __forceinline__ void sort_sample(PartShared& sh, const RankArgs& a, const uint32_t (&v)[kSamplePer]) {
  const int tid = threadIdx.x, B = a.n_buckets, need = max(4 * B, 1024);
  const int thin = a.n_s >= 8 * need ? 3 : a.n_s >= 4 * need ? 2 : a.n_s >= 2 * need ? 1 : 0;
  const int n_s = min(a.n_s >> thin, kSortedSample);
  uint16_t* num = reinterpret_cast<uint16_t*>(sh.s.bin);
#pragma unroll
  for (int u = 0; u < kSamplePer; ++u) {
    const int j = tid + u * kSortThreads, i = j >> thin;
    const uint32_t pick = (uint32_t)i * 2654435761u >> 24;                   // any of the group's, for periodic scores
    if ((((uint32_t)j ^ pick) & ((1u << thin) - 1u)) == 0u && i < n_s) {
      sh.key[i] = v[u];
      num[i] = (uint16_t)j;
    }
  }
  __syncthreads();
  sort_by_digits<kSortedSample / kSortThreads>(sh.key, num, sh.digit, sh.s.red, n_s);
  uint2 first = make_uint2(0u, 0u);
  if (tid < B) {
    const int i = (int)((uint32_t)tid * (uint32_t)n_s / (uint32_t)B);
    first = make_uint2(sh.key[i], sel_sample_position(num[i], a.stride));
  }
  __syncthreads();                                      // num is read
  if (tid < B) reinterpret_cast<uint2*>(sh.s.bin)[tid] = first;
  __syncthreads();
}
// Bucket of token t with this key, by such borders: the last that is not behind the pair.
__device__ __forceinline__ uint32_t bucket_by_borders(const PartShared& sh, int B, uint32_t key, uint32_t t) {
  const uint2* border = reinterpret_cast<const uint2*>(sh.s.bin);
  int b = 0;
  for (int step = kRankMaxBuckets / 2; step > 0; step >>= 1) {
    if (b + step < B) {
      const uint2 x = border[b + step];
      if (x.x < key || (x.x == key && x.y <= t)) b += step;
    }
  }
  return (uint32_t)b;
}

// Bucket of token t (in tile `me`) with this key, where the sample has heavy bins.  Monotone in (key, token).
__device__ __forceinline__ uint32_t bucket_of_token(const PartShared& sh, const RankArgs& a, uint32_t lo, uint32_t hi, int shift, uint32_t key,
                                                    int t, int me) {
  const uint32_t* sub = &sh.sub4[0].x;
  const uint32_t e = (&sh.s.bin[0].x)[clamped_bin(key, lo, hi, shift)];
  if ((e & kHeavyBin) == 0u) return e;
  uint32_t h = e & 0xffffu, place = sh.place[h] & 0xffffu, held = sh.place[h] >> 16;
  uint32_t b0 = bucket_of_place(a, place), b1 = bucket_of_place(a, place + held);
  if (sh.lo[h] != sh.hi[h]) {
    // in buckets of their own, if there are any between the neighbours'
    const uint32_t at = sh.cut[h] & 0xffffu, e2 = sub[sub_bin(sh, h, key)], least = b1 > b0 + 1u ? b0 + 1u : b0, last = b1 > b0 + 1u ? b1 - 1u : b1;
    place += (e2 & 0xffffu) - (sub[at] & 0xffffu);
    b0 = min(max(bucket_of_place(a, place), least), last);
    h = (e2 >> 16) - 1u;
    if (e2 >> 16 == 0u || sh.lo[h] != sh.hi[h]) return b0;
    held = sh.place[h] >> 16;
    b1 = min(max(bucket_of_place(a, place + held), least), last);
  }
  if (key < sh.lo[h]) return b0;
  if (key > sh.lo[h] || b1 <= b0 + 1u) return b1;
  const uint32_t before = sh.here[2u * h] + (sh.here[2u * h + 1u] * (uint32_t)(t - (me << a.tile_log)) >> a.tile_log);   // <= held
  return b0 + 1u + min((uint32_t)((float)(before * (b1 - b0 - 1u)) * __builtin_amdgcn_rcpf((float)held)), b1 - b0 - 2u);
}

// Launch 1 for tile `me` (kSortThreads threads, R tokens each): the tile's (key, token) pairs, grouped by bucket and
// in token order inside one, go to the tile's own stretch of `pairs`, and where each bucket's begin to `count`.
// Every tile works out the same bucket borders from the same sample, so tiles agree on nothing else and wait for
// nobody.  Bound by latency: the loads, three counts with a scan each, the stores.
// Borders are those of the sample's histogram bins: bucket b holds the bins whose first sampled key has a place in
// [b, b + 1) n_s / B.  Where a bin holds more than a.heavy sampled keys, see heavy_bins, and sort_sample.
template <int R>
__device__ __forceinline__ void partition_body(PartShared& sh, const RankArgs& a, int me) {
  const int tid = threadIdx.x, wave = uniform_wave(), lane = tid & 63, T = a.T, B = a.n_buckets;
  constexpr int kTile = kSortThreads * R;
  const int e0 = me * kTile + wave * (64 * R) + lane;   // this thread's token r: e0 + 64 r
  float f[R];
  uint32_t v[kSamplePer];
#pragma unroll
  for (int r = 0; r < R; ++r) f[r] = a.s[min(e0 + 64 * r, T - 1)];
  load_sample(a.s, a.sample, a.n_s, a.stride, v);
  uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int u = 0; u < kSamplePer; ++u) {
    lo = min(lo, v[u]);
    hi = max(hi, v[u]);
  }
  block_min_max(sh.s.red, lo, hi);
  const int shift = bin_shift(lo, hi, kSampleBinBits);
  sample_count<true>(sh.s, v, a.n_s, lo, hi, shift);
  const uint4 c = sh.s.bin[tid];
  const uint32_t cs[4] = {c.x, c.y, c.z, c.w};
  uint32_t first = c.x + c.y + c.z + c.w, total;        // sampled keys before the thread's bins | heavy bins before << 16
#pragma unroll
  for (int i = 0; i < 4; ++i) first += cs[i] > (uint32_t)a.heavy ? 65536u : 0u;
  block_prefix(sh.s.red, first, first, total);
  const uint32_t n_heavy = total >> 16;
  const bool deep = n_heavy != 0u;                      // uniform
  uint32_t* lut = &sh.s.bin[0].x;
  uint32_t key[R], d[R], off[R];
#pragma unroll
  for (int r = 0; r < R; ++r) key[r] = order_key(f[r]);
  if (me == 0 && tid == 0) a.edge[B + 1] = deep ? 1u : 0u;
  if (__builtin_expect(deep, 0)) {
    if (me == 0 && tid == 0) {
      a.edge[0] = lo;
      a.edge[B] = hi;
    }
    if (heavy_bins(sh, a, v, lo, shift, c, first & 0xffffu, first >> 16, n_heavy, me)) {       // uniform
      sort_sample(sh, a, v);
#pragma unroll
      for (int r = 0; r < R; ++r) d[r] = bucket_by_borders(sh, B, key[r], (uint32_t)(e0 + 64 * r));
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) d[r] = bucket_of_token(sh, a, lo, hi, shift, key[r], e0 + 64 * r, me);
    }
    __syncthreads();                                    // the tables are read, the counts go there
  } else {
    const uint32_t past = (hi - lo) >> shift;
    uint32_t bucket[4], f1 = first;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bucket[i] = min((uint32_t)((float)f1 * a.per_key), (uint32_t)B - 1u);     // monotone whatever the rounding
      f1 += cs[i];
    }
    sh.s.bin[tid] = make_uint4(bucket[0], bucket[1], bucket[2], bucket[3]);   // own counts only were read
    __syncthreads();
    if (me == 0) {
      // first key of every bucket (empty ones: of the next that is not); bins behind the last key's: that key
      uint32_t prev = tid == 0 ? 0xffffffffu : lut[4 * tid - 1];             // + 1 = 0: bucket 0 begins with bin 0
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t j = (uint32_t)(4 * tid + i);
        for (uint32_t b = prev + 1u; b <= bucket[i]; ++b) a.edge[b] = j <= past ? lo + (j << shift) : hi;
        prev = bucket[i];
      }
      if (tid == kSortThreads - 1)
        for (uint32_t b = prev + 1u; b <= (uint32_t)B; ++b) a.edge[b] = hi;
    }
  }
  {
    // clear the wavefronts' counts
    uint32_t* w = reinterpret_cast<uint32_t*>(&sh.cnt[0][0]);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(sh.cnt) / 4 / kSortThreads); ++i) w[i * kSortThreads + tid] = 0u;
  }
  __syncthreads();

  // places inside the tile: equal buckets of a wavefront are ranked by ballots, stable by construction
  const int n_bits = B > 1 ? 32 - __clz(B - 1) : 0;
  if (!deep) {                                          // uniform
#pragma unroll
    for (int r = 0; r < R; ++r) d[r] = lut[clamped_bin(key[r], lo, hi, shift)];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool valid = e0 + 64 * r < T;
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < n_bits; ++b) {
      const bool bit = (d[r] >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const uint32_t before = lanes_below(peers);
    uint32_t old = 0;
    if (valid) old = sh.cnt[wave][d[r]];
    if (valid && before == 0) sh.cnt[wave][d[r]] = (uint16_t)(old + (uint32_t)__popcll(peers));
    off[r] = old + before;
  }
  __syncthreads();
  uint32_t tot = 0;
  if (tid < B) {
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) tot += sh.cnt[w][tid];
  }
  uint32_t start;
  block_prefix(sh.s.red, tot, start, total);
  if (tid < B) {
    a.count[(int64_t)me * B + tid] = start | (tot << 16);
    uint32_t run = start;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      const uint32_t c = sh.cnt[w][tid];
      sh.cnt[w][tid] = (uint16_t)run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = e0 + 64 * r;
    if (e < T) {
      const int dest = me * kTile + (int)(sh.cnt[wave][d[r]] + off[r]);
      if (dest < T) a.pairs[dest] = make_uint2(key[r], (uint32_t)e);          // always true
    }
  }
}

// ---------------------------------------------------------------------------------------------
constexpr int kBucketCap = 7168;                        // pairs one workgroup orders in LDS: two workgroups a compute unit
constexpr int kBucketPer = kBucketCap / kSortThreads;
constexpr int kBucketBins = 2 * kSortThreads;           // two per thread
constexpr int kBucketBinBits = 11;
static_assert(kBucketBins == 1 << kBucketBinBits, "bucket bins");

struct BucketShared {
  uint32_t key[kBucketCap];
  uint32_t tok[kBucketCap];
  union {
    struct {
      uint32_t bin[kBucketBins + 1];
      uint32_t cut[kBucketBins];                        // bucket_by_sub_bins
    };
    DigitShared digit;
  };
  uint32_t red[2 * kSortWaves];
  uint32_t seg_off[kRankMaxTiles + 1];                  // place of each tile's pairs in the bucket
  uint32_t seg_src[kRankMaxTiles];                      // ... and in `pairs`
  struct Pairs {                                        // operands of bucket_by_ranges
    const uint2* pairs;
    int32_t* rank_out;
    int T, n_tiles, tile_step;
  } args;
  uint32_t n, base;
};

// Pairs of the bin at places i0 .. i1 - 1 that come before (key, tok): four at a time, a bin's length in memory round trips
// otherwise.
__device__ __forceinline__ uint32_t before_in_bin(const BucketShared& sh, uint32_t i0, uint32_t i1, uint32_t key, uint32_t tok) {
  uint32_t c = 0;
  if (i1 - i0 > 1u)
#pragma unroll 1
    for (uint32_t i = i0; i < i1; i += 4u) {
#pragma unroll
      for (uint32_t q = 0; q < 4u; ++q) {
        const uint32_t j = min(i + q, i1 - 1u), k = sh.key[j], t = sh.tok[j];
        c += (i + q < i1 && (k < key || (k == key && t < tok))) ? 1u : 0u;
      }
    }
  return c;
}

// Ranks of the bucket's pairs (as bucket_by_bins has them: key, tok, slot of pair tid + r kSortThreads) where bins longer than
// kBinMax hold one key each: a run of equal keys is ordered by token, which is the pairs' order.  Its pairs are counted
// by groups of 64 (a wavefront's for one r), by ballots over the run's number; every later group begins where the ones before
// end.  The other bins as in bucket_by_bins.  c0, c1, first: the thread's bins and the pairs before them.
template <int R>
__device__ __forceinline__ void bucket_with_runs(BucketShared& sh, int n, uint32_t lo, uint32_t hi, const uint32_t (&key)[R], const uint32_t (&tok)[R],
                                                 uint32_t (&slot)[R], uint32_t c0, uint32_t c1, uint32_t first, uint32_t base, int T,
                                                 int32_t* __restrict__ rank_out) {
  constexpr int kRuns = 16 * R, kGroups = R * kSortWaves;                      // of more than kBinMax pairs each: fewer than 1024 R / 64
  static_assert(kRuns * kGroups <= 2 * kBucketBins && kBinMax >= 64, "two counts a word of sh.cut");
  const int tid = threadIdx.x, wave = uniform_wave(), shift = bin_shift(lo, hi, kBucketBinBits);
  uint16_t* cnt = reinterpret_cast<uint16_t*>(sh.cut);  // [kGroups][kRuns]
  uint32_t run = (c0 > kBinMax ? 1u : 0u) + (c1 > kBinMax ? 1u : 0u), n_runs;
  const uint32_t mine = run;
  block_prefix(sh.red, run, run, n_runs);
  // first place | number of its run + 1 << 16
  sh.bin[2 * tid] = first | (c0 > kBinMax ? (run + 1u) << 16 : 0u);
  sh.bin[2 * tid + 1] = (first + c0) | (c1 > kBinMax ? (run + mine) << 16 : 0u);
  if (tid == 0) sh.bin[kBucketBins] = (uint32_t)n;
  sh.cut[tid] = 0;
  sh.cut[tid + kSortThreads] = 0;
  __syncthreads();
  const int n_bits = 32 - __clz((int)n_runs);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t w = tid + r * kSortThreads < n ? sh.bin[clamped_bin(key[r], lo, hi, shift)] >> 16 : 0u;
    uint64_t peers = __ballot(w != 0u);
    for (int b = 0; b < n_bits; ++b) {
      const bool bit = (w >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    if (w != 0u) {
      slot[r] = lanes_below(peers);
      if (slot[r] == 0u) cnt[(r * kSortWaves + wave) * kRuns + (int)w - 1] = (uint16_t)__popcll(peers);
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  if (tid < (int)n_runs) {
    uint32_t sum = 0;
    for (int g = 0; g < kGroups; g += 16) {             // 16 reads in flight together
      uint32_t c[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) c[q] = cnt[(g + q) * kRuns + tid];
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        cnt[(g + q) * kRuns + tid] = (uint16_t)sum;
        sum += c[q];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t w = sh.bin[clamped_bin(key[r], lo, hi, shift)], i = (w & 0xffffu) + slot[r];
      if (w >> 16 == 0u) {                              // then i < n
        sh.key[i] = key[r];
        sh.tok[i] = tok[r];
      }
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t b = clamped_bin(key[r], lo, hi, shift), w = sh.bin[b], i0 = w & 0xffffu, i1 = sh.bin[b + 1] & 0xffffu;
      uint32_t c = base + i0;
      if (w >> 16 != 0u)
        c += cnt[(r * kSortWaves + wave) * kRuns + (int)(w >> 16) - 1] + slot[r];
      else
        c += before_in_bin(sh, i0, i1, key[r], tok[r]);
      if (tok[r] < (uint32_t)T) rank_out[tok[r]] = (int32_t)c;               // always true
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
}

// Ranks of the bucket's pairs (as bucket_by_bins has them) where the bins longer than kBinMax lie together, which is what keys
// close to each other beside outliers do: the bins from the first of them to the last are cut into 2048 in turn, between the
// smallest and the largest key there.  Returns false, with sh.key and sh.tok as they were, where that is not enough.
// (Ranking alone, us, these buckets by digits and so: a million scores within 2 % beside 64 outliers, pooled over 7, 68, 56; 40000
// denormal ones 27, 20.  A try that fails costs ~1.5.)
template <int R>
__device__ __forceinline__ bool bucket_by_two_levels(BucketShared& sh, int n, uint32_t lo, uint32_t hi, const uint32_t (&key)[R],
                                                     const uint32_t (&tok)[R], uint32_t (&slot)[R], uint32_t c0, uint32_t c1, uint32_t first,
                                                     uint32_t base, int T, int32_t* __restrict__ rank_out) {
  const int tid = threadIdx.x, shift = bin_shift(lo, hi, kBucketBinBits);
  uint32_t b0 = c0 > kBinMax ? 2u * tid : c1 > kBinMax ? 2u * tid + 1u : 0xffffffffu, b1 = c1 > kBinMax ? 2u * tid + 1u : c0 > kBinMax ? 2u * tid : 0u;
  block_min_max(sh.red, b0, b1);
  if (b1 - b0 >= (uint32_t)kBucketBins / 8u) return false;                     // uniform: they do not lie together
  uint32_t k0 = 0xffffffffu, k1 = 0u;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t b = clamped_bin(key[r], lo, hi, shift);
    const bool in = b >= b0 && b <= b1;                 // positions past the end repeat the last pair
    k0 = min(k0, in ? key[r] : 0xffffffffu);
    k1 = max(k1, in ? key[r] : 0u);
  }
  sh.cut[tid] = 0;
  sh.cut[tid + kSortThreads] = 0;
  sh.bin[2 * tid] = 0;
  sh.bin[2 * tid + 1] = 0;
  block_min_max(sh.red, k0, k1);
  const int shift2 = bin_shift(k0, k1, kBucketBinBits);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t b = clamped_bin(key[r], lo, hi, shift);
    if (tid + r * kSortThreads < n) slot[r] = atomicAdd(b >= b0 && b <= b1 ? &sh.cut[(key[r] - k0) >> shift2] : &sh.bin[b], 1u);
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  const uint32_t a0 = sh.cut[2 * tid], a1 = sh.cut[2 * tid + 1];
  uint32_t at, total, most;
  block_scan<true>(sh.red, a0 + a1, max(a0, a1), at, total, most);
  if (most > kBinMax) return false;                     // uniform
  sh.cut[2 * tid] = at;
  sh.cut[2 * tid + 1] = at + a0;
  sh.bin[2 * tid] = first;
  sh.bin[2 * tid + 1] = first + c0;
  if (tid == 0) sh.bin[kBucketBins] = (uint32_t)n;
  __syncthreads();
  const uint32_t p0 = sh.bin[b0], p1 = sh.bin[b1 + 1u];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t b = clamped_bin(key[r], lo, hi, shift);
      const uint32_t i = (b >= b0 && b <= b1 ? p0 + sh.cut[(key[r] - k0) >> shift2] : sh.bin[b]) + slot[r];   // < n
      sh.key[i] = key[r];
      sh.tok[i] = tok[r];
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t b = clamped_bin(key[r], lo, hi, shift);
      uint32_t i0, i1;
      if (b >= b0 && b <= b1) {
        const uint32_t x = (key[r] - k0) >> shift2;
        i0 = p0 + sh.cut[x];
        i1 = x + 1u < (uint32_t)kBucketBins ? p0 + sh.cut[x + 1u] : p1;
      } else {
        i0 = sh.bin[b];
        i1 = sh.bin[b + 1u];
      }
      const uint32_t c = base + i0 + before_in_bin(sh, i0, i1, key[r], tok[r]);
      if (tok[r] < (uint32_t)T) rank_out[tok[r]] = (int32_t)c;               // always true
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  return true;
}

// Ranks of the bucket's pairs where some bin is longer than kBinMax (keys close together beside outliers, or repeated): every
// bin of c >= 8 keys is cut into about c / 6 sub-bins, two counts a word of sh.bin; where every long bin is one key,
// bucket_with_runs.  key, tok, slot, c0, c1, first: as there.  Returns false, with sh.key and sh.tok as they were, where
// repeated keys share bins or a sub-bin is still too long.
// 131040 scores within 2 %, one far away: 24.2 us by digits, so 16.0; of a few values 28.4 by digits, so 26.2.
template <int R>
__device__ __forceinline__ bool bucket_by_sub_bins(BucketShared& sh, int n, uint32_t lo, uint32_t hi, uint32_t (&key)[R], uint32_t (&tok)[R],
                                                   uint32_t (&slot)[R], uint32_t c0, uint32_t c1, uint32_t first, uint32_t base, int T,
                                                   int32_t* __restrict__ rank_out) {
  const int tid = threadIdx.x, shift = bin_shift(lo, hi, kBucketBinBits);
  uint32_t alike = 0, total;                            // long bins' keys that are the one picked | those that are not << 16
#pragma unroll
  for (int r = 0; r < R; ++r)                           // any of the bin's keys
    __hip_atomic_store(&sh.cut[clamped_bin(key[r], lo, hi, shift)], key[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t b = clamped_bin(key[r], lo, hi, shift);
    if (tid + r * kSortThreads < n && sh.bin[b] > kBinMax) alike += sh.cut[b] == key[r] ? 1u : 65536u;
  }
  block_prefix(sh.red, alike, alike, total);
  if (total >> 16 == 0u) {                              // uniform
    bucket_with_runs<R>(sh, n, lo, hi, key, tok, slot, c0, c1, first, base, T, rank_out);
    return true;
  }
  if (8u * (total & 0xffffu) > total >> 16) return false;   // uniform: repeated keys, several to a bin
  auto log_of = [&](uint32_t c) { return c < 8u ? 0 : min(29 - __clz((int)c), shift); };
  const int l0 = log_of(c0), l1 = log_of(c1);
  uint32_t at, most;
  block_prefix(sh.red, (1u << l0) + (1u << l1), at, total);                    // total <= kBucketBins + kBucketCap / 4
  static_assert(kBucketCap / 4 <= kBucketBins, "two counts a word");
  sh.cut[2 * tid] = at | (uint32_t)l0 << 16;
  sh.cut[2 * tid + 1] = (at + (1u << l0)) | (uint32_t)l1 << 16;
  sh.bin[2 * tid] = 0;
  sh.bin[2 * tid + 1] = 0;
  __syncthreads();
  auto sub_of = [&](uint32_t k) {
    const uint32_t off = min(max(k, lo), hi) - lo, cut = sh.cut[off >> shift];
    return (cut & 0xffffu) + ((off & ((1u << shift) - 1u)) >> (shift - (int)(cut >> 16)));
  };
  auto first_of = [&](uint32_t b) { return (sh.bin[b >> 1] >> (16u * (b & 1u))) & 0xffffu; };
#pragma unroll
  for (int r = 0; r < R; ++r) {
    slot[r] = 0;
    if (tid + r * kSortThreads < n) {
      const uint32_t b = sub_of(key[r]), up = 16u * (b & 1u);
      slot[r] = (atomicAdd(&sh.bin[b >> 1], 1u << up) >> up) & 0xffffu;
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  const uint32_t w0 = sh.bin[2 * tid], w1 = sh.bin[2 * tid + 1];
  const uint32_t a0 = w0 & 0xffffu, a1 = w0 >> 16, a2 = w1 & 0xffffu, a3 = w1 >> 16;
  block_scan<true>(sh.red, a0 + a1 + a2 + a3, max(max(a0, a1), max(a2, a3)), at, total, most);
  if (most > kBinMax) return bucket_by_two_levels<R>(sh, n, lo, hi, key, tok, slot, c0, c1, first, base, T, rank_out);   // uniform
  sh.bin[2 * tid] = at | (at + a0) << 16;               // first places, at most n < 2^16
  sh.bin[2 * tid + 1] = (at + a0 + a1) | (at + a0 + a1 + a2) << 16;
  if (tid == 0) sh.bin[kBucketBins] = (uint32_t)n;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t i = first_of(sub_of(key[r])) + slot[r];     // < n
      sh.key[i] = key[r];
      sh.tok[i] = tok[r];
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t b = sub_of(key[r]), i0 = first_of(b), i1 = first_of(b + 1u);
      const uint32_t c = base + i0 + before_in_bin(sh, i0, i1, key[r], tok[r]);
      if (tok[r] < (uint32_t)T) rank_out[tok[r]] = (int32_t)c;               // always true
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  return true;
}

// Ranks of the bucket's n <= R * kSortThreads pairs in sh.key / sh.tok, whose keys lie in or near [lo, hi]: that range is cut
// into 2048 bins of equal width, a key's place is its bin's first plus the smaller keys of its bin.  sh.bin is clear.
// A count, a scan and a short loop over the own bin; the order of the atomic additions decides only where inside its
// bin a key waits to be compared.  Where a bin is longer than kBinMax, see bucket_by_sub_bins.
template <int R>
__device__ __forceinline__ bool bucket_by_bins(BucketShared& sh, int n, uint32_t lo, uint32_t hi, uint32_t base, int T,
                                               int32_t* __restrict__ rank_out) {
  const int tid = threadIdx.x, shift = bin_shift(lo, hi, kBucketBinBits);
  uint32_t key[R], tok[R], slot[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = min(tid + r * kSortThreads, n - 1);
    key[r] = sh.key[e];
    tok[r] = sh.tok[e];
    slot[r] = 0;
    if (tid + r * kSortThreads < n) slot[r] = atomicAdd(&sh.bin[clamped_bin(key[r], lo, hi, shift)], 1u);
    if (R > 2) __builtin_amdgcn_sched_barrier(0);       // one element's temporaries at a time: 64 registers are all there are
  }
  __syncthreads();
  const uint32_t c0 = sh.bin[2 * tid], c1 = sh.bin[2 * tid + 1];
  uint32_t first, total, most;
  block_scan<true>(sh.red, c0 + c1, max(c0, c1), first, total, most);
  if (__builtin_expect(most > kBinMax, 0)) {            // uniform
    if constexpr (R > 4) return bucket_by_two_levels<R>(sh, n, lo, hi, key, tok, slot, c0, c1, first, base, T, rank_out);
    else return bucket_by_sub_bins<R>(sh, n, lo, hi, key, tok, slot, c0, c1, first, base, T, rank_out);
  }
  sh.bin[2 * tid] = first;
  sh.bin[2 * tid + 1] = first + c0;
  if (tid == 0) sh.bin[kBucketBins] = (uint32_t)n;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t i = sh.bin[clamped_bin(key[r], lo, hi, shift)] + slot[r];   // < n
      sh.key[i] = key[r];
      sh.tok[i] = tok[r];
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (tid + r * kSortThreads < n) {
      const uint32_t b = clamped_bin(key[r], lo, hi, shift), i0 = sh.bin[b], i1 = sh.bin[b + 1];
      const uint32_t c = base + i0 + before_in_bin(sh, i0, i1, key[r], tok[r]);
      if (tok[r] < (uint32_t)T) rank_out[tok[r]] = (int32_t)c;               // always true
    }
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
  }
  return true;
}

// Pair number i of the bucket (i < seg_off[n_tiles]).
template <typename Args>
__device__ __forceinline__ uint2 bucket_pair(const BucketShared& sh, const Args& a, uint32_t i) {
  int t = 0;                                            // last tile whose pairs begin at or before i
  for (int step = a.tile_step; step > 0; step >>= 1)
    if (t + step < a.n_tiles && sh.seg_off[t + step] <= i) t += step;
  const uint32_t p = sh.seg_src[t] + (i - sh.seg_off[t]);
  return a.pairs[min(p, (uint32_t)a.T - 1u)];           // p < T
}

// Next range [from, to] of a large bucket's keys, `from` given: as many bins as LDS holds the pairs of, or (true) the
// single key from = to, which has more.  At least one pair has a key >= from; returns with to < from if none has.
__device__ __forceinline__ bool next_range(BucketShared& sh, const BucketShared::Pairs& a, uint32_t n, uint32_t& from, uint32_t& to) {
  const int tid = threadIdx.x;
  to = 0xffffffffu;
  for (;;) {                                            // at most three trips: 11 bits of the range each
    const int shift = bin_shift(from, to, kBucketBinBits);
    __syncthreads();
    sh.bin[2 * tid] = 0;
    sh.bin[2 * tid + 1] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < n; i += kSortThreads) {
      const uint32_t k = bucket_pair(sh, a, i).x;
      if (k >= from && k <= to) atomicAdd(&sh.bin[(k - from) >> shift], 1u);
    }
    __syncthreads();
    const uint32_t c0 = sh.bin[2 * tid], c1 = sh.bin[2 * tid + 1];
    uint32_t first, total, most;
    block_scan<true>(sh.red, c0 + c1, 0u, first, total, most);
    // leading bins that fit together, and how many pairs they hold
    const uint32_t i0 = first + c0, i1 = i0 + c1;
    uint32_t fit = i1 <= (uint32_t)kBucketCap ? 2u * tid + 2u : i0 <= (uint32_t)kBucketCap ? 2u * tid + 1u : 0u;
    uint32_t held = i1 <= (uint32_t)kBucketCap ? i1 : i0 <= (uint32_t)kBucketCap ? i0 : 0u;
    uint32_t lowest = 0u;
    block_min_max(sh.red, lowest, fit);
    block_min_max(sh.red, lowest, held);
    if (total == 0u) {                                  // cannot happen
      to = from - 1u;
      return false;
    }
    if (held > 0u) {
      if (fit < (uint32_t)kBucketBins) to = min(to, from + (fit << shift) - 1u);
      return false;
    }
    // the first bin that holds anything holds too much
    const uint32_t mask = (1u << shift) - 1u;
    from += fit << shift;
    to = to - from < mask ? to : from + mask;
    if (shift == 0) return true;
  }
}

// Buckets that bins do not order: many keys equal, or so close that the sample's bins do not tell them apart.  Up to
// what LDS holds (the pairs are there) they are ordered by digits.  Larger ones take their keys in ascending
// ranges that LDS holds, or single keys, whose order is the token order; each range costs two or more sweeps over the
// bucket's pairs by this one workgroup (128 K equal scores: one sweep to find that out, one to write the ranks).
// A function of its own, with its operands in LDS: inlined, it cost the ordinary path 60 registers or its spills.
__device__ __forceinline__ void bucket_by_ranges(BucketShared& sh) {
  const BucketShared::Pairs& a = sh.args;
  const uint32_t n = sh.n, base = sh.base;
  const bool in_lds = n <= (uint32_t)kBucketCap;
  uint32_t from = 0, to = 0xffffffffu, done = 0;        // keys below `from` are ranked: `done` of them
  while (done < n) {                                    // uniform; every trip ranks at least one pair or ends the loop
    uint32_t m = n;                                     // pairs of this trip
    bool single = false;
    if (!in_lds) {
      single = next_range(sh, a, n, from, to);
      // in token order: the pairs of the range to LDS, or the ranks of the single key
      m = 0;
      for (uint32_t i0 = 0; i0 < n; i0 += kSortThreads) {
        const uint32_t i = i0 + threadIdx.x;
        uint2 p = make_uint2(0u, 0u);
        if (i < n) p = bucket_pair(sh, a, i);
        const bool in = i < n && p.x >= from && p.x <= to;
        uint32_t at, total, most;
        block_scan<true>(sh.red, in ? 1u : 0u, 0u, at, total, most);
        at += m;
        if (in && single && p.y < (uint32_t)a.T) a.rank_out[p.y] = (int32_t)(base + done + at);
        if (in && !single && at < (uint32_t)kBucketCap) {
          sh.key[at] = p.x;
          sh.tok[at] = p.y;
        }
        m += total;
      }
      if (m == 0u) return;                              // cannot happen
      __syncthreads();
    }
    if (!single) {
      const uint32_t held = min(m, (uint32_t)kBucketCap);
      sort_by_digits<kBucketPer>(sh.key, sh.tok, sh.digit, sh.red, (int)held);
      for (uint32_t i = threadIdx.x; i < held; i += kSortThreads) {
        const uint32_t tok = sh.tok[i];
        if (tok < (uint32_t)a.T) a.rank_out[tok] = (int32_t)(base + done + i);   // always true
      }
    }
    __syncthreads();
    done += m;
    from = to + 1u;                                     // to = 2^32 - 1: nothing is left
  }
}

// Launch 2 for bucket b: collects its pairs, a stretch from every tile, and writes their ranks.  The tiles' counts say
// where the stretches are and how many tokens come before the bucket.
__device__ __forceinline__ void bucket_body(BucketShared& sh, const RankArgs& a, int b) {
  const int tid = threadIdx.x, B = a.n_buckets, n_tiles = a.n_tiles;
  uint32_t start = 0, cnt = 0;
  if (tid < n_tiles) {                                  // n_tiles <= kRankMaxTiles <= kSortThreads
    const uint32_t w = a.count[(int64_t)tid * B + b];
    start = w & 0xffffu;
    cnt = w >> 16;
  }
  uint32_t lo = a.edge[b], hi = a.edge[b + 1];
  const bool no_edges = a.edge[B + 1] != 0u;
  const uint32_t s0 = a.edge[0], s1 = a.edge[B];        // smallest and largest sampled key
  const bool outer = no_edges || lo == s0 || hi == s1;  // uniform: the edges don't say where the keys are
  if (b + 1 < B && hi > lo) hi -= 1u;
  if (no_edges) {
    lo = 0xffffffffu;
    hi = 0u;
  }
  sh.bin[2 * tid] = 0;
  sh.bin[2 * tid + 1] = 0;
  uint32_t at, n, base;
  block_scan<false>(sh.red, cnt, start, at, n, base);
  if (tid < n_tiles) {
    sh.seg_off[tid] = at;
    sh.seg_src[tid] = ((uint32_t)tid << a.tile_log) + start;
  }
  if (tid == 0) sh.seg_off[n_tiles] = n;
  __syncthreads();
  if (n == 0u) return;                                  // uniform
  const bool in_lds = n <= (uint32_t)kBucketCap;        // uniform
  if (in_lds) {
    // pair by pair, each looking up its tile: stretches may be as uneven as they like (a bucket of equal scores is a
    // run of tokens)
    for (uint32_t i = tid; i < n; i += 2 * kSortThreads) {
      const uint32_t i2 = i + kSortThreads < n ? i + kSortThreads : i;
      const uint2 p = bucket_pair(sh, a, i), p2 = bucket_pair(sh, a, i2);
      sh.key[i] = p.x;
      sh.tok[i] = p.y;
      sh.key[i2] = p2.x;
      sh.tok[i2] = p2.y;
    }
    __syncthreads();
    if (outer) {
      for (uint32_t i = tid; i < n; i += kSortThreads) {
        lo = min(lo, sh.key[i]);
        hi = max(hi, sh.key[i]);
      }
      block_min_max(sh.red, lo, hi);
      if (lo == hi) {                                   // uniform: a share of a key's tokens, in token order
        for (uint32_t i = tid; i < n; i += kSortThreads) a.rank_out[min(sh.tok[i], (uint32_t)a.T - 1u)] = (int32_t)(base + i);   // < T
        return;
      }
      // keys far beyond all sampled ones (few) stay with the bins at the ends
      const uint32_t far = (s1 - s0) / 4u + 1u, least = s0 > far ? s0 - far : 0u, last = s1 < 0xffffffffu - far ? s1 + far : 0xffffffffu;
      if (max(lo, least) <= min(hi, last)) {
        lo = max(lo, least);
        hi = min(hi, last);
      }
    }
    if (n <= 2u * kSortThreads   ? bucket_by_bins<2>(sh, (int)n, lo, hi, base, a.T, a.rank_out)
        : n <= 4u * kSortThreads ? bucket_by_bins<4>(sh, (int)n, lo, hi, base, a.T, a.rank_out)
                                 : bucket_by_bins<kBucketPer>(sh, (int)n, lo, hi, base, a.T, a.rank_out))
      return;
  }
  if (tid == 0) {
    sh.args = {a.pairs, a.rank_out, a.T, n_tiles, a.tile_step};
    sh.n = n;
    sh.base = base;
  }
  __syncthreads();
  bucket_by_ranges(sh);
}

// Geometry of a ranking of T scores (T <= kRankMaxT), without its operands.
RankArgs rank_plan(int T);
// ... with the workspace's buffers.  sample: rank_plan(T).n_s keys of s in compact form, or null.
RankArgs rank_args(const Workspace& ws, const float* s, int T, const uint32_t* sample, int32_t* rank_out);

}  // namespace asl
