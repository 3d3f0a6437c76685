// A row's sample in LDS: what the top-k takes its bound from (select_body.h) and the ranking the borders of its
// buckets (rank_body.h).  Every workgroup that needs either works it out from the same few thousand sampled keys: one
// histogram of 4096 bins of equal width over the sample's range resolves both (~1.5 us beside the workgroup's own
// loads), where a launch in front of it that did so once per row took 8 us, boundary included.
#pragma once
#include "asl_internal.h"

namespace asl {

constexpr int kRowThreads = 1024;                      // workgroup of the ranking and of the selection kernels
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kSampleBins = 4 * kRowThreads;           // four neighbouring bins per thread
constexpr int kSampleBinBits = 12;
constexpr int kSamplePer = kSelMaxSample / kRowThreads;
static_assert(kSampleBins == 1 << kSampleBinBits && kSelMaxSample % kRowThreads == 0, "sample geometry");

struct SampleShared {
  uint4 bin[kRowThreads];                              // [kSampleBins]
  uint32_t red[2 * kRowWaves];
  uint32_t out[4];
};

// Keys u * kRowThreads + tid of a sample of n_s keys (positions past its end repeat another of its keys): compact in
// `sample`, or, where that is null, read from the row itself.  All loads are in flight together.
__device__ __forceinline__ void load_sample(const float* __restrict__ row, const uint32_t* __restrict__ sample, int n_s, int stride,
                                            uint32_t (&v)[kSamplePer]) {
  const int tid = threadIdx.x;
  if (sample != nullptr) {
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u)
      if (u * kRowThreads < n_s) v[u] = sample[min(tid + u * kRowThreads, n_s - 1)];          // uniform
  } else {
    float f[kSamplePer];
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u)
      if (u * kRowThreads < n_s) f[u] = row[sel_sample_position((uint32_t)min(tid + u * kRowThreads, n_s - 1), stride)];
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u) v[u] = u * kRowThreads < n_s ? order_key(f[u]) : 0u;
  }
#pragma unroll
  for (int u = 1; u < kSamplePer; ++u)
    if (u * kRowThreads >= n_s) v[u] = v[0];
}

// The wavefronts' totals red[0 .. kRowWaves - 1], one per lane of a row of 16, summed along the row; lane 15 of the
// result has the sum.  (Every thread reading all totals held 32 registers and as many masks.)
static_assert(kRowWaves == 16, "one row of lanes");
__device__ __forceinline__ uint32_t row_prefix_sum(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);   // row_shr:8
  return x;
}
__device__ __forceinline__ int uniform_wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

// Smallest and largest of the workgroup's values.
__device__ __forceinline__ void block_min_max(uint32_t* red, uint32_t& lo, uint32_t& hi) {
  const int wave = uniform_wave(), lane = threadIdx.x & 63;
  lo = wave_min(lo);
  hi = wave_max(hi);
  __syncthreads();                                     // red may still be in use
  if (lane == 0) {
    red[wave] = lo;
    red[kRowWaves + wave] = hi;
  }
  __syncthreads();
  lo = wave_min(red[lane & (kRowWaves - 1)]);
  hi = wave_max(red[kRowWaves + (lane & (kRowWaves - 1))]);
}

// Exclusive prefix over the workgroup's threads of `x`, and its total.
__device__ __forceinline__ void block_prefix(uint32_t* red, uint32_t x, uint32_t& excl, uint32_t& total) {
  const int wave = uniform_wave(), lane = threadIdx.x & 63;
  const uint32_t incl = wave_prefix_sum(x);
  __syncthreads();                                     // red may still be in use
  if (lane == 63) red[wave] = incl;
  __syncthreads();
  const uint32_t before = row_prefix_sum(red[lane & (kRowWaves - 1)]);
  total = (uint32_t)__builtin_amdgcn_readlane((int)before, kRowWaves - 1);
  excl = incl - x + (wave == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)before, wave - 1));
}

// Exclusive prefix over the workgroup's threads of `x`, its total, and the total of `y` (MAX: its largest).
template <bool MAX>
__device__ __forceinline__ void block_scan(uint32_t* red, uint32_t x, uint32_t y, uint32_t& excl, uint32_t& total, uint32_t& y_total) {
  const int wave = uniform_wave(), lane = threadIdx.x & 63;
  const uint32_t incl = wave_prefix_sum(x), yw = MAX ? wave_max(y) : wave_sum(y);
  __syncthreads();                                     // red may still be in use
  if (lane == 63) {
    red[wave] = incl;
    red[kRowWaves + wave] = yw;
  }
  __syncthreads();
  const uint32_t before = row_prefix_sum(red[lane & (kRowWaves - 1)]), ys = red[kRowWaves + (lane & (kRowWaves - 1))];
  total = (uint32_t)__builtin_amdgcn_readlane((int)before, kRowWaves - 1);
  excl = incl - x + (wave == 0 ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)before, wave - 1));
  y_total = MAX ? wave_max(ys) : (uint32_t)__builtin_amdgcn_readlane((int)row_prefix_sum(ys), kRowWaves - 1);
}

// Shift that maps key - lo, for keys in [lo, hi], to fewer than 2^bits bins.
__device__ __forceinline__ int bin_shift(uint32_t lo, uint32_t hi, int bits) {
  const uint32_t span = hi - lo;
  const int b = span == 0 ? 0 : 32 - __clz((int)span);
  return b > bits ? b - bits : 0;
}
__device__ __forceinline__ uint32_t clamped_bin(uint32_t key, uint32_t lo, uint32_t hi, int shift) {
  return (min(max(key, lo), hi) - lo) >> shift;
}

// LDS atomics of a wavefront on one word come one after the other, ~4 cycles a lane.  Words that two of the wavefront's
// lanes want, if at least a sixth of it does (else 2^32 - 1): their lanes then add together.  Looked for only where some
// neighbours want the same word: counting words that hardly repeat must not pay for it (a few instructions, 0.1 us).
struct Repeated {
  uint32_t w0, w1;
  __device__ __forceinline__ bool none() const { return __builtin_expect((w0 & w1) == 0xffffffffu, 1); }
};
__device__ __forceinline__ Repeated find_repeated(uint32_t i, bool valid) {
  Repeated r = {0xffffffffu, 0xffffffffu};
  const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp((int)~i, (int)i, 0x111, 0xf, 0xf, false);   // row_shr:1
  if (__builtin_expect(__popcll(__ballot(valid && i == next)) < 3, 1)) return r;                          // uniform
  r.w0 = (uint32_t)__builtin_amdgcn_readlane((int)i, 0);
  r.w1 = (uint32_t)__builtin_amdgcn_readlane((int)i, 37);
  if (__popcll(__ballot(valid && i == r.w0)) < 11) r.w0 = 0xffffffffu;
  if (r.w1 == r.w0 || __popcll(__ballot(valid && i == r.w1)) < 11) r.w1 = 0xffffffffu;
  return r;
}
// What the lane adds to word i (0: another lane adds for it).  The whole wavefront calls it.
__device__ __forceinline__ uint32_t add_for(const Repeated& r, uint32_t i, bool valid) {
  const uint64_t m0 = __ballot(valid && i == r.w0), m1 = __ballot(valid && i == r.w1), mine = i == r.w0 ? m0 : m1;
  if (!valid) return 0u;
  if (i != r.w0 && i != r.w1) return 1u;
  return lanes_below(mine) == 0u ? (uint32_t)__popcll(mine) : 0u;
}

// Adds one to bin[i] for every valid lane and returns what it was before, lanes of one word in order.  The whole wavefront
// calls it.
__device__ __forceinline__ uint32_t slot_for(const Repeated& r, uint32_t* bin, uint32_t i, bool valid) {
  const uint64_t m0 = __ballot(valid && i == r.w0), m1 = __ballot(valid && i == r.w1), mine = i == r.w0 ? m0 : m1;
  const bool shared = i == r.w0 || i == r.w1;
  const uint32_t below = lanes_below(mine);
  uint32_t old = 0;
  if (valid && (!shared || below == 0u)) old = atomicAdd(&bin[i], shared ? (uint32_t)__popcll(mine) : 1u);
  const uint32_t b0 = m0 != 0ull ? (uint32_t)__builtin_amdgcn_readlane((int)old, __ffsll((unsigned long long)m0) - 1) : 0u;
  const uint32_t b1 = m1 != 0ull ? (uint32_t)__builtin_amdgcn_readlane((int)old, __ffsll((unsigned long long)m1) - 1) : 0u;
  return !shared ? old : (i == r.w0 ? b0 : b1) + below;
}

// Counts the sample's keys in bins of width 2^shift from lo: all of them (ALL: they are in [lo, hi], and many may want the
// same bin), or those in [lo, hi].
template <bool ALL>
__device__ __forceinline__ void sample_count(SampleShared& sh, const uint32_t (&v)[kSamplePer], int n_s, uint32_t lo, uint32_t hi, int shift) {
  const int tid = threadIdx.x;
  uint32_t* bin = &sh.bin[0].x;
  sh.bin[tid] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  auto in = [&](int u) { return tid + u * kRowThreads < n_s && (ALL || (v[u] >= lo && v[u] <= hi)); };
  const Repeated rep = ALL ? find_repeated((v[0] - lo) >> shift, in(0)) : Repeated{0xffffffffu, 0xffffffffu};
  if (!ALL || rep.none()) {                            // uniform
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u)
      if (in(u)) atomicAdd(&bin[(v[u] - lo) >> shift], 1u);
  } else {
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u)
      if (u * kRowThreads < n_s) {
        const uint32_t n = add_for(rep, (v[u] - lo) >> shift, in(u));
        if (n != 0u) atomicAdd(&bin[(v[u] - lo) >> shift], n);
      }
  }
  __syncthreads();
}

// The m-th smallest key of the sample (1 <= m <= n_s), rounded up to its bin's last key: `bound` lets at most `slack`
// more of the sample's keys pass (further rounds, 4096 bins within the bin, until that holds).  `below`: the first
// key of the bin that holds the m_low-th key (m_low <= m).
__device__ __forceinline__ void sample_bound(SampleShared& sh, const uint32_t (&v)[kSamplePer], int n_s, uint32_t m, uint32_t m_low,
                                             uint32_t slack, uint32_t& bound, uint32_t& below) {
  const int tid = threadIdx.x;
  uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int u = 0; u < kSamplePer; ++u) {
    lo = min(lo, v[u]);
    hi = max(hi, v[u]);
  }
  block_min_max(sh.red, lo, hi);
  below = lo;
  for (int round = 0;; ++round) {
    const int shift = bin_shift(lo, hi, kSampleBinBits);
    sample_count<false>(sh, v, n_s, lo, hi, shift);
    const uint4 c = sh.bin[tid];
    uint32_t excl, total, most;
    block_scan<true>(sh.red, c.x + c.y + c.z + c.w, 0u, excl, total, most);
    const uint32_t cs[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t incl = excl + cs[q];
      if (excl < m && m <= incl) {                     // exactly one bin of the workgroup
        sh.out[0] = (uint32_t)(4 * tid + q);
        sh.out[1] = m - excl;
        sh.out[2] = incl - m;
      }
      if (excl < m_low && m_low <= incl) sh.out[3] = (uint32_t)(4 * tid + q);
      excl = incl;
    }
    __syncthreads();
    const uint32_t first = lo + (sh.out[0] << shift), mask = (1u << shift) - 1u,
                   last = hi - first < mask ? hi : first + mask, over = sh.out[2];
    if (round == 0) below = lo + (sh.out[3] << shift);
    if (over <= slack || shift == 0) {                 // uniform
      bound = last;
      return;
    }
    m = sh.out[1];
    m_low = 0;
    lo = first;
    hi = last;
  }
}

}  // namespace asl
