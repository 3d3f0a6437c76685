// asl_rank: RankDesc of the all-head score vector (Alg. 1 step 11 of the paper):
// rank[t] = position of t in the order (score descending, token index ascending).
//
// Keys are an order-preserving 32-bit transform of the fp32 score.  Two launches that wait for nothing but each
// other's end (rank_body.h):
//  1. partition  a sample of the vector cuts the key range into buckets of ~512 tokens; every tile groups its own
//                tokens by bucket, in place, and notes where each bucket's begin;
//  2. buckets    one workgroup per bucket collects the bucket's tokens from all tiles, orders them in LDS and writes
//                their ranks: what comes before the bucket is the sum of the tiles' notes.
// The sample decides only how even the buckets are; a bucket that outgrows LDS is ordered from memory.
// (Four passes of an LSD radix sort with the tiles' counts exchanged inside each launch took 33.5 us at 131040 tokens
// and 101 us at a million; this takes 16 and 31.)
//
// Short vectors (kShortT) are ranked in one launch instead (rank_short_body), unless the ranks overwrite the scores.
#include <cstdio>
#include <mutex>

#include "rank_stat_body.h"

namespace asl {

// Rows of n_s keys from `s`, one per stride (see load_sample), in compact form.
__global__ void __launch_bounds__(256) rank_sample_kernel(const float* __restrict__ s, int n_s, int stride, uint32_t* __restrict__ out) {
  const uint32_t j = blockIdx.x * 256 + threadIdx.x;
  if (j < (uint32_t)n_s) out[j] = order_key(s[sel_sample_position(j, stride)]);
}

template <int R>
__global__ void __launch_bounds__(kSortThreads) rank_partition_kernel(RankArgs a) {
  __shared__ PartShared sh;
  partition_body<R>(sh, a, (int)blockIdx.x);
}

// dynamic LDS: sizeof(BucketShared)
__global__ void __launch_bounds__(kSortThreads, 8) rank_bucket_kernel(RankArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  bucket_body(*reinterpret_cast<BucketShared*>(lds_dyn), a, (int)blockIdx.x);
}

// dynamic LDS: sizeof(ShortRankShared)
__global__ void __launch_bounds__(kSortThreads) rank_short_kernel(const float* __restrict__ s, int T, int32_t* __restrict__ rank_out) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  rank_short_body(*reinterpret_cast<ShortRankShared*>(lds_dyn), s, T, PutRank{rank_out}, (int)blockIdx.x);
}

// dynamic LDS: sizeof(RankStatShared)
__global__ void __launch_bounds__(kSortThreads) rank_stat_short_kernel(const float* __restrict__ s, int32_t* __restrict__ rank_row, RankvarArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_dyn[];
  rank_stat_short_body(*reinterpret_cast<RankStatShared*>(lds_dyn), s, rank_row, a, (int)blockIdx.x, (int)gridDim.x);
}

RankArgs rank_plan(int T) {
  RankArgs a = {};
  a.T = T;
  a.tile_log = T <= 131072 ? 11 : T <= 1048576 ? 12 : 13;     // up to 64 tiles, then up to 256
  a.n_tiles = (T + (1 << a.tile_log) - 1) >> a.tile_log;
  a.tile_step = 1;
  while (2 * a.tile_step < a.n_tiles) a.tile_step *= 2;
  // ~512 tokens a bucket, more where that keeps them to one round of workgroups: one per compute unit (240, beside the
  // top-k's) up to ~1100 tokens a bucket, two up to 2048, which is the most that four pairs a thread take without many
  // buckets going beyond.  Ranking + statistic, us, with 512 buckets and with one per 1024 tokens: 400 K tokens 28.8, 29.3;
  // 700 K 36.0, 39.7; 1 M 43.5, 57.7; 2 M 135, 72.7 (there: 1024).
  a.n_buckets = (T + 511) / 512;
  if (a.n_buckets > 240) a.n_buckets = T <= 264000 ? 240 : T <= 512 * 2048 ? 512 : (T + 2047) / 2048;
  if (a.n_buckets > kRankMaxBuckets) a.n_buckets = kRankMaxBuckets;
  a.n_s = sel_sample_size(T);
  a.stride = sel_sample_stride(T);
  // three buckets' worth, or two where a bucket with the end of one before it would outgrow kBucketCap
  a.heavy = (T / a.n_buckets > 1400 ? 2 * a.n_s : 3 * a.n_s) / a.n_buckets;
  a.per_key = (float)a.n_buckets / (float)a.n_s;
  a.per_key_deep = (float)(a.n_buckets - 1) / (float)a.n_s;
  return a;
}

RankArgs rank_args(const Workspace& ws, const float* s, int T, const uint32_t* sample, int32_t* rank_out) {
  RankArgs a = rank_plan(T);
  a.s = s;
  a.sample = sample;
  a.pairs = ws.rank_pairs;
  a.count = ws.rank_count;
  a.edge = ws.rank_edge;
  a.rank_out = rank_out;
  return a;
}

// Sampled keys that the partition's workgroups read straight from the vector, each for itself; beyond, a launch in front
// of it collects them.
constexpr int64_t kSampleDirect = 64 * 4096;

// Whether a ranking is one launch.  Its workgroups read all scores while others already write ranks; the partition reads them in its
// first launch and writes ranks in its last, so it takes the calls that rank a vector in place.
static bool one_launch(const float* s, int T, const int32_t* rank_out) {
  const uintptr_t s0 = reinterpret_cast<uintptr_t>(s), r0 = reinterpret_cast<uintptr_t>(rank_out), bytes = (uintptr_t)T * 4;
  const bool in_place = s0 < r0 + bytes && r0 < s0 + bytes;
  return T <= kShortT && !in_place;
}

hipError_t launch_rank_stat(const Workspace& ws, const float* s, int32_t* rank_row, const RankvarArgs& stat, hipStream_t st) {
  if (one_launch(s, stat.T, rank_row)) {
    static OncePerDevice once;
    const hipError_t attr = allow_lds(once, reinterpret_cast<const void*>(rank_stat_short_kernel), sizeof(RankStatShared));
    if (attr != hipSuccess) return attr;
    ASL_LAUNCH(ws.prof, kKernSortScatter, st, rank_stat_short_kernel, dim3(short_rank_blocks(stat.T)), dim3(kSortThreads),
               sizeof(RankStatShared), st, s, rank_row, stat);
    return hipGetLastError();
  }
  const hipError_t e = launch_rank(ws, s, stat.T, rank_row, st);
  if (e != hipSuccess) return e;
  if (stat.skip != 0) return launch_stat_skip(ws.prof, stat.out, stat.state, stat.layer_idx, stat.l_obs, stat.push, st);
  return launch_rankvar(ws, stat.ring, stat.l_obs, stat.T, stat.layer_idx, stat.k, stat.tau, stat.push, stat.state, stat.out, st);
}

hipError_t launch_rank(const Workspace& ws, const float* s, int T, int32_t* rank_out, hipStream_t st) {
  if (one_launch(s, T, rank_out)) {
    static OncePerDevice once;
    const hipError_t attr = allow_lds(once, reinterpret_cast<const void*>(rank_short_kernel), sizeof(ShortRankShared));
    if (attr != hipSuccess) return attr;
    ASL_LAUNCH(ws.prof, kKernSortScatter, st, rank_short_kernel, dim3(short_rank_blocks(T)), dim3(kSortThreads), sizeof(ShortRankShared), st,
               s, T, rank_out);
    return hipGetLastError();
  }
  if (T > kRankMaxT) return hipErrorInvalidConfiguration;
  static OncePerDevice once;
  const hipError_t attr = allow_lds(once, reinterpret_cast<const void*>(rank_bucket_kernel), sizeof(BucketShared));
  if (attr != hipSuccess) return attr;
  RankArgs a = rank_args(ws, s, T, nullptr, rank_out);
  if ((int64_t)a.n_tiles * a.n_s > kSampleDirect) {
    ASL_LAUNCH(ws.prof, kKernSortHist, st, rank_sample_kernel, dim3((a.n_s + 255) / 256), dim3(256), 0, st, s, a.n_s, a.stride,
               ws.rank_sample);
    a.sample = ws.rank_sample;
  }
  const dim3 grid(a.n_tiles), block(kSortThreads);
  if (a.tile_log == 11)
    ASL_LAUNCH(ws.prof, kKernSortScatter, st, rank_partition_kernel<2>, grid, block, 0, st, a);
  else if (a.tile_log == 12)
    ASL_LAUNCH(ws.prof, kKernSortScatter, st, rank_partition_kernel<4>, grid, block, 0, st, a);
  else
    ASL_LAUNCH(ws.prof, kKernSortScatter, st, rank_partition_kernel<8>, grid, block, 0, st, a);
  ASL_LAUNCH(ws.prof, kKernSortScatter, st, rank_bucket_kernel, dim3(a.n_buckets), block, sizeof(BucketShared), st, a);
  return hipGetLastError();
}

}  // namespace asl

// ---------------------------------------------------------------------------------------------
// asl_rank_static: asl_rank for callers that cannot allocate.  The ranking's scratch (pairs, counts, bucket borders,
// sample) lives in a file-scope device array instead of a context's workspace; every call writes what it reads of it.
// In host code the array's name is only a handle: its device address is looked up once per device and that pointer
// is what the kernels get.
namespace {

constexpr int kStaticMaxT = ASL_RANK_STATIC_MAX_T;
constexpr size_t kStaticWords = 3 * (size_t)kStaticMaxT + asl::kSelMaxSample + asl::kRankMaxBuckets + 64;
static_assert(kStaticMaxT % 64 == 0 && kStaticMaxT <= asl::kRankMaxT, "keeps the buffers 256-byte aligned");

static __device__ __align__(256) uint32_t scratch[kStaticWords];

constexpr int kMaxDevices = 64;
uint32_t* g_scratch_ptr[kMaxDevices];            // device address of `scratch` on each device
std::mutex g_scratch_mutex;
thread_local char g_static_err[192] = "";

// Device address of this device's copy of `scratch` (the current device must be `device`).
hipError_t static_scratch(int device, uint32_t** out) {
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[device] == nullptr) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[device] = static_cast<uint32_t*>(ptr);
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

asl_status static_fail(asl_status st, const char* msg, const char* detail = "") {
  snprintf(g_static_err, sizeof(g_static_err), "%s%s", msg, detail);
  return st;
}

}  // namespace

namespace asl {
hipError_t rank_static_prepare(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  uint32_t* p = nullptr;
  return static_scratch(device, &p);
}
}  // namespace asl

extern "C" {
#pragma GCC visibility push(default)

asl_status asl_rank_static(const float* s, int32_t T, int32_t* rank_out, void* stream) {
  if (!s || !rank_out) return static_fail(ASL_EINVAL, "asl_rank_static: null tensor pointer");
  if (T < 1) return static_fail(ASL_EINVAL, "asl_rank_static: need T >= 1");
  if (T > kStaticMaxT) {
    char detail[64];
    snprintf(detail, sizeof(detail), " (T=%d, limit %d)", T, kStaticMaxT);
    return static_fail(ASL_ENOMEM, "asl_rank_static: T exceeds ASL_RANK_STATIC_MAX_T", detail);
  }
  int device = -1;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return static_fail(ASL_EHIP, "hipGetDevice: ", hipGetErrorString(e));
  if (device < 0 || device >= kMaxDevices) return static_fail(ASL_EUNSUPPORTED, "asl_rank_static: device index too large");
  uint32_t* base = nullptr;
  e = static_scratch(device, &base);
  if (e != hipSuccess) return static_fail(ASL_EHIP, "hipGetSymbolAddress(scratch): ", hipGetErrorString(e));
  asl::Workspace ws = {};
  ws.rank_pairs = reinterpret_cast<uint2*>(base);
  ws.rank_count = base + 2 * (size_t)kStaticMaxT;
  ws.rank_sample = base + 3 * (size_t)kStaticMaxT;
  ws.rank_edge = ws.rank_sample + asl::kSelMaxSample;
  ws.prof = nullptr;
  e = asl::launch_rank(ws, s, T, rank_out, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return static_fail(ASL_EHIP, "rank launch: ", hipGetErrorString(e));
  return ASL_OK;
}

const char* asl_static_last_error(void) { return g_static_err; }

#pragma GCC visibility pop
}  // extern "C"
