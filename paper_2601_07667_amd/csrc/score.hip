// asl_score: window-query x all-key softmax scores, column-summed over the window rows and the
// GQA group (Alg. 1 steps 5, 6, 8 of the paper; Sec. 4.1 PA equation before pooling).
//
// For one KV head the G heads x W window rows form M = G*W query rows that all read the same
// keys.  score_j = sum_r exp(l_rj - m_r) / Z_r mixes rows with different normalisers, so the
// final (m_r, Z_r) of every row must be known before rows are added: pass 1 streams K once for
// the row statistics, pass 2 streams K again for the normalised column sums.  When the caller
// hands over the rows' log-sum-exp, pass 1 is skipped.
//
// Work split: a workgroup owns one KV head and every so many-th of its key tiles (one wavefront: a contiguous share); wave w owns RB blocks of
// 32 query rows (RB = 1 up to M = 128 rows, 2 above for the main bf16 shapes) and keeps their
// fragments in registers for the whole kernel; K tiles of 64 or 32 keys stream global -> LDS directly
// (ring of 3 buffers, XOR-swizzled) and every wave reads all of them as the other MFMA operand
// (v_mfma_f32_32x32x16_bf16, or v_mfma_f32_32x32x2_f32 for fp32), each fragment once for all its row
// blocks.  Pass 1 puts keys on the accumulator's register axis (row statistics reduce in-lane), pass 2
// puts query rows there (column sums reduce in-lane).  More rows per KV head than a workgroup holds
// take further launches.  All reductions have a fixed order: results are deterministic.
#include <type_traits>

#include "asl_internal.h"
#include "score_split.h"

namespace asl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#ifndef ASL_SCORE_STAGES
#define ASL_SCORE_STAGES 3
#endif
// A key row is handled as 16-byte pieces, P of them per (padded) row: 8 bf16 or 4 fp32 elements each.
typedef uint32_t Piece __attribute__((ext_vector_type(4)));
// Keys per LDS tile (a multiple of 32): tiles of at most 16 KB up to 512-byte rows, so that the rings of
// the two or three workgroups a compute unit works best with fit it (six with 8 KB tiles; see score_chunks).
template <int P> constexpr int key_tile() { return P <= 16 ? 64 : 32; }
// LDS tile buffers of the K ring: STAGES-1 tiles in flight while one is consumed (four or more: the same
// or slower, the longer prologue costs what the depth gains).  RB = 32-row query blocks per wavefront: 1
// for M <= 128 query rows, 2 above.
constexpr int kStages = ASL_SCORE_STAGES;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kNegBig = -1.0e30f;           // finite stand-in for "no maximum yet"

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Row of the 32x32 accumulator held by register r of a lane in half `half` (lanes 32..63 = 1).
__device__ __forceinline__ int acc_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// K tile staging: global memory -> LDS directly (global_load_lds_dwordx4: each lane names its own
// 16-byte global source, the hardware writes lane i's data to  wave base + 16*i  in LDS), a ring of
// LDS buffers, one workgroup barrier per tile.  Bank conflicts on the fragment reads are avoided by an
// XOR swizzle applied on the global side: LDS slot (row r, piece c') holds the row's 16-byte piece
// c = c' ^ (r mod 16)  (mod 8 where P is no multiple of 16).
// Rows past N are clamped to the last key (they are masked or discarded later).  With PAD the row has
// only np <= P pieces: the slots behind them repeat the row's last piece; the fragments of both operands
// hold zeros there (zeros in one are not enough: 0 * Inf is NaN).
// Per-thread constants of the tile loader: for each of its NLOAD pieces the byte offset of the
// (swizzled) source piece from the tile's first key.
// The first NT threads of the workgroup do the loading, NT = the largest power of two that is at most
// the workgroup size and the number of pieces (see loader_threads): every loading wavefront then
// issues the same number of loads per tile, which the counted waits below rely on; the other
// wavefronts issue none and are held by the workgroup barrier alone.
template <int P, int NT>
struct TilePieces {
  static constexpr int KT = key_tile<P>();
  static constexpr int SWZ = (P % 16 == 0) ? 15 : 7;
  static_assert(P % 8 == 0, "the swizzle permutes the pieces of a row in aligned groups of 8 or 16");
  static constexpr int SLOTS = KT * P;
  static_assert(SLOTS % NT == 0, "loader threads must divide the pieces of a tile");
  static constexpr int NLOAD = SLOTS / NT;
  uint32_t src_off[NLOAD];
  // tile row and (swizzled) source piece of this thread's i-th load; `last` = the row's last piece
  static __device__ __forceinline__ int row(int i, int tid) { return (i * NT + tid) / P; }
  static __device__ __forceinline__ int piece(int i, int tid, int last) {
    const int q = i * NT + tid;
    return min((q % P) ^ ((q / P) & SWZ), last);
  }
  __device__ __forceinline__ void init(int64_t row_stride_bytes, int tid, int last) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) src_off[i] = (uint32_t)((int64_t)row(i, tid) * row_stride_bytes + piece(i, tid, last) * 16);
  }
};

// kg, rsb: first key of the KV head and the key stride in bytes.  AUX: cache policy of the loads (STREAM, kAuxStream: see
// stream_keys).
constexpr int kAuxPlain = 0, kAuxStream = 2;          // the non-temporal bit
template <int P, int NT, bool FULL, int AUX>
__device__ __forceinline__ void issue_tile_loads_impl(const TilePieces<P, NT>& tp, const char* __restrict__ kg,
                                                      int64_t rsb, int key0, int N, int last_piece,
                                                      Piece* __restrict__ lds_buf, int tid) {
  constexpr int NLOAD = TilePieces<P, NT>::NLOAD;
  const int wave_slot0 = __builtin_amdgcn_readfirstlane(tid) & ~63;
  if (wave_slot0 >= NT) return;                         // not a loading wavefront (wave-uniform)
  const char* tile_base = kg + (int64_t)key0 * rsb;     // uniform
  if (FULL) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const char* src = tile_base + tp.src_off[i];
      Piece* dst = lds_buf + (i * NT + wave_slot0);     // wave-uniform base
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)dst, 16, 0, AUX);
    }
  } else {
    // last, partial tile of a head: rows past N - 1 read key N - 1 instead.  Kept as a loop (it runs
    // once per head and launch; unrolled it would hold NLOAD row addresses in registers all along)
    const int last = N - 1 - key0;                        // last valid row of the tile
#pragma unroll 1
    for (int i = 0; i < NLOAD; ++i) {
      const int r = min(TilePieces<P, NT>::row(i, tid), last);
      const char* src = tile_base + (int64_t)r * rsb + TilePieces<P, NT>::piece(i, tid, last_piece) * 16;
      Piece* dst = lds_buf + (i * NT + wave_slot0);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)dst, 16, 0, AUX);
    }
  }
}

// Full tiles take the precomputed offsets; only a tile that reaches past N pays for clamping.
template <int P, int NT, bool STREAM>
__device__ __forceinline__ void issue_tile_loads(const TilePieces<P, NT>& tp, const char* __restrict__ kg, int64_t rsb,
                                                 int key0, int N, int last_piece, Piece* __restrict__ lds_buf, int tid) {
  if (key0 + key_tile<P>() <= N)
    issue_tile_loads_impl<P, NT, true, STREAM ? kAuxStream : kAuxPlain>(tp, kg, rsb, key0, N, last_piece, lds_buf, tid);
  else
    issue_tile_loads_impl<P, NT, false, kAuxPlain>(tp, kg, rsb, key0, N, last_piece, lds_buf, tid);
}

// Wait until at most CNT of this wave's vector-memory operations (incl. its LDS-direct loads) are
// still outstanding; they complete in issue order, so everything older than the last CNT is done.
// The same instruction waits for all of the wave's LDS operations (lgkmcnt 0): every use of it is
// followed by the workgroup barrier that hands this wave's LDS writes (pass 2's column partials) to
// other waves, and the wait the compiler derives from the barrier's fence was seen to disappear next
// to this hand-written one (the partials of a tile's last sub-tile were then read before they landed).
template <int CNT>
__device__ __forceinline__ void wait_vmem() {
  static_assert(CNT >= 0 && CNT < 64, "vmcnt is a 6-bit count");
  // vmcnt(CNT): low 4 bits in [3:0], high 2 bits in [15:14]; expcnt [6:4] left at "no wait"; lgkmcnt [11:8] = 0
  __builtin_amdgcn_s_waitcnt(0x0070 | (CNT & 0xF) | ((CNT >> 4) << 14));
}

// Threads of an NW-wavefront workgroup that load the K tiles.
template <int P, int NW>
constexpr int loader_threads() {
  int n = 64;
  while (n * 2 <= NW * 64 && n * 2 <= key_tile<P>() * P) n *= 2;
  return n;
}

// Top-of-iteration wait: the current tile must have landed.  `younger` = tiles issued after it that
// are still in flight (at most STAGES-2).  With a uniform per-wave load count those may stay
// outstanding; otherwise wait for everything.
template <int L, int Y>
__device__ __forceinline__ void wait_younger(int younger) {
  if constexpr (Y == 0) {
    wait_vmem<0>();
  } else {
    if (younger >= Y) wait_vmem<Y * L>();
    else wait_younger<L, Y - 1>(younger);
  }
}
template <int P, int NT, int STAGES>
__device__ __forceinline__ void wait_tile(int younger) {
  constexpr int L = TilePieces<P, NT>::NLOAD;           // loads each loading wave issues per tile
  static_assert(STAGES >= 2, "ring depth");
  if constexpr (L > 0 && L * (STAGES - 2) < 64)
    wait_younger<L, STAGES - 2>(younger);
  else
    wait_vmem<0>();
}

// K fragment of step ks for the 32-key sub-tile `sub`: lane (ln, half) holds piece 2*ks + half of key
// ln (un-swizzled here).  The query fragments hold the same pieces of their rows, so whatever elements
// a step covers, both operands of its MFMAs cover the same ones.
template <int P>
__device__ __forceinline__ Piece load_k_frag(const Piece* buf, int sub, int ln, int half, int ks) {
  const int r = sub * 32 + ln;
  return buf[r * P + ((2 * ks + half) ^ (r & TilePieces<P, 64>::SWZ))];
}

// One fragment step: a 32x32x16 bf16 MFMA, or the four 32x32x2 fp32 MFMAs whose two elements per row
// are element i of the two lane halves' pieces.
template <typename TE>
__device__ __forceinline__ f32x16 mma_step(const Piece& a, const Piece& b, f32x16 acc) {
  if constexpr (sizeof(TE) == 2) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  } else {
    const f32x4 av = __builtin_bit_cast(f32x4, a), bv = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], bv[i], acc, 0, 0, 0);
    return acc;
  }
}

// Shortest row, in pieces, that a padded row length P is used for (see dispatch_padded).
template <int P> constexpr int least_pieces() { return P <= 32 ? P - 7 : P - 15; }

// QK^T of one 32-key sub-tile against this wave's RB blocks of 32 query rows (P/2 chained steps
// per block; every K fragment is read from LDS once and used for all RB blocks).
// KEYS_ON_REGS: accumulator register axis = keys (pass 1), else = query rows (pass 2).
// PAD: pieces from np on are zeros; only the steps that a padded row can end in pay for the test.
template <typename TE, int P, bool KEYS_ON_REGS, int RB, bool PAD>
__device__ __forceinline__ void mma_subtile(const Piece* __restrict__ buf, int sub, int ln, int half, int np,
                                            const Piece (&qf)[RB][P / 2], f32x16 (&acc)[RB]) {
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[rb][r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < P / 2; ++ks) {
    Piece kf = load_k_frag<P>(buf, sub, ln, half, ks);
    if (PAD && 2 * ks + 1 >= least_pieces<P>() && 2 * ks + half >= np) kf = Piece{0u, 0u, 0u, 0u};
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      acc[rb] = KEYS_ON_REGS ? mma_step<TE>(kf, qf[rb][ks], acc[rb]) : mma_step<TE>(qf[rb][ks], kf, acc[rb]);
  }
}

// Query fragments of this wave's RB 32-row blocks (block rb = rows row0 + 32*rb ..): lane (ln, half)
// holds pieces 2*ks + half of row ln of each block; pieces from np on are zeros.  Rows from m1 on, whose
// results are dropped, repeat row m1 - 1: their logits are then whatever a real row's are (a row of zeros
// would make NaN of an infinite key and of pass 2's column sum over it).
#define ASL_LOAD_Q_FRAGS()                                                                        \
  Piece qf[RB][KS];                                                                               \
  _Pragma("unroll") for (int rb = 0; rb < RB; ++rb) {                                             \
    const int qr_ = row0 + rb * 32 + ln;                                                          \
    const Piece* qg_ = reinterpret_cast<const Piece*>(q_obs) + ((int64_t)g * M + min(qr_, m1 - 1)) * (PAD ? np : P); \
    _Pragma("unroll") for (int ks = 0; ks < KS; ++ks) {                                           \
      const int c_ = 2 * ks + half;                                                               \
      Piece raw_ = qg_[PAD ? min(c_, np - 1) : c_];                                               \
      if (PAD && c_ >= np) raw_ = Piece{0u, 0u, 0u, 0u};                                          \
      qf[rb][ks] = raw_;                                                                          \
    }                                                                                             \
  }
// Wait for the query fragments here (the loads issued after theirs stay in flight): without it the compiler waits at
// their first use, which is inside the tile loop and would be met in every round (8B shape, 128K, `lse` supplied, 65.1
// us without, 63.0 with).
#define ASL_WAIT_Q_FRAGS()                                                                        \
  _Pragma("unroll") for (int rb = 0; rb < RB; ++rb)                                               \
    _Pragma("unroll") for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[rb][ks]));


// This file is compiled with NaNs assumed absent, so this is a bare v_max_f32 / v_max3_f32
// (inputs are finite or -inf here).
__device__ __forceinline__ float max2(float a, float b) { return __builtin_fmaxf(a, b); }

// Fold the logits of one 32-key sub-tile (keys on the accumulator's register axis; `key_lo` = key of
// this lane's register 0) into the running (reference, sum) of the lane's query row, per row block:  sum of the
// exponentials = z_run * 2^m_run.
// LAZY: the reference is the largest logit up to some sub-tile, and stays until a sub-tile's sum of 16 is above kRescale: no term
// is then more than 2^8 times the reference's, which the fp32 sum holds as exactly as the terms below it, and the maximum of the 16 and
// the rescaling, a fifth of the vector work, are left out (256K, W = 64, pass 1 147.7 -> 138.5 us; the layer step, on a slow box,
// 128K 132.9 -> 130.8, 64K 84.2 -> 81.1).  One branch for all row blocks, behind all of their arithmetic: with one per block half of it stood in
// a basic block without MFMAs (144.6).  Not for the shapes whose calls are start-up mostly: their one or two sub-tiles take the
// branch every time (d = 256, 8K, 17.2 -> 17.7); nor for up to 64 query rows, where the key stream bounds the pass and another loop
// is only more code (28 heads, W = 5, the scoring, 64K 36.9, without 36.1; 128K 60.5, 59.2); nor for 97 to 128 rows of d = 64 (two heads,
// 128 rows, 120K 31.2, 30.4; 242K 48.7, 47.1; but 96 rows 39.6, 40.7; why those gain and these lose has not been taken apart).  And a wavefront whose references move in more than an eighth of the sub-tiles goes on
// with the running maximum: logits of hundreds that grow (lognormal key lengths, 256K, W = 64) took
// 166 us without that, 149 with it, 147 with the running maximum throughout.
constexpr float kRescale = 256.f;
template <typename TE, int P, int NW, int RB, bool PAD>
constexpr bool kLazy = sizeof(TE) == 2 && P <= 16 && !PAD && NW > 2 && !(P <= 8 && NW == 4 && RB == 1);
template <int RB, bool MASK, bool LAZY>
__device__ __forceinline__ void rowstats_fold(const f32x16 (&acc)[RB], int key_lo, int N, int T,
                                              const int (&wi)[RB], float c1, float (&m_run)[RB], float (&z_run)[RB], int& raised) {
  float x[RB][16], sum[RB];
  bool far = false;
  auto raise = [&](int rb) {                              // the reference up to the sub-tile's largest logit, the sum with it
    float mx = x[rb][0];
#pragma unroll
    for (int r = 1; r < 16; r += 2) mx = max2(mx, max2(x[rb][r], x[rb][(r + 1) & 15]));
    const float m_new = max2(m_run[rb], mx * c1);
    sum[rb] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[rb] += fast_exp2(fmaf(x[rb][r], c1, -m_new));
    z_run[rb] *= fast_exp2(m_run[rb] - m_new);
    m_run[rb] = m_new;
  };
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[rb][r] = acc[rb][r];
    if (MASK) {
      // visible iff key < N and (key < T or key - T <= wi)  <=>  key < min(N, T + wi + 1)
      const int lim = min(N, T + wi[rb] + 1) - key_lo;
#pragma unroll
      for (int r = 0; r < 16; ++r) x[rb][r] = (8 * (r >> 2) + (r & 3) < lim) ? x[rb][r] : -INFINITY;
    }
    if (LAZY) {
      sum[rb] = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[rb] += fast_exp2(fmaf(x[rb][r], c1, -m_run[rb]));
      far |= sum[rb] > kRescale;
    } else {
      raise(rb);
    }
  }
  if (LAZY && __builtin_expect(__ballot(far) != 0ull, 0)) {   // uniform; so for the first visible keys, whose m_run is kNegBig
    ++raised;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) raise(rb);
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) z_run[rb] += sum[rb];
}

// One tile of pass 1: start the next tile's LDS-direct loads into `nxt`, then work on the tile in
// `cur`.  The two LDS buffers are distinct restrict pointers so that the compiler knows the fragment
// reads of `cur` need not wait for the loads into `nxt`.
// Software pipeline over the 32-key sub-tiles, across tile boundaries: the MFMAs of a sub-tile stand
// in one block of straight-line code with the softmax arithmetic of the sub-tile before it (`acc`, the
// last sub-tile of the tile before on entry), so that a wavefront's own vector instructions fill the
// time its MFMAs take.  MASK: tiles that touch the window block or the tail past N (they come last).
template <typename TE, int P, int NT, int RB, bool PAD, bool STREAM, bool MASK, bool LAZY>
__device__ __forceinline__ void rowstats_tile(const Piece* __restrict__ cur, Piece* __restrict__ nxt,
                                              bool prefetch, const TilePieces<P, NT>& tp, const char* __restrict__ kg, int64_t rsb,
                                              int prefetch_key0, int np, int last_piece, int tile, int prev, int N, int T, const int (&wi)[RB],
                                              int tid, int ln, int half, const Piece (&qf)[RB][P / 2], float c1,
                                              f32x16 (&acc)[RB], float (&m_run)[RB], float (&z_run)[RB], int& raised) {
  constexpr int KT = key_tile<P>();
  if (prefetch) issue_tile_loads<P, NT, STREAM>(tp, kg, rsb, prefetch_key0, N, last_piece, nxt, tid);
#pragma unroll
  for (int sub = 0; sub < KT / 32; ++sub) {
    f32x16 nxt_acc[RB];
    mma_subtile<TE, P, true, RB, PAD>(cur, sub, ln, half, np, qf, nxt_acc);
    // the sub-tile before this one: the last of tile `prev`, or of this tile
    rowstats_fold<RB, MASK, LAZY>(acc, (sub == 0 ? prev * KT + KT - 32 : tile * KT + (sub - 1) * 32) + 4 * half, N, T, wi, c1, m_run, z_run, raised);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[rb] = nxt_acc[rb];
  }
}

// ---------------------------------------------------------------------------------------------
// Pass 1: per-row running (max, sum) over this workgroup's key chunk, in the log2 domain, for query
// rows [m0, m1) of every KV head (m1 - m0 <= NW * 32 * RB).  ksh, kst: head and key strides in bytes.
// row_part[((g*n_chunks + chunk)*M + row)*2 + {0,1}] = (m, z) with  sum_j 2^(c1*l_j) = z * 2^m.
template <typename TE, int P, int NW, int RB, bool PAD, bool STREAM>
__global__ void __launch_bounds__(NW * 64)
score_rowstats_kernel(const char* __restrict__ q_obs, const char* __restrict__ k, int64_t ksh,
                      int64_t kst, int np, int Hk, int M, int m0, int m1, int W, int N, TileSplit<kInTurn<NW>> split,
                      float c1, float* __restrict__ row_part) {
  constexpr int NT = loader_threads<P, NW>();      // threads that load the K tiles
  constexpr int KS = P / 2, KT = key_tile<P>();
  constexpr int TILE_ELEMS = KT * P;
  constexpr int STAGES = kStages;
  __shared__ Piece lds_k[STAGES * TILE_ELEMS];

  const int g = blockIdx.x % Hk, chunk = blockIdx.x / Hk;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, ln = lane & 31, half = lane >> 5;
  const int T = N - W;
  const int row0 = m0 + wave * 32 * RB;         // first query row of this wave
  const int last_piece = PAD ? np - 1 : P - 1;
  int wi[RB];                                   // window row of this lane's query row, per block
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) wi[rb] = (row0 + rb * 32 + ln) % W;
  const char* kg = k + (int64_t)g * ksh;
  const int n_my = split.count(chunk);
  int ahead = split.tile(chunk, 0);             // next tile to load

  ASL_LOAD_Q_FRAGS();
  TilePieces<P, NT> tp;
  tp.init(kst, tid, last_piece);
  // prologue: STAGES-1 tiles in flight (after the Q loads, so the in-order wait counts line up)
#pragma unroll
  for (int j = 0; j < STAGES - 1; ++j) {
    if (j < n_my) issue_tile_loads<P, NT, STREAM>(tp, kg, kst, ahead * KT, N, last_piece, lds_k + j * TILE_ELEMS, tid);
    ahead += split.step(j);
  }

  ASL_WAIT_Q_FRAGS();

  float m_run[RB], z_run[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    m_run[rb] = kNegBig;
    z_run[rb] = 0.f;
  }
  f32x16 acc[RB];                                 // "no sub-tile before the first": adds nothing
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[rb][r] = -INFINITY;
  int stage = 0;                                  // buffer that holds tile `tile`
  int it = 0, tile = split.tile(chunk, 0), prev = tile;
  int raised = 0;                                 // sub-tiles that moved the references (uniform in the wavefront)
  auto step = [&](auto mask, auto lazy) {
    wait_tile<P, NT, STAGES>(min(STAGES - 2, n_my - 1 - it));
    __syncthreads();      // tile `tile` has landed for every wave; the buffer of the tile before is free again
    const int free_stage = (stage == 0) ? STAGES - 1 : stage - 1;
    rowstats_tile<TE, P, NT, RB, PAD, STREAM, decltype(mask)::value, decltype(lazy)::value>(
        lds_k + stage * TILE_ELEMS, lds_k + free_stage * TILE_ELEMS, it + STAGES - 1 < n_my, tp, kg, kst,
        ahead * KT, np, last_piece, tile, prev, N, T, wi, tid, ln, half, qf, c1, acc, m_run, z_run, raised);
    stage = (stage + 1 == STAGES) ? 0 : stage + 1;
    ahead += split.step(it + STAGES - 1);
    prev = tile;
    tile += split.step(it);
    ++it;
  };
  // Tiles of visible keys only, then those that touch the window block or the end.  `raised` is the wavefront's own, so the wavefronts of
  // a workgroup may be in different loops here and meet at barriers that are different statements: every turn of either loop passes
  // exactly one, in step(), and all wavefronts take n_my turns, and s_barrier counts the workgroup's arrivals wherever they come
  // from.  No turn may get another barrier, or none.  (One loop with a branch around the two foldings in it: 256K, W = 64, 289 us the
  // scoring, so 300; a vote of the wavefronts in LDS: 28 heads, W = 13, 128K 60.6, 61.4.)
  const int plain = T / KT;
  if constexpr (kLazy<TE, P, NW, RB, PAD>) {
    while (it < n_my && tile < plain && raised <= 3 + it / 4) step(std::false_type(), std::true_type());
  }
  while (it < n_my && tile < plain) step(std::false_type(), std::false_type());
  while (it < n_my) step(std::true_type(), std::false_type());
  if (n_my > 0)                                   // the last sub-tile is still to be folded
    rowstats_fold<RB, true, false>(acc, prev * KT + KT - 32 + 4 * half, N, T, wi, c1, m_run, z_run, raised);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    // the two lane halves hold disjoint keys of the same query row
    const float m_o = __shfl_xor(m_run[rb], 32), z_o = __shfl_xor(z_run[rb], 32);
    const float m = max2(m_run[rb], m_o);
    const float za = z_run[rb] * fast_exp2(m_run[rb] - m), zb = z_o * fast_exp2(m_o - m);
    const float z = (half == 0) ? (za + zb) : (zb + za);
    const int qrow = row0 + rb * 32 + ln;
    if (half == 0 && qrow < m1) {
      float* dst = row_part + ((int64_t)(g * split.n_chunks + chunk) * M + qrow) * 2;
      dst[0] = m;
      dst[1] = z;
    }
  }
}

// Fold the per-chunk partials (m_c, z_c) of one query row into the row's log2-domain softmax offset
// m + log2(Z).  Two lanes share a row (`half` = 0 or 1, partner = lane ^ 32): each takes every
// second chunk, in chunk order with a running maximum; the two halves are added in a fixed order,
// so all workgroups of a launch get the same bits for the same partials (score_combine_kernel adds in another order).
// p points at the row's partial of chunk 0; consecutive chunks are M float2 apart.
// Batches of kB chunks per lane: all loads of a batch are issued before the first is used.  The callers' counts fit one batch;
// written without the loop, the compiler contracts the sums in another way: other last bits, and at 10 K keys an error against
// 64 bits of 2.4e-7 instead of 1.9e-7.
// NR rows at once (pointers p[0..NR-1]): the loads of a batch go out for all of them before the first
// is used, so NR rows cost as many memory round trips as one.
// kFoldChunks: most partials that pass 2's workgroups fold themselves, two lanes a row in one round of loads.  Beyond, every
// workgroup reading all of them costs more than a launch in front of pass 2 that does so once (28 heads, 128K, 128 chunks:
// 92.7 us the scoring with the fold in two rounds, 88.8 with that launch; 7 heads on one, W = 64, 200K, 256 chunks: 78.3,
// 67.6; but 64 chunks, 8B shape: 32K 37.2, 37.9).
constexpr int kFoldChunks = 64;
// m + log2(z), z about 1 to 2^30, as if rounded once: the logarithm's own rounding is taken back by one exponential and the sum's
// is carried along.  An error here is one of all probabilities of a row (128K, offsets around 21: with m + log2f(z) the scores are
// 2.3 to 2.7e-7 off their values in 64 bits, so 0.9 to 1.6e-7).
__device__ __forceinline__ float row_offset(float m, float z) {
  const float l = __builtin_amdgcn_logf(z), s = m + l, b = s - m;
  const float lost = (m - (s - b)) + (l - b);
  return s + fmaf(fmaf(z, fast_exp2(-l), -1.0f), kLog2e, lost);
}
template <int NR, int kB>
__device__ __forceinline__ void combine_rows(const float2* const (&p)[NR], int M, int n_chunks, int half,
                                             float (&out)[NR]) {
  float m[NR], z[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    m[q] = kNegBig;
    z[q] = 0.f;
  }
  for (int c0 = half; c0 < n_chunks; c0 += 2 * kB) {
    float2 v[NR][kB];
#pragma unroll
    for (int q = 0; q < NR; ++q)
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        const int c = c0 + 2 * j;
        v[q][j] = p[q][(int64_t)min(c, n_chunks - 1) * M];
        if (c >= n_chunks) v[q][j] = make_float2(kNegBig, 0.f);
      }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      float mb = m[q];
#pragma unroll
      for (int j = 0; j < kB; ++j) mb = fmaxf(mb, v[q][j].x);
      float zb = 0.f;
#pragma unroll
      for (int j = 0; j < kB; ++j) zb += v[q][j].y * fast_exp2(v[q][j].x - mb);
      z[q] = z[q] * fast_exp2(m[q] - mb) + zb;
      m[q] = mb;
    }
  }
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const float mo = __shfl_xor(m[q], 32), zo = __shfl_xor(z[q], 32);
    const float mm = fmaxf(m[q], mo);
    const float za = z[q] * fast_exp2(m[q] - mm), zb2 = zo * fast_exp2(mo - mm);
    const float zs = (half == 0) ? (za + zb2) : (zb2 + za);
    out[q] = row_offset(mm, zs);
  }
}

// The offsets of all Hk*M rows, 16 rows a workgroup: row_const[r] = m + log2(Z) and, where the rows' log-sum-exp is asked
// for, as a natural logarithm, lse_out[r].  16 threads share a row, each every 16th chunk; their results are added in a
// fixed order.
constexpr int kCombineRows = 16;
__global__ void __launch_bounds__(256)
score_combine_kernel(const float* __restrict__ row_part, int Hk, int M, int n_chunks,
                     float* __restrict__ row_const, float* __restrict__ lse_out) {
  __shared__ float2 part[4][kCombineRows];
  const int tid = threadIdx.x, j = tid >> 4, wave = tid >> 6;
  const int r = blockIdx.x * kCombineRows + (tid & 15), rr = min(r, Hk * M - 1);
  const int g = rr / M, row = rr % M;
  const float2* p = reinterpret_cast<const float2*>(row_part) + (int64_t)g * n_chunks * M + row;
  constexpr int kB = kMaxChunks / 16;
  float2 v[kB];
#pragma unroll
  for (int i = 0; i < kB; ++i) {
    const int c = j + 16 * i;
    v[i] = make_float2(kNegBig, 0.f);
    if (16 * i < n_chunks) v[i] = p[(int64_t)min(c, n_chunks - 1) * M];
    if (c >= n_chunks) v[i] = make_float2(kNegBig, 0.f);
  }
  float m = kNegBig, z = 0.f;
#pragma unroll
  for (int i = 0; i < kB; ++i) m = fmaxf(m, v[i].x);
#pragma unroll
  for (int i = 0; i < kB; ++i) z += v[i].y * fast_exp2(v[i].x - m);
  auto add = [&](float mo, float zo, bool first) {
    const float mm = fmaxf(m, mo), za = z * fast_exp2(m - mm), zb = zo * fast_exp2(mo - mm);
    z = first ? za + zb : zb + za;
    m = mm;
  };
#pragma unroll
  for (int d = 16; d < 64; d <<= 1) add(__shfl_xor(m, d), __shfl_xor(z, d), (tid & d) == 0);
  if ((tid & 63) < 16) part[wave][tid & 15] = make_float2(m, z);
  __syncthreads();
  if (tid < 16) {
    m = part[0][tid].x;
    z = part[0][tid].y;
#pragma unroll
    for (int w = 1; w < 4; ++w) add(part[w][tid].x, part[w][tid].y, true);
    const float c = row_offset(m, z);
    if (r < Hk * M) {
      row_const[r] = c;
      if (lse_out != nullptr) lse_out[r] = c * kLn2;
    }
  }
}

// This lane's share of the column sums of one 32-key sub-tile (query rows on the accumulator's
// register axis): the normalised probabilities of its 16 rows per block, added in a fixed order.
// DENORM: probabilities below 2^-126 keep their (denormal) value instead of becoming zero.
template <int RB, bool DENORM>
__device__ __forceinline__ float colsum_fold(const f32x16 (&acc)[RB], const float (&rc)[RB][16], float c1) {
  float cs = 0.f;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = fmaf(acc[rb][r], c1, -rc[rb][r]);
      cs += DENORM ? exp2f(x) : fast_exp2(x);
    }
  return cs;
}

// This wave's column partials of one 32-key sub-tile, lane halves added (all lanes get the sum; the
// halves swap through the vector ALU, not through LDS).
template <int RB, bool DENORM>
__device__ __forceinline__ float colsum_subtile(const f32x16 (&acc)[RB], const float (&rc)[RB][16], float c1) {
  const uint32_t cs = __float_as_uint(colsum_fold<RB, DENORM>(acc, rc, c1));
  const auto sw = __builtin_amdgcn_permlane32_swap(cs, cs, false, false);    // {low half, high half} in every lane
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// One tile of pass 2: start the next tile's loads into `nxt`, then the MFMAs of the tile in `cur`
// beside the column partial sums of the sub-tile before each (`acc`; the last sub-tile of the tile
// before on entry): the same pipeline as pass 1's.  red_prev, red_cur: this wave's partial sums of the
// KT keys of the tile before and of this one.  ONLY: a workgroup's only tile; nothing is before it.
template <typename TE, int P, int NT, int RB, bool PAD, bool DENORM, bool STREAM, bool ONLY>
__device__ __forceinline__ void colsum_tile(const Piece* __restrict__ cur, Piece* __restrict__ nxt,
                                            bool prefetch, const TilePieces<P, NT>& tp, const char* __restrict__ kg, int64_t rsb,
                                            int prefetch_key0, int np, int last_piece, int N, int tid, int ln, int half,
                                            const Piece (&qf)[RB][P / 2], const float (&rc)[RB][16], float c1,
                                            f32x16 (&acc)[RB], float* __restrict__ red_prev, float* __restrict__ red_cur) {
  constexpr int KT = key_tile<P>();
  if (prefetch) issue_tile_loads<P, NT, STREAM>(tp, kg, rsb, prefetch_key0, N, last_piece, nxt, tid);
#pragma unroll
  for (int sub = 0; sub < KT / 32; ++sub) {
    f32x16 nxt_acc[RB];
    mma_subtile<TE, P, false, RB, PAD>(cur, sub, ln, half, np, qf, nxt_acc);
    if (!ONLY || sub > 0) {
      const float cs = colsum_subtile<RB, DENORM>(acc, rc, c1);
      float* red = (sub == 0) ? red_prev + KT - 32 : red_cur + (sub - 1) * 32;
      if (half == 0) red[ln] = cs;
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[rb] = nxt_acc[rb];
  }
}

// ---------------------------------------------------------------------------------------------
// Pass 2: u_group[g][j] = sum over query rows [m0, m1) of 2^(c1*l_rj - rc_r),  j < T,
// rc_r = rc_mul * row_const[g*M + r]  (log2-domain offset that already contains log2 Z_r).
// From the second row group on (m0 > 0) the sum is added to what the launch before left there.
template <typename TE, int P, int NW, int RB, bool PAD, bool DENORM, bool STREAM>
__global__ void __launch_bounds__(NW * 64)
score_colsum_kernel(const char* __restrict__ q_obs, const char* __restrict__ k, int64_t ksh,
                    int64_t kst, int np, int Hk, int M, int m0, int m1, int N, int T, TileSplit<kInTurn<NW>> split, float c1,
                    const float* __restrict__ row_const, float rc_mul, const float* __restrict__ row_part,
                    int n_parts, float* __restrict__ u_group) {
  constexpr int NT = loader_threads<P, NW>();      // threads that load the K tiles
  constexpr int NTHREADS = NW * 64;
  constexpr int KS = P / 2, KT = key_tile<P>();
  constexpr int TILE_ELEMS = KT * P;
  constexpr int STAGES = kStages;
  __shared__ Piece lds_k[STAGES * TILE_ELEMS];
  __shared__ float red[3][NW][KT];              // per-wave column partials of three tiles in turn

  const int g = blockIdx.x % Hk, chunk = blockIdx.x / Hk;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, ln = lane & 31, half = lane >> 5;
  const int row0 = m0 + wave * 32 * RB;         // first query row of this wave
  const int last_piece = PAD ? np - 1 : P - 1;
  const char* kg = k + (int64_t)g * ksh;

  ASL_LOAD_Q_FRAGS();
  TilePieces<P, NT> tp;
  tp.init(kst, tid, last_piece);
  // The tiles are taken from the last to the first: pass 1 took them first to last, so those read most recently are the ones this
  // pass reads first, and of keys that go through the last-level cache (not STREAM) finds there.
  const int n_my = split.count(chunk);
  int ahead = split.tile(chunk, n_my - 1), tile = ahead, prev = ahead, prev2 = ahead;   // next tile to load; this one, the two before
  // prologue: STAGES-1 tiles in flight before the row offsets are worked out, so that their latency
  // hides behind the first tiles' (later loads complete later: the counted waits below stay valid)
#pragma unroll
  for (int j = 0; j < STAGES - 1; ++j) {
    if (j < n_my) issue_tile_loads<P, NT, STREAM>(tp, kg, kst, ahead * KT, N, last_piece, lds_k + j * TILE_ELEMS, tid);
    ahead -= split.step(n_my - 2 - j);
  }

  // Log2-domain softmax offsets of this lane's accumulator rows: from the caller's log-sum-exp
  // (row_const, scaled by rc_mul), or folded here from pass 1's per-chunk partials (row_part).
  float rc[RB][16];
  float mine[RB];                                       // offsets of rows  row0 + 32*rb + ln
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) mine[rb] = 0.f;
  if (row_part != nullptr) {
    const float2* ps[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      ps[rb] = reinterpret_cast<const float2*>(row_part) + (int64_t)g * n_parts * M + min(row0 + rb * 32 + ln, m1 - 1);
    // the smallest batch that takes all partials: a batch is worked through whole, whatever it holds (always 48, pass 2
    // took 12.1 us at N = 512, 16.4 at 16K; so 8.7, 14.3)
    const auto& rows = reinterpret_cast<const float2* const (&)[RB]>(ps);
    if (n_parts <= 2 * 8)
      combine_rows<RB, 8>(rows, M, n_parts, half, mine);
    else if (n_parts <= 2 * 16)
      combine_rows<RB, 16>(rows, M, n_parts, half, mine);
    else
      combine_rows<RB, kFoldChunks / 2>(rows, M, n_parts, half, mine);
  }
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = row0 + rb * 32 + acc_row(r, half);
      float v;
      if (row_part != nullptr)
        v = __shfl(mine[rb], acc_row(r, half));         // lanes 0..31 hold rows 0..31 of the block
      else
        v = row_const[(int64_t)g * M + min(row, m1 - 1)] * rc_mul;
      rc[rb][r] = (row < m1) ? v : INFINITY;             // padded rows add 2^-inf = 0
    }
  }
  ASL_WAIT_Q_FRAGS();
  // sum the waves' partials of one finished tile in a fixed order and store the past columns
  auto reduce_store = [&](int buf_idx, int kbase) {
    for (int j = tid; j < KT; j += NTHREADS) {
      float s = red[buf_idx][0][j];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += red[buf_idx][w][j];
      if (kbase + j < T) {
        float* dst = u_group + (int64_t)g * T + kbase + j;
        *dst = (m0 > 0) ? *dst + s : s;
      }
    }
  };

  f32x16 acc[RB];                                 // "no sub-tile before the first"
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[rb][r] = -INFINITY;
  int stage = 0;                                  // buffer that holds the current tile
  int cur_red = 0, prev_red = 2;                  // red buffers of this tile and of the one before
  auto step = [&](int it, auto only) {
    wait_tile<P, NT, STAGES>(min(STAGES - 2, n_my - 1 - it));
    __syncthreads();      // the tile has landed; tile it-1's fragment reads and tile it-2's partials are done
    if (it > 1) reduce_store(3 - cur_red - prev_red, prev2 * KT);
    const int free_stage = (stage == 0) ? STAGES - 1 : stage - 1;
    colsum_tile<TE, P, NT, RB, PAD, DENORM, STREAM, decltype(only)::value>(
        lds_k + stage * TILE_ELEMS, lds_k + free_stage * TILE_ELEMS, it + STAGES - 1 < n_my, tp, kg, kst,
        ahead * KT, np, last_piece, N, tid, ln, half, qf, rc, c1, acc, &red[prev_red][wave][0], &red[cur_red][wave][0]);
    stage = (stage + 1 == STAGES) ? 0 : stage + 1;
    prev_red = cur_red;
    cur_red = (cur_red == 2) ? 0 : cur_red + 1;
    ahead -= split.step(n_my - 1 - STAGES - it);
    prev2 = prev;
    prev = tile;
    tile -= split.step(n_my - 2 - it);
  };
  // Calls of one tile per workgroup are start-up from end to end; without the turn of the pipeline that has nothing
  // before it they take 7.0 instead of 7.3 us (2 heads, d = 64, 4K, `lse` supplied).  The first of several tiles
  // stays in the loop: another copy of its code in front of it costs 0.5 us in instruction fetches.
  if (n_my == 1)
    step(0, std::true_type());
  else
    for (int it = 0; it < n_my; ++it) step(it, std::false_type());
  if (n_my > 0) {
    const float cs = colsum_subtile<RB, DENORM>(acc, rc, c1);
    if (half == 0) red[prev_red][wave][KT - 32 + ln] = cs;
    __syncthreads();
    if (n_my > 1) reduce_store(3 - cur_red - prev_red, prev2 * KT);
    reduce_store(prev_red, prev * KT);
  }
}

// ---------------------------------------------------------------------------------------------
// Generic path (any d, any M, fp32 or bf16 storage, plain fp32 FMA): rows that are no whole 16-byte pieces
// or longer than 256 elements, and the on-GPU cross-check of the MFMA path.
template <typename TIn> __device__ __forceinline__ float ldf(const TIn* p);
template <> __device__ __forceinline__ float ldf<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ldf<__bf16>(const __bf16* p) { return (float)*p; }

// one workgroup per global query row r = h*W + wi: log2-domain offset m + log2 Z (or from lse)
template <typename TIn>
__global__ void __launch_bounds__(256)
score_rowstats_generic(const TIn* __restrict__ q_obs, const TIn* __restrict__ k, int64_t ksh, int64_t kst,
                       int G, int W, int N, int D, float c1, float* __restrict__ row_const,
                       float* __restrict__ lse_out) {
  extern __shared__ float sm[];                // D floats of q, then 2*256 for the reduction
  float* qs = sm;
  float* red_m = sm + D;
  float* red_z = red_m + 256;
  const int r = blockIdx.x, h = r / W, wi = r % W, g = h / G;
  const int T = N - W;
  for (int c = threadIdx.x; c < D; c += 256) qs[c] = ldf<TIn>(q_obs + (int64_t)r * D + c);
  __syncthreads();
  const TIn* kg = k + (int64_t)g * ksh;
  const int n_vis = T + wi + 1;                // past keys + window keys 0..wi
  float m = kNegBig, z = 0.f;
  for (int j = threadIdx.x; j < n_vis; j += 256) {
    const TIn* kr = kg + (int64_t)j * kst;
    float dot = 0.f;
    for (int c = 0; c < D; ++c) dot = fmaf(qs[c], ldf<TIn>(kr + c), dot);
    float x = dot * c1;
    float mn = fmaxf(m, x);
    z = z * exp2f(m - mn) + exp2f(x - mn);
    m = mn;
  }
  red_m[threadIdx.x] = m;
  red_z[threadIdx.x] = z;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      float m1 = red_m[threadIdx.x], m2 = red_m[threadIdx.x + s];
      float mn = fmaxf(m1, m2);
      red_z[threadIdx.x] = red_z[threadIdx.x] * exp2f(m1 - mn) + red_z[threadIdx.x + s] * exp2f(m2 - mn);
      red_m[threadIdx.x] = mn;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float c = red_m[0] + log2f(red_z[0]);
    row_const[r] = c;
    if (lse_out != nullptr) lse_out[r] = c * kLn2;
  }
}

// one thread per (KV head g, past key j): loop over the M rows of the group
template <typename TIn>
__global__ void __launch_bounds__(256)
score_colsum_generic(const TIn* __restrict__ q_obs, const TIn* __restrict__ k, int64_t ksh, int64_t kst,
                     int M, int T, int D, float c1, const float* __restrict__ row_const, float rc_mul,
                     float* __restrict__ u_group) {
  const int g = blockIdx.y;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= T) return;
  const TIn* kr = k + (int64_t)g * ksh + (int64_t)j * kst;
  const TIn* qg = q_obs + (int64_t)g * M * D;
  float s = 0.f;
  for (int r = 0; r < M; ++r) {
    float dot = 0.f;
    for (int c = 0; c < D; ++c) dot = fmaf(ldf<TIn>(qg + (int64_t)r * D + c), ldf<TIn>(kr + c), dot);
    s += exp2f(fmaf(dot, c1, -row_const[(int64_t)g * M + r] * rc_mul));
  }
  u_group[(int64_t)g * T + j] = s;
}

// ---------------------------------------------------------------------------------------------
// Largest number of query rows per KV head (G*W) one launch of the MFMA kernels takes: eight
// wavefronts of two 32-row blocks.
constexpr int kMaxMfmaRows = 512;

bool score_mfma_supported(const asl_params& p) {
  const int M = (p.n_q_heads / p.n_kv_heads) * p.window;
  return p.dtype == ASL_BF16 && (p.head_dim == 64 || p.head_dim == 128) && M <= kMaxMfmaRows;
}

// Compute units of the current device (256 on MI355X).
static int device_cu_count() {
  static const int n = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
      v = 256;
    return v;
  }();
  return n;
}

// Key chunks per KV head of a launch, one workgroup each, of which a compute unit holds `resident` at once: at
// most one resident round of workgroups, so that no second, partly filled round trails behind.
//
// fold = false (the caller's log-sum-exp): only the key stream counts, and it lives on workgroups in flight: three per
// unit, four where a tile is 8 KB (8 heads, d = 64, 32 rows, 64K: 18.4 us with four, 22.3 with two), one fewer where
// that leaves each more than one tile but less than four.  From 65 rows of 16 pieces, or 97 of 8, a unit's pipes are
// as busy as its share of the stream: two, from five tiles each, else one (28 heads, 8K: 13.5 us with two, 12.6 with
// one; 8B shape, 128K layer step: 111.8 us with two, 115.0 with three); of 8 pieces from two tiles each (8 heads, 128
// rows, 16K: 12.4 us with two, 13.5 with one; 50K: 19.1 with two, 20.5 with three).
//
// fold = true: the rows' partials, one per chunk, are folded by every workgroup of pass 2 (up to kFoldChunks) or by a
// launch of their own.  The chunk count with the least estimated time is taken.  Estimated, in us, fitted to graph-replayed
// calls (1 to 8 KV heads, 16 to 448 rows, d = 64 and 128 in bf16 and some fp32, 4K to 200K keys, six chunk counts each; of 150 such
// calls in bf16 with nine counts each the choice is 2.5 % off the best on average, at worst 18 %: four heads of 128 rows from 128K
// on, where more chunks would do, and one head of 16 rows at 4K):
//  - the launch that combines partials: 4;
//  - a tile, both passes: 1.4, or 4.4 in fp32 (four MFMAs per fragment step);
//  - a unit takes `alone` workgroups before they slow each other down: its share of the stream feeds one with tiles
//    of 16 KB (1.15 of 64 rows a wavefront, 2.5 of one wavefront), and 5.2 wavefronts with tiles of 8 KB; in fp32 the four
//    matrix pipes are shared;
//  - 0.6, or 1.5 with 64 rows a wavefront, for every further workgroup of a unit (start-up).
// Examples, whole call, now and with all folding in pass 2 (fewer chunks): two heads, d = 64, 16 rows, 64K 19.5 and 25.9,
// 200K 34.0 and 41.3; one head, 128 rows, 20K 17.0 and 19.1, 200K 36.4 and 44.9; one head, 448 rows, 20K 28.7 and 35.6;
// 8B shape unchanged.
template <typename TE, int P, int NW, int RB>
static int score_chunks(int Hk, int n_tiles, int n_cu, int resident, bool fold) {
  auto fit = [&](int per_cu) {
    const int c = n_cu * (resident < per_cu ? resident : per_cu) / Hk, most = n_tiles < kMaxChunks ? n_tiles : kMaxChunks;
    return c < 1 ? 1 : (c < most ? c : most);
  };
  const bool f32 = sizeof(TE) == 4, narrow = P <= 8 && RB == 1 && !f32;
  if (!fold) {
    const bool busy = !f32 && (NW > 3 || RB > 1 || (NW == 3 && P > 8));
    if (!busy) {
      const int want = P <= 8 ? 4 : 3, per_cu = resident < want ? resident : want, c = fit(per_cu);
      return c < n_tiles && n_tiles < 4 * c ? fit(per_cu - 1) : c;
    }
    return n_tiles >= (P > 8 ? 5 : 2) * fit(2) ? fit(2) : fit(1);
  }
  const float alone = narrow ? 5.2f / NW : f32 ? (NW == 1 ? 3.5f : 1.0f) : NW == 1 ? 2.5f : NW == 2 && P > 16 ? 1.3f : RB > 1 ? 1.15f : 1.06f;
  const int most = fit(3), counts[] = {32, 64, RB > 1 ? 64 : 96, 128, RB > 1 ? 128 : 192, 256, most};
  int best = most;
  float best_us = INFINITY;
  for (const int c : counts) {
    if (c > most) continue;
    const float per_unit = (float)c * (float)Hk / (float)n_cu;
    const float tiles = n_tiles <= 2 * c ? (float)((n_tiles + c - 1) / c) : (float)n_tiles / (float)c;
    const float us = (c > kFoldChunks ? 4.0f : 0.0f) + tiles * (f32 ? 4.4f : 1.4f) * fmaxf(1.0f, per_unit / alone) +
                     (RB > 1 ? 1.5f : 0.6f) * fmaxf(0.0f, per_unit - 1.0f);
    if (us < best_us) {
      best_us = us;
      best = c;
    }
  }
  return best;
}

// Workgroups of `kernel` that fit on one compute unit at once (registers, LDS, wave slots).
template <typename K>
static int resident_per_cu(K kernel, int threads, size_t dynamic_lds = 0) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, dynamic_lds) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    n = 1;
  }
  return n;
}

// PAD: rows of fewer than P pieces.  DENORM: see colsum_fold.
template <typename TE, int P, int NW, int RB, bool PAD, bool DENORM>
static hipError_t launch_score_mfma(const asl_params& p, const Workspace& ws, const void* q_obs, const void* k_ptr,
                                    const float* lse, float* lse_out, float c1, hipStream_t st) {
  constexpr int KT = key_tile<P>(), kRows = NW * 32 * RB;
  const int Hk = p.n_kv_heads, M = (p.n_q_heads / Hk) * p.window, N = p.seq_len, T = N - p.window;
  const char *q = static_cast<const char*>(q_obs), *k = static_cast<const char*>(k_ptr);
  const int64_t ksh = p.k_stride_head * (int64_t)sizeof(TE), kst = p.k_stride_tok * (int64_t)sizeof(TE);
  const int np = p.head_dim * (int)sizeof(TE) / 16;
  // both passes use the same LDS ring and nearly the same registers; take the smaller residency
  static const int resident = [] {
    const int a = resident_per_cu(score_rowstats_kernel<TE, P, NW, RB, PAD, false>, NW * 64);
    const int b = resident_per_cu(score_colsum_kernel<TE, P, NW, RB, PAD, DENORM, false>, NW * 64);
    return a < b ? a : b;
  }();
  const int n_cu = device_cu_count();
  const int n_chunks = score_chunks<TE, P, NW, RB>(Hk, (N + KT - 1) / KT, n_cu, resident, lse == nullptr);
  const bool combine = n_chunks > kFoldChunks;
  // Kernels that load past the last-level cache (stream_keys), for keys read once (kOnce) or more often, are built where they gain:
  // not in fp32, bound by its arithmetic (both passes, us, without and with: 8 heads of d = 64, 96 MB 60.6, 63.3; of d = 128 59.3, 61.9;
  // `lse` supplied at most 1 % either way), nor, read more than once, with two row blocks a wavefront (28 heads, 256K 186.5, 185.9, alone
  // 158.4, 163.9; 1024 rows a head, `lse` supplied, 200 MB 294.6, 300.3) or padded rows (d = 80, 252 MB 158, 161).  A branch
  // in front of every tile's loads instead costs calls that do not stream up to 3 % (28 heads, W = 5, 67K 36.8, 38.0).
  constexpr bool kOnce = sizeof(TE) == 2, kTwice = kOnce && RB == 1 && !PAD;
  auto* rowstats = score_rowstats_kernel<TE, P, NW, RB, PAD, false>;
  auto* colsum = score_colsum_kernel<TE, P, NW, RB, PAD, DENORM, false>;
  if constexpr (kOnce) {
    const int reads = (M + kRows - 1) / kRows * (lse ? 1 : 2);
    if ((reads == 1 || kTwice) && stream_keys((int64_t)Hk * N * p.head_dim * (int64_t)sizeof(TE), reads, Hk > 1 && ksh == 0)) {
      colsum = score_colsum_kernel<TE, P, NW, RB, PAD, DENORM, true>;
      if constexpr (kTwice) rowstats = score_rowstats_kernel<TE, P, NW, RB, PAD, true>;
    }
  }
  if (!lse) {
    for (int m0 = 0; m0 < M; m0 += kRows)
      ASL_LAUNCH(ws.prof, kKernRowstats, st, rowstats, dim3(Hk * n_chunks), dim3(NW * 64), 0,
                 st, q, k, ksh, kst, np, Hk, M, m0, M < m0 + kRows ? M : m0 + kRows, p.window, N, split_tiles<kInTurn<NW>>(Hk, n_chunks, (N + KT - 1) / KT, n_cu, RB > 1), c1,
                 ws.row_part);
    if (lse_out || combine) {
      ASL_LAUNCH(ws.prof, kKernCombine, st, score_combine_kernel, dim3((Hk * M + kCombineRows - 1) / kCombineRows), dim3(256), 0, st,
                 ws.row_part, Hk, M, n_chunks, ws.row_const, lse_out);
      if (lse_out) return hipGetLastError();             // only the row normalisers were asked for
    }
  }
  const int n_tiles2 = (T + KT - 1) / KT;
  const int n_chunks2 = n_chunks < n_tiles2 ? n_chunks : n_tiles2;
  // without the caller's log-sum-exp or a launch that combined them every pass-2 workgroup folds pass 1's partials of
  // its own rows
  for (int m0 = 0; m0 < M; m0 += kRows)
    ASL_LAUNCH(ws.prof, kKernColsum, st, colsum, dim3(Hk * n_chunks2), dim3(NW * 64), 0, st,
               q, k, ksh, kst, np, Hk, M, m0, M < m0 + kRows ? M : m0 + kRows, N, T, split_tiles<kInTurn<NW>>(Hk, n_chunks2, n_tiles2, n_cu, RB > 1), c1, lse ? lse : ws.row_const,
               lse ? kLog2e : 1.0f, lse || combine ? nullptr : ws.row_part, n_chunks, ws.u_group);
  return hipGetLastError();
}

// Wavefronts and 32-row blocks per wavefront for M query rows per KV head (bf16, d = 8 P): one block per
// wavefront up to 128 rows; two above, with ceil(M / 64) wavefronts (up to eight: more than 512 rows
// take several launches of 512).
template <int P>
static hipError_t dispatch_nw(int M, const asl_params& p, const Workspace& ws, const void* q,
                              const void* k, const float* lse, float* lse_out, float c1, hipStream_t st) {
  if (M <= 128) {
    switch ((M + 31) / 32) {
      case 1: return launch_score_mfma<__bf16, P, 1, 1, false, false>(p, ws, q, k, lse, lse_out, c1, st);
      case 2: return launch_score_mfma<__bf16, P, 2, 1, false, false>(p, ws, q, k, lse, lse_out, c1, st);
      case 3: return launch_score_mfma<__bf16, P, 3, 1, false, false>(p, ws, q, k, lse, lse_out, c1, st);
      default: return launch_score_mfma<__bf16, P, 4, 1, false, false>(p, ws, q, k, lse, lse_out, c1, st);
    }
  }
  switch ((M + 63) / 64) {
    case 3: return launch_score_mfma<__bf16, P, 3, 2, false, false>(p, ws, q, k, lse, lse_out, c1, st);
    case 4: return launch_score_mfma<__bf16, P, 4, 2, false, false>(p, ws, q, k, lse, lse_out, c1, st);
    case 5: return launch_score_mfma<__bf16, P, 5, 2, false, false>(p, ws, q, k, lse, lse_out, c1, st);
    case 6: return launch_score_mfma<__bf16, P, 6, 2, false, false>(p, ws, q, k, lse, lse_out, c1, st);
    case 7: return launch_score_mfma<__bf16, P, 7, 2, false, false>(p, ws, q, k, lse, lse_out, c1, st);
    case 8: return launch_score_mfma<__bf16, P, 8, 2, false, false>(p, ws, q, k, lse, lse_out, c1, st);
    default: return launch_score_mfma<__bf16, P, 8, 2, false, true>(p, ws, q, k, lse, lse_out, c1, st);
  }
}

// The other row lengths and fp32.  Latency-bound at ordinary sizes; the plain kernels, which this replaced
// for whole-piece rows, walk M rows x d elements one after the other per key: fp32 Hq4/Hk2/d64, N = 512,
// W = 16: 247 + 6.5 us, here 4.5 + 4.5; bf16 Hq8/Hk4/d256, N = 8192, W = 32: the whole call 2274 us, here
// 17.1.  fp32 MFMA multiplies and adds in full fp32.
// np pieces of a row in the next longer of the built row lengths P; one
// 32-row block per wavefront, up to 128 query rows per launch.  Rows that fill P (the powers of two, mostly) have
// kernels of their own, without the test for pieces behind a row: d = 256, N = 8192, `lse` supplied, 12.6 -> 12.0 us.
template <typename TE, int P, bool PAD>
static hipError_t dispatch_padded_nw(int M, const asl_params& p, const Workspace& ws, const void* q,
                                     const void* k, const float* lse, float* lse_out, float c1, hipStream_t st) {
  if (M <= 32) return launch_score_mfma<TE, P, 1, 1, PAD, true>(p, ws, q, k, lse, lse_out, c1, st);
  if (M <= 64) return launch_score_mfma<TE, P, 2, 1, PAD, true>(p, ws, q, k, lse, lse_out, c1, st);
  return launch_score_mfma<TE, P, 4, 1, PAD, true>(p, ws, q, k, lse, lse_out, c1, st);
}
template <typename TE, int P>
static hipError_t dispatch_row_length(int np, int M, const asl_params& p, const Workspace& ws, const void* q,
                                      const void* k, const float* lse, float* lse_out, float c1, hipStream_t st) {
  if constexpr (sizeof(TE) == 4 || P > 16) {          // full bf16 rows of 8 and 16 pieces are dispatch_nw's
    if (np == P) return dispatch_padded_nw<TE, P, false>(M, p, ws, q, k, lse, lse_out, c1, st);
  }
  return dispatch_padded_nw<TE, P, true>(M, p, ws, q, k, lse, lse_out, c1, st);
}
template <typename TE>
static hipError_t dispatch_padded(int M, const asl_params& p, const Workspace& ws, const void* q,
                                  const void* k, const float* lse, float* lse_out, float c1, hipStream_t st) {
  const int np = p.head_dim * (int)sizeof(TE) / 16;
  if (np <= 8) return dispatch_row_length<TE, 8>(np, M, p, ws, q, k, lse, lse_out, c1, st);
  if (np <= 16) return dispatch_row_length<TE, 16>(np, M, p, ws, q, k, lse, lse_out, c1, st);
  if (np <= 24) return dispatch_row_length<TE, 24>(np, M, p, ws, q, k, lse, lse_out, c1, st);
  if constexpr (sizeof(TE) == 4) {
    if (np > 48) return dispatch_row_length<TE, 64>(np, M, p, ws, q, k, lse, lse_out, c1, st);
    if (np > 32) return dispatch_row_length<TE, 48>(np, M, p, ws, q, k, lse, lse_out, c1, st);
  }
  return dispatch_row_length<TE, 32>(np, M, p, ws, q, k, lse, lse_out, c1, st);
}

// Whether the MFMA kernels can read these operands: whole 16-byte pieces on 16-byte boundaries, rows
// of at most 256 elements, and a tile's rows within the loader's 32-bit byte offsets.
static bool mfma_takes(const asl_params& p, const void* q_obs, const void* k) {
  const int64_t eb = p.dtype == ASL_BF16 ? 2 : 4;
  const int64_t low = reinterpret_cast<intptr_t>(q_obs) | reinterpret_cast<intptr_t>(k) | (p.head_dim * eb) |
                      (p.k_stride_tok * eb) | (p.k_stride_head * eb);
  return (low & 15) == 0 && p.head_dim <= 256 && p.k_stride_tok * eb * 64 < (int64_t(1) << 32);
}

template <typename TIn>
static hipError_t launch_score_generic(const asl_params& p, const Workspace& ws, const TIn* q,
                                       const TIn* k, const float* lse, float* lse_out, float c1,
                                       hipStream_t st) {
  const int Hk = p.n_kv_heads, G = p.n_q_heads / Hk, W = p.window, M = G * W, N = p.seq_len, T = N - W;
  const int D = p.head_dim;
  if (!lse) {
    size_t sm = (size_t)(D + 512) * sizeof(float);
    ASL_LAUNCH(ws.prof, kKernScoreGeneric, st, (score_rowstats_generic<TIn>), dim3(p.n_q_heads * W), dim3(256), sm, st, q, k,
                       p.k_stride_head, p.k_stride_tok, G, W, N, D, c1, ws.row_const, lse_out);
  }
  if (lse_out) return hipGetLastError();
  ASL_LAUNCH(ws.prof, kKernScoreGeneric, st, (score_colsum_generic<TIn>), dim3((T + 255) / 256, Hk), dim3(256), 0, st, q, k,
                     p.k_stride_head, p.k_stride_tok, M, T, D, c1, lse ? lse : ws.row_const,
                     lse ? kLog2e : 1.0f, ws.u_group);
  return hipGetLastError();
}

// lse != null: the rows' log-sum-exp is given, only the column-sum pass runs.  lse_out != null (and
// lse == null): only the row-statistics pass runs and the rows' log-sum-exp is written there.
hipError_t launch_score(const asl_params& p, const Workspace& ws, const void* q_obs, const void* k,
                        const float* lse, float* lse_out, hipStream_t st) {
  const float scale = p.scale > 0.f ? p.scale : 1.0f / sqrtf((float)p.head_dim);
  const float c1 = scale * kLog2e;
  const int M = (p.n_q_heads / p.n_kv_heads) * p.window;
  if (!(p.flags & ASL_FLAG_GENERIC_SCORE)) {
    const bool takes = mfma_takes(p, q_obs, k);
    if (score_mfma_supported(p) || (takes && p.dtype == ASL_BF16 && (p.head_dim == 64 || p.head_dim == 128)))
      return p.head_dim == 128 ? dispatch_nw<16>(M, p, ws, q_obs, k, lse, lse_out, c1, st)
                               : dispatch_nw<8>(M, p, ws, q_obs, k, lse, lse_out, c1, st);
    if (takes)
      return p.dtype == ASL_BF16 ? dispatch_padded<__bf16>(M, p, ws, q_obs, k, lse, lse_out, c1, st)
                                 : dispatch_padded<float>(M, p, ws, q_obs, k, lse, lse_out, c1, st);
  }
  if (p.dtype == ASL_BF16)
    return launch_score_generic<__bf16>(p, ws, static_cast<const __bf16*>(q_obs),
                                        static_cast<const __bf16*>(k), lse, lse_out, c1, st);
  return launch_score_generic<float>(p, ws, static_cast<const float*>(q_obs),
                                     static_cast<const float*>(k), lse, lse_out, c1, st);
}

}  // namespace asl
