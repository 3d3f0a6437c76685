// Device code of the row-gather kernel (see gather.hip), written as a function so that another
// kernel can host it beside a second body.
#pragma once
#include "asl_internal.h"

namespace asl {

constexpr int kGatherThreads = 256;
constexpr int kGatherUnroll = 4;      // pieces per thread (the body is written out for four)

// Workgroup (bx, h, which, layer) of NT threads: bx = block of NT * kGatherUnroll pieces of the slab
// of KV head h, tensor `which` (0 = K, 1 = V), layer `layer`.  Pieces of a slab are numbered
// q = row * cpr + c (row = output row, c = 16-byte piece of the row).
// STREAM: rows and outputs pass the caches by (transfers that do not fit them anyway).
template <bool POW2, int NT, bool STREAM = false>
__device__ __forceinline__ void gather_body(const GatherArgs& a, int bx, int h, int which, int layer) {
  const char* src_base;
  char* dst_base;
  if (a.k_ptrs != nullptr) {                        // per-layer allocations
    src_base = static_cast<const char*>(which == 0 ? a.k_ptrs[layer] : a.v_ptrs[layer]);
    dst_base = static_cast<char*>(which == 0 ? a.k_out_ptrs[layer] : a.v_out_ptrs[layer]);
  } else {
    src_base = which == 0 ? a.k : a.v;
    dst_base = which == 0 ? a.k_out : a.v_out;
  }
  const int64_t sh = which == 0 ? a.ksh : a.vsh, stt = which == 0 ? a.kst : a.vst;
  src_base += (int64_t)h * sh;
  dst_base += (int64_t)h * a.n_idx * ((int64_t)a.cpr * 16);
  const int32_t* idx = a.idx + ((int64_t)layer * a.idx_rows + (a.idx_rows == 1 ? 0 : h)) * a.n_idx;
  const uint32_t total = (uint32_t)a.n_idx * (uint32_t)a.cpr;          // < 2^31, checked by the host
  const uint32_t q0 = (uint32_t)bx * (NT * kGatherUnroll) + threadIdx.x;
  // The tensors are device (global) memory: say so, so that plain global loads and stores are used.
  typedef const char __attribute__((address_space(1))) * GSrc;
  typedef char __attribute__((address_space(1))) * GDst;
  typedef uint32_t Piece __attribute__((ext_vector_type(4)));          // 16 bytes
  typedef const Piece __attribute__((address_space(1))) * GSrc16;
  typedef Piece __attribute__((address_space(1))) * GDst16;
  typedef const int32_t __attribute__((address_space(1))) * GIdx;
  const GSrc src = (GSrc)src_base;
  const GDst dst = (GDst)dst_base;
  const GIdx gi = (GIdx)idx;
  auto load = [](GSrc16 p) -> Piece { return STREAM ? __builtin_nontemporal_load(p) : *p; };
  auto store = [](Piece v, GDst16 p) {
    if (STREAM)
      __builtin_nontemporal_store(v, p);
    else
      *p = v;
  };
  // Loads are unconditional (piece numbers past the end are clamped to the last piece) so that all
  // four index loads, then all four row loads, are in flight together; only the stores are
  // predicated.  Written out rather than looped: the values must stay in registers.
  const uint32_t last = total - 1u;
  const uint32_t qa = q0, qb = q0 + NT, qc = q0 + 2 * NT, qd = q0 + 3 * NT;
  const uint32_t ca = min(qa, last), cb = min(qb, last), cc = min(qc, last), cd = min(qd, last);
  const uint32_t cpr = (uint32_t)a.cpr;
  const uint32_t ra = POW2 ? (ca >> a.cpr_shift) : (ca / cpr), rb = POW2 ? (cb >> a.cpr_shift) : (cb / cpr);
  const uint32_t rc = POW2 ? (cc >> a.cpr_shift) : (cc / cpr), rd = POW2 ? (cd >> a.cpr_shift) : (cd / cpr);
  const int ta = gi[ra], tb = gi[rb], tc = gi[rc], td = gi[rd];
  const Piece va = load((GSrc16)(src + (int64_t)ta * stt + (int64_t)(ca - ra * cpr) * 16));
  const Piece vb = load((GSrc16)(src + (int64_t)tb * stt + (int64_t)(cb - rb * cpr) * 16));
  const Piece vc = load((GSrc16)(src + (int64_t)tc * stt + (int64_t)(cc - rc * cpr) * 16));
  const Piece vd = load((GSrc16)(src + (int64_t)td * stt + (int64_t)(cd - rd * cpr) * 16));
  if (qa < total) store(va, (GDst16)(dst + (int64_t)qa * 16));
  if (qb < total) store(vb, (GDst16)(dst + (int64_t)qb * 16));
  if (qc < total) store(vc, (GDst16)(dst + (int64_t)qc * 16));
  if (qd < total) store(vd, (GDst16)(dst + (int64_t)qd * 16));
}

// Pieces per thread of a compaction beside its selection: fewer than above, since its latency follows the selection's (layer step, us,
// with four, two, one: two heads of d = 64, 10K 25.2, 24.4, 24.1; 8 heads, 4K 25.2, 25.5, 26.5; 12K 33.8, 33.4, 34.9).
constexpr int kPickedUnroll = 2;
// The same for rows that another workgroup of this launch is still selecting: the block's source tokens are read from the words
// (tag, token) in which it leaves them, T + i for the row's last, window tokens.  A word that carries the launch's tag is whole
// and this launch's, whatever it held before, so nothing else is ordered between the two.  k: the row's selected tokens; picks:
// the row's words.  Returns false, the wavefront's part not written, if its words have not come after kFlagSpinLimit polls.
template <bool POW2, int NT>
__device__ __forceinline__ bool gather_picked_body(const GatherArgs& a, int bx, int h, int which, int T, int k,
                                                   const unsigned long long* picks, uint32_t tag) {
  typedef uint32_t Piece __attribute__((ext_vector_type(4)));          // 16 bytes
  typedef const Piece __attribute__((address_space(1))) * GSrc16;
  typedef Piece __attribute__((address_space(1))) * GDst16;
  const char* src = (which == 0 ? a.k : a.v) + (int64_t)h * (which == 0 ? a.ksh : a.vsh);
  char* dst = (which == 0 ? a.k_out : a.v_out) + (int64_t)h * a.n_idx * ((int64_t)a.cpr * 16);
  const int64_t stt = which == 0 ? a.kst : a.vst;
  const uint32_t total = (uint32_t)a.n_idx * (uint32_t)a.cpr, last = total - 1u, cpr = (uint32_t)a.cpr;
  uint32_t q[kPickedUnroll], c[kPickedUnroll], r[kPickedUnroll], tok[kPickedUnroll];
#pragma unroll
  for (int u = 0; u < kPickedUnroll; ++u) {
    q[u] = (uint32_t)bx * (NT * kPickedUnroll) + threadIdx.x + u * NT;
    const uint32_t cq = min(q[u], last);
    r[u] = POW2 ? (cq >> a.cpr_shift) : (cq / cpr);
    c[u] = cq - r[u] * cpr;
  }
  if (threadIdx.x < 64) {                               // one wavefront looks for the row's last word first: fewer polls
    for (int spins = 0; spins < kFlagSpinLimit; ++spins) {
      const unsigned long long w = __hip_atomic_load(picks + k - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((uint32_t)__builtin_amdgcn_readfirstlane((int)(w >> 32)) == tag) break;
      __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
  for (int spins = 0;; ++spins) {
    bool ok = true;
#pragma unroll
    for (int u = 0; u < kPickedUnroll; ++u) {
      const unsigned long long w = __hip_atomic_load(picks + min(r[u], (uint32_t)k - 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ok = ok && (uint32_t)(w >> 32) == tag;
      tok[u] = r[u] < (uint32_t)k ? (uint32_t)w : (uint32_t)T + (r[u] - (uint32_t)k);
    }
    if (__ballot(!ok) == 0ull) break;                   // uniform
    if (spins >= kFlagSpinLimit) return false;
    __builtin_amdgcn_s_sleep(2);
  }
  Piece v[kPickedUnroll];
#pragma unroll
  for (int u = 0; u < kPickedUnroll; ++u) v[u] = *(GSrc16)(src + (int64_t)tok[u] * stt + (int64_t)c[u] * 16);
#pragma unroll
  for (int u = 0; u < kPickedUnroll; ++u)
    if (q[u] < total) *(GDst16)(dst + (int64_t)q[u] * 16) = v[u];
  return true;
}

}  // namespace asl
