// Depths and cumulative values of a tree whose rows lie in LDS (internal; hs_tree_prune, hs_adaptive_control).
//
// A node's cumulative value is a chain of float32 adds, root first, and its path is known node first: a thread walks
// from its node to the root, keeping the confidences in registers, and then adds them up in the other order.  No thread
// waits for another one.  Trees deeper than WALK_DEPTH are settled level by level, a barrier to a level.  (511 rows
// of six levels: a launch of the pruning 7.2 us level by level, 6.3 by walks.)
#pragma once
#include "hs_common.h"

namespace hs {

// Float order on unsigned numbers.
__device__ __forceinline__ unsigned order_bits(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}

// Largest of the lanes' numbers, in every lane, by DPP moves.
__device__ __forceinline__ unsigned wave_max_u32(unsigned x) {
#define HS_DPP_STEP(ctrl, rows, banks) x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, banks, false))
  HS_DPP_STEP(0x111, 0xf, 0xf);  // row_shr:1
  HS_DPP_STEP(0x112, 0xf, 0xf);  // row_shr:2
  HS_DPP_STEP(0x114, 0xf, 0xe);  // row_shr:4
  HS_DPP_STEP(0x118, 0xf, 0xc);  // row_shr:8
  HS_DPP_STEP(0x142, 0xa, 0xf);  // row_bcast:15
  HS_DPP_STEP(0x143, 0xc, 0xf);  // row_bcast:31
#undef HS_DPP_STEP
  return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long x) {
  const unsigned hi = wave_max_u32((unsigned)(x >> 32));
  const unsigned lo = wave_max_u32((unsigned)(x >> 32) == hi ? (unsigned)x : 0u);
  return ((unsigned long long)hi << 32) | lo;
}

// A settled node in one word that other threads read whole (0: not settled yet): cumulative value, depth, a flag.
__device__ __forceinline__ unsigned long long node_word(float sum, int depth, bool ok) {
  return ((unsigned long long)((unsigned)(depth + 1) | (ok ? 0x80000000u : 0u)) << 32) | __builtin_bit_cast(unsigned, sum);
}
__device__ __forceinline__ float node_sum(unsigned long long w) { return __builtin_bit_cast(float, (unsigned)w); }
__device__ __forceinline__ int node_depth(unsigned long long w) { return (int)((unsigned)(w >> 32) & 0x7fffffffu) - 1; }
__device__ __forceinline__ bool node_ok(unsigned long long w) { return (w >> 63) != 0ull; }

constexpr int WALK_DEPTH = 16;
// Row i's word by a walk to the root (0 if that is more than WALK_DEPTH levels away).  ok(up, v, d): the flag of a node
// of value v and depth d whose parent's flag is `up`.  A row whose path does not end in row 0 gets no flag, a row without
// a parent depth and value 0.
template <typename Ok>
__device__ __forceinline__ unsigned long long walk_node(const int* par, const float* logc, int i, int n, Ok ok) {
  float c[WALK_DEPTH];
  int j = i, d = 0;
  bool up = true;  // row j may have a parent
#pragma unroll
  for (int t = 0; t < WALK_DEPTH; ++t) {
    const int p = par[j];
    c[t] = logc[j];
    up = up && p >= 0 && p < n;
    if (up) {
      d = t + 1;
      j = p;
    }
    if (__ballot(up) == 0ull) break;
  }
  if (up) {  // (a walk of the most levels may have ended in a root)
    const int p = par[j];
    if (p >= 0 && p < n) return 0ull;
  }
  float v = 0.f;
  bool flag = j == 0;
#pragma unroll
  for (int t = WALK_DEPTH - 1; t >= 0; --t)
    if (t < d) {
      v = v + fminf(c[t], 0.f);
      flag = ok(flag, v, d - t);
    }
  return node_word(v, d, flag);
}

// Settles rows 1 .. n-1 level by level; node[0] holds the root's word, the others 0, and unsettled[0 .. 2] are 0, before a
// barrier.  Of a malformed tree rows may stay unsettled.  Called by all
// THREADS threads; ends with a barrier.
template <int THREADS, int MAX_NODES, typename Ok>
__device__ __forceinline__ void settle_nodes(const int* par, const float* logc, unsigned long long* node, int* unsettled,
                                             int n, Ok ok) {
  static_assert(MAX_NODES <= 32 * THREADS, "a bit for each of a thread's nodes");
  const int tid = threadIdx.x, lane = tid & 63;
  unsigned left = 0u;  // this thread's nodes that are not settled: bit k for node tid + k * THREADS
#pragma unroll
  for (int k = 0; k < MAX_NODES / THREADS; ++k)
    if (tid + k * THREADS < n) left |= 1u << k;
  if (tid == 0) left &= ~1u;
  for (int round = 0; round < n; ++round) {  // (as many levels as there can be)
    for (unsigned todo = left; todo != 0u; todo &= todo - 1u) {
      const int k = __ffs((int)todo) - 1, i = tid + k * THREADS;
      const int p = par[i];
      unsigned long long w;
      if (p < 0 || p >= n) {
        w = node_word(0.f, 0, false);
      } else {
        // (a parent that was settled in this very round may be found or not: its word is final)
        const unsigned long long up = __hip_atomic_load(&node[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (up == 0ull) continue;
        const int d = node_depth(up) + 1;
        const float v = node_sum(up) + fminf(logc[i], 0.f);
        w = node_word(v, d, ok(node_ok(up), v, d));
      }
      __hip_atomic_store(&node[i], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      left &= ~(1u << k);
    }
    const int slot = round % 3;
    if (__ballot(left != 0u) != 0ull && lane == 0) unsettled[slot] = 1;
    __syncthreads();
    if (unsettled[slot] == 0) break;
    if (tid == 0) unsettled[(round + 2) % 3] = 0;  // (used again two rounds from here; read last a round ago)
  }
}

}  // namespace hs
