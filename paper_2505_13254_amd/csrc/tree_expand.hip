// hs_tree_expand: one level of Top-K growth of the draft trees, on the device (Section 2.2,
// Expansion; Section 4.3, Dynamic Extended Drafting: per-sequence depth limits).
//
// Nothing to stream: at most F * K new rows per sequence.  One workgroup per sequence appends the
// children of the frontier rows (their values are the single float32 add per node that the
// reranking step defines), ranks the new rows by counting under (value descending, row ascending)
// and lists the F best, in row order, as the next frontier.  The host never sees the tree: the
// calls of a step can be queued back to back, or captured in a graph.
//
// What bounds it is latency: two trips to memory (the frontier, then its rows' values) and the ranking.  Four threads
// share a row's comparisons, four values to an LDS read, and the frontier's order is found among the F chosen.
// (A thread to a row, one value a read and a loop over all rows' flags: 2.7 and 1 us of a launch of 5.7 for 100 new
// rows; a launch takes 3.5 now.)
#include <limits.h>

#include "tree_settle.h"

namespace hs {

constexpr int EXP_THREADS = 512;
constexpr int EXP_SHARE = 4;       // threads that share a row's comparisons (neighbours: their counts meet by DPP moves)
constexpr int EXP_MAX_NEW = 4096;  // F * K

struct ExpandArgs {
  int32_t* parent;
  int32_t* token;
  float* logc;
  float* cumlogp;
  int32_t* depth;
  float* ent;
  int32_t* n_nodes;
  int32_t* level;
  int32_t* frontier;
  int32_t* n_frontier;
  int32_t* frontier_rows;
  const int32_t* topk_idx;
  const float* topk_logp;
  const float* ent_topk;
  const int32_t* d_limit;
  int cap, F, K, first;
};

__global__ __launch_bounds__(EXP_THREADS) void k_tree_expand(ExpandArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned cv[EXP_MAX_NEW];  // values of the new rows, as ordered numbers
  __shared__ __attribute__((aligned(16))) int chosen[EXP_MAX_NEW];  // the F best of them, best first
  __shared__ int fr_old[EXP_MAX_NEW];     // the frontier being expanded
  const int s = blockIdx.x, tid = threadIdx.x;
  const int F = a.F, K = a.K;
  const int64_t base = (int64_t)s * a.cap;
  const float inv_K = 1.0f / (float)K;
  // e / K for e < EXP_MAX_NEW: (e + 0.5) / K is at least 1 / (2 K) away from an integer, far more than its rounding
  auto frontier_slot = [&](int e) { return (int)(((float)e + 0.5f) * inv_K); };
  int n, lvl, nf;
  if (a.first) {
    n = 1;
    lvl = 0;
    nf = 1;
    if (tid == 0) {
      a.parent[base] = -1;
      a.token[base] = -1;
      a.logc[base] = 0.f;
      a.cumlogp[base] = 0.f;
      a.depth[base] = 0;
      a.ent[base] = 0.f;
      fr_old[0] = 0;
    }
  } else {
    n = a.n_nodes[s];
    lvl = a.level[s];
    nf = a.n_frontier[s];
    nf = nf < 0 ? 0 : (nf > F ? F : nf);
    for (int j = tid; j < F; j += EXP_THREADS) fr_old[j] = a.frontier[(int64_t)s * F + j];  // (slots beyond nf: not read again)
  }
  const bool idle = nf == 0 || (a.d_limit != nullptr && lvl >= a.d_limit[s]);
  if (idle) {
    if (tid == 0) {
      a.n_frontier[s] = 0;
      if (a.first) {
        a.n_nodes[s] = 1;
        a.level[s] = 0;
      }
    }
    if (a.frontier_rows != nullptr)
      for (int j = tid; j < F; j += EXP_THREADS) a.frontier_rows[(int64_t)s * F + j] = (int32_t)base;
    return;
  }
  __syncthreads();  // fr_old is complete (and the root row written)

  // children of the frontier rows whose K children fit the capacity (a prefix of the frontier)
  int n_fit = (a.cap - n) / K;
  n_fit = n_fit > nf ? nf : n_fit;
  const int m = n_fit * K;
  for (int e = tid; e < m; e += EXP_THREADS) {
    const int j = frontier_slot(e);
    const int f = fr_old[j];
    // (of the results only the rows of frontier slots that exist are there to be read; they come with the parents' values)
    const int64_t src = (int64_t)s * F * K + e;
    const float lc = a.topk_logp[src];
    const int tok = a.topk_idx[src];
    // the root's value is 0 by definition (on a first call its row may not be visible yet)
    const float up = (a.first || f == 0) ? 0.f : a.cumlogp[base + f];
    const float v = up + fminf(lc, 0.f);
    const int dep = (a.first || f == 0) ? 0 : a.depth[base + f];
    const int64_t row = base + n + e;
    a.parent[row] = f;
    a.token[row] = tok;
    a.logc[row] = lc;
    a.cumlogp[row] = v;
    a.depth[row] = dep + 1;
    a.ent[row] = 0.f;
    cv[e] = order_bits(v);
  }
  for (int e = m + tid; e < ((m + 127) & ~127); e += EXP_THREADS) cv[e] = 0u;  // (above nothing)
  for (int j = tid; j < nf; j += EXP_THREADS) a.ent[base + fr_old[j]] = a.ent_topk[(int64_t)s * F + j];
  __syncthreads();

  // the F best new rows: rank by counting (the order is strict, so ranks are a permutation)
  const int nf_new = m < F ? m : F;
  if (m > F) {
    constexpr int PER = 128 / (EXP_SHARE * 4);  // LDS reads of a thread for 128 rows, requested together
    const int part = tid & (EXP_SHARE - 1);
    for (int e0 = 0; e0 < m; e0 += EXP_THREADS / EXP_SHARE) {  // (uniform: all lanes take part in the sum)
      const int e = e0 + tid / EXP_SHARE;
      const unsigned v = cv[e < m ? e : 0];
      int r = 0;
      for (int o0 = 0; o0 < m; o0 += 128) {
        uint4 c[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) c[q] = *reinterpret_cast<const uint4*>(&cv[o0 + (q * EXP_SHARE + part) * 4]);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
          const int o = o0 + (q * EXP_SHARE + part) * 4;
          // (better: a larger value, or as large and a lower row)
          r += c[q].x > v - (o < e ? 1u : 0u) ? 1 : 0;
          r += c[q].y > v - (o + 1 < e ? 1u : 0u) ? 1 : 0;
          r += c[q].z > v - (o + 2 < e ? 1u : 0u) ? 1 : 0;
          r += c[q].w > v - (o + 3 < e ? 1u : 0u) ? 1 : 0;
        }
      }
      r += __builtin_amdgcn_update_dpp(0, r, 0xb1, 0xf, 0xf, false);  // lanes 1, 0, 3, 2 of each four
      r += __builtin_amdgcn_update_dpp(0, r, 0x4e, 0xf, 0xf, false);  // lanes 2, 3, 0, 1
      if (part == 0 && e < m && r < F) chosen[r] = e;
    }
  } else {
    for (int e = tid; e < m; e += EXP_THREADS) chosen[e] = e;
  }
  __syncthreads();
  // in row order: a chosen row's place is the number of chosen rows before it
  for (int j = tid; j < nf_new; j += EXP_THREADS) {
    const int e = chosen[j];
    int pos = j;
    if (m > F) {
      pos = 0;
      for (int o = 0; o < nf_new; ++o) pos += chosen[o] < e ? 1 : 0;
    }
    a.frontier[(int64_t)s * F + pos] = n + e;
    if (a.frontier_rows != nullptr) {
      a.frontier_rows[(int64_t)s * F + pos] = (int32_t)(base + n + e);
      if (pos == nf_new - 1)  // the last valid slot also fills the unused ones
        for (int k = nf_new; k < F; ++k) a.frontier_rows[(int64_t)s * F + k] = (int32_t)(base + n + e);
    }
  }
  if (nf_new == 0 && a.frontier_rows != nullptr)
    for (int j = tid; j < F; j += EXP_THREADS) a.frontier_rows[(int64_t)s * F + j] = (int32_t)base;
  if (tid == 0) {
    a.n_nodes[s] = n + m;
    a.level[s] = lvl + 1;
    a.n_frontier[s] = nf_new;
  }
}

}  // namespace hs

using namespace hs;

extern "C" hs_status hs_tree_expand(int32_t* parent, int32_t* token, float* logc, float* cumlogp, int32_t* depth,
                                    float* ent, int32_t* n_nodes, int32_t* level, int32_t* frontier,
                                    int32_t* n_frontier, int32_t* frontier_rows, const int32_t* topk_idx,
                                    const float* topk_logp, const float* ent_topk, const int32_t* d_limit, int32_t B,
                                    int32_t cap, int32_t F, int32_t K, int32_t first, hs_stream stream) {
  clear_error();
  HS_REQUIRE(B >= 0, HS_ERR_SHAPE, "hs_tree_expand: B=%d", B);
  HS_REQUIRE(K >= 1 && K <= HS_MAX_TOPK, HS_ERR_SHAPE, "hs_tree_expand: K=%d must be in 1..%d", K, HS_MAX_TOPK);
  HS_REQUIRE(F >= 1 && (int64_t)F * K <= EXP_MAX_NEW, HS_ERR_SHAPE, "hs_tree_expand: F=%d, F * K must be in 1..%d", F,
             EXP_MAX_NEW);
  HS_REQUIRE(cap >= 1 + K, HS_ERR_SHAPE, "hs_tree_expand: cap=%d holds no level (K=%d)", cap, K);
  HS_REQUIRE((int64_t)B * cap < ((int64_t)1 << 31), HS_ERR_SHAPE, "hs_tree_expand: B * cap exceeds 2^31 rows");
  if (B == 0) return HS_OK;
  HS_REQUIRE(parent && token && logc && cumlogp && depth && ent && n_nodes && level && frontier && n_frontier &&
                 topk_idx && topk_logp && ent_topk,
             HS_ERR_NULL, "hs_tree_expand: NULL argument");
  ExpandArgs a{parent, token, logc, cumlogp, depth, ent, n_nodes, level, frontier, n_frontier, frontier_rows,
               topk_idx, topk_logp, ent_topk, d_limit, cap, F, K, first != 0 ? 1 : 0};
  hipLaunchKernelGGL(k_tree_expand, dim3((unsigned)B), dim3(EXP_THREADS), 0, static_cast<hipStream_t>(stream), a);
  return launch_status("tree expand");
}
