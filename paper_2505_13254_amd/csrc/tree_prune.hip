// hs_tree_prune: reranking of the draft tree by cumulative confidence (Section 2.2) under a depth
// cap, a threshold on the cumulative log-probability and a per-sequence node budget (Section 4.3).
//
// Nothing to stream: a few hundred nodes per sequence.  One workgroup per sequence keeps the tree in
// LDS (global scratch for very large trees), fills depth and the cumulative sums from parent to child so
// that every sum is the single float32 add the definition states, finds the last candidate that the budget
// keeps digit by digit, and scans the keep flags; a second launch turns per-sequence counts into packed
// offsets and emits the renumbered tree.
//
// What bounds it is the chain of barriers, LDS round trips and two trips to memory, at a few hundred
// cycles each, so the LDS form takes as few of them as it can: a node to a thread up to 512 nodes; depth and
// sum from one walk to the root, where depths by a walk and sums by a barrier to a level took three times as long; digits of
// eight bits over the range of the values that are there (two rounds for the usual tree; six bits from the sign downwards took
// four or five); positions from ballots.  One tree of 511 nodes: a launch took 10.0 us and takes 6.3; 16 of 311 to 911 nodes 18.9 and 8.8.
#include <limits.h>

#include "tree_settle.h"

namespace hs {

constexpr int PR_SMALL = 512, PR_BIG = 1024;  // threads of a workgroup: a node to a thread where the trees are not larger
constexpr int PR_LDS_NODES = 4096;  // trees up to this size live in LDS
static_assert(PR_LDS_NODES / 64 <= 64, "the runs of 64 nodes are counted by one wave");

// (value, index) as one 45-bit key, index < 8192: larger key = better (larger value, then lower
// index).  Values count from the lowest one that is there, so that the key's upper digits differ.
constexpr int KEY_INDEX_BITS = 13;
constexpr int DIGIT_BITS = 8;
constexpr int N_BINS = 1 << DIGIT_BITS;
constexpr int N_ROUNDS = (32 + KEY_INDEX_BITS + DIGIT_BITS - 1) / DIGIT_BITS;
static_assert(PR_LDS_NODES <= 1 << KEY_INDEX_BITS, "the index fits its bits");
__device__ __forceinline__ unsigned long long order_key(unsigned above_lowest, int i) {
  return ((unsigned long long)above_lowest << KEY_INDEX_BITS) | (unsigned)((1 << KEY_INDEX_BITS) - 1 - i);
}

struct PruneArgs {
  const int32_t *parent, *node_offsets, *node_counts, *d_max, *max_nodes;
  const float *logc, *theta;
  int32_t* depth;
  float* cumlogp;
  uint8_t* keep;
  int32_t *ws_pos, *ws_parent, *ws_count;  // of a node: its new row (-1: dropped) and its parent's; of a sequence: its rows
  int32_t *out_offsets, *out_src, *out_parent;
  int B, NN;
};

// Trees beyond PR_LDS_NODES nodes: the output arrays and the workspace are the scratch (ws_pos is not written
// before the last phase, so it can hold the budget flags meanwhile; ws_parent holds the path filter's).
template <int PR_THREADS>
__device__ __forceinline__ void prune_large(const PruneArgs& a, int s, int o, int n) {
  constexpr int PR_WAVES = PR_THREADS / 64;
  __shared__ int red[PR_WAVES];
  __shared__ int chunk_sum[PR_THREADS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int32_t* par = a.parent + o;
  const float* lc = a.logc + o;
  int32_t *dep = a.depth + o, *ok = a.ws_parent + o, *nxt = a.ws_pos + o;
  float* sum = a.cumlogp + o;
  const int dcap = a.d_max[s], budget = a.max_nodes[s];
  const float th = a.theta[s];
  auto block_sum = [&](int v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) red[tid >> 6] = v;
    __syncthreads();
    int r = 0;
    for (int w = 0; w < PR_WAVES; ++w) r += red[w];
    __syncthreads();
    return r;
  };
  // depth: walk to the root
  for (int i = tid; i < n; i += PR_THREADS) {
    int d = 0;
    for (int j = par[i]; j >= 0; j = par[j]) ++d;
    dep[i] = d;
  }
  if (tid == 0) {
    sum[0] = 0.f;
    ok[0] = 1;
  }
  __syncthreads();
  // cumulative log-confidence and the path filter, one level at a time (parents are final first)
  for (int level = 1, left = n - 1; left > 0 && level < n; ++level) {
    int here = 0;
    for (int i = tid; i < n; i += PR_THREADS) {
      if (dep[i] == level) {
        const int p = par[i];
        const float v = sum[p] + fminf(lc[i], 0.f);
        sum[i] = v;
        ok[i] = (ok[p] != 0 && level <= dcap && v >= th) ? 1 : 0;
        ++here;
      }
    }
    here = block_sum(here);
    if (here == 0) break;
    left -= here;
  }
  // node budget: keep the first max_nodes candidates under (sum descending, index ascending)
  int mine = 0;
  for (int i = tid; i < n; i += PR_THREADS) mine += (i >= 1 && ok[i]) ? 1 : 0;
  const int n_cand = block_sum(mine);
  if (budget > 0 && n_cand > budget) {
    for (int i = tid; i < n; i += PR_THREADS) {
      int flag = ok[i];
      if (i >= 1 && flag) {
        const float v = sum[i];
        int r = 0;
        for (int j = 1; j < n; ++j) r += (ok[j] && better(sum[j], j, v, i)) ? 1 : 0;
        flag = r < budget ? 1 : 0;
      }
      nxt[i] = flag;
    }
    __syncthreads();
    for (int i = tid; i < n; i += PR_THREADS) ok[i] = nxt[i];
    __syncthreads();
  }
  // positions of the kept nodes: each thread owns a contiguous chunk, then a scan of chunk totals
  const int per = (n + PR_THREADS - 1) / PR_THREADS;
  const int lo = min(tid * per, n), hi = min(lo + per, n);
  int c = 0;
  for (int i = lo; i < hi; ++i) c += ok[i] ? 1 : 0;
  chunk_sum[tid] = c;
  __syncthreads();
  if (tid < 64) {
    int loc[PR_WAVES], tot = 0;  // (a lane to PR_WAVES chunks)
#pragma unroll
    for (int q = 0; q < PR_WAVES; ++q) {
      loc[q] = tot;
      tot += chunk_sum[tid * PR_WAVES + q];
    }
    const int incl = wave_prefix_sum(tot);
#pragma unroll
    for (int q = 0; q < PR_WAVES; ++q) chunk_sum[tid * PR_WAVES + q] = incl - tot + loc[q];
    if (tid == 63) a.ws_count[s] = incl;
  }
  __syncthreads();
  int pos = chunk_sum[tid];
  for (int i = lo; i < hi; ++i) {
    const int k = ok[i] ? 1 : 0;
    nxt[i] = k ? pos : -1;
    a.keep[o + i] = (uint8_t)k;
    pos += k;
  }
  __syncthreads();
  for (int i = tid; i < n; i += PR_THREADS) ok[i] = par[i] < 0 ? -1 : nxt[par[i]];  // (what k_prune_emit reads as ws_parent)
}

template <int PR_THREADS>
__global__ __launch_bounds__(PR_THREADS) void k_prune_select(PruneArgs a) {
  __shared__ int l_par[PR_LDS_NODES];
  __shared__ unsigned long long l_node[PR_LDS_NODES];
  __shared__ float l_logc[PR_LDS_NODES];
  __shared__ int l_new[PR_LDS_NODES];
  __shared__ __attribute__((aligned(16))) int hist[N_ROUNDS][N_BINS];
  __shared__ int unsettled[3];
  __shared__ int n_cand_s;
  __shared__ unsigned lowest_s, highest_s;
  __shared__ int run_count[PR_LDS_NODES / 64];  // kept nodes of each run of 64

  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // a single sequence: its packed offset is 0, so the renumbered tree is written right here
  const bool emit = gridDim.x == 1 && a.NN <= PR_LDS_NODES;
  // Everything that does not depend on the offsets is requested with them.  A single sequence begins at row 0 as a
  // rule: its nodes are requested too, before its offset is known to be 0.
  const int o = a.node_offsets[s];
  const int o_next = a.node_counts != nullptr ? 0 : a.node_offsets[s + 1];
  const int counted = a.node_counts != nullptr ? a.node_counts[s] : 0;
  const int dcap = a.d_max[s], budget = a.max_nodes[s];
  const float th = a.theta[s];
  int first_par = 0;
  float first_logc = 0.f;
  if (emit && tid < a.NN) {
    first_par = a.parent[tid];
    first_logc = a.logc[tid];
  }
  for (int b = tid; b < N_ROUNDS * N_BINS; b += PR_THREADS) (&hist[0][0])[b] = 0;
  if (tid < 3) unsettled[tid] = 0;
  if (tid < PR_LDS_NODES / 64) run_count[tid] = 0;
  if (tid == 0) {
    n_cand_s = 0;
    lowest_s = ~0u;
    highest_s = 0u;
  }
  const int n = a.node_counts != nullptr ? counted : o_next - o;
  if (n <= 0) {
    if (tid == 0) {
      a.ws_count[s] = 0;
      if (emit) a.out_offsets[0] = a.out_offsets[1] = 0;  // (else k_prune_emit writes them)
    }
    if (emit)
      for (int i = tid; i < a.NN; i += PR_THREADS) {
        a.out_src[i] = 0;
        a.out_parent[i] = 0;
      }
    return;
  }
  if (n > PR_LDS_NODES) {
    prune_large<PR_THREADS>(a, s, o, n);
    return;
  }
  for (int i = tid; i < n; i += PR_THREADS) {
    const bool have = emit && o == 0 && i < PR_THREADS && i < a.NN;
    l_par[i] = have ? first_par : a.parent[o + i];
    l_logc[i] = have ? first_logc : a.logc[o + i];
  }
  __syncthreads();

  // ---- depth, cumulative log-confidence and the path filter
  auto filter = [&](bool up, float v, int d) { return up && d <= dcap && v >= th; };
  bool deep = false;
  for (int i = tid; i < n; i += PR_THREADS) {
    const unsigned long long w = walk_node(l_par, l_logc, i, n, filter);
    l_node[i] = w;  // (only this thread reads it, unless the tree is deep)
    deep = deep || w == 0ull;
  }
  if (__syncthreads_or(deep ? 1 : 0)) {
    for (int i = tid; i < n; i += PR_THREADS) l_node[i] = i == 0 ? node_word(0.f, 0, true) : 0ull;
    __syncthreads();
    settle_nodes<PR_THREADS, PR_LDS_NODES>(l_par, l_logc, l_node, unsettled, n, filter);
  }

  // ---- candidates: how many, and the range of their values
  if (budget > 0) {
    int mine = 0;
    float lo = HS_INF, hi = -HS_INF;
    for (int i = tid; i < n; i += PR_THREADS) {
      const unsigned long long w = l_node[i];
      if (i >= 1 && node_ok(w)) {
        ++mine;
        lo = fminf(lo, node_sum(w));
        hi = fmaxf(hi, node_sum(w));
      }
    }
    if (__ballot(mine != 0) != 0ull) {
      const int cnt = __builtin_amdgcn_readlane(wave_prefix_sum(mine), 63);
      const float lowest = -wave_max(-lo), highest = wave_max(hi);
      if (lane == 0) {
        atomicAdd(&n_cand_s, cnt);
        atomicMin(&lowest_s, order_bits(lowest));
        atomicMax(&highest_s, order_bits(highest));
      }
    }
  }
  __syncthreads();

  // ---- node budget: keep the first max_nodes candidates under (sum descending, index ascending).  The budget-th best
  // key, digit by digit from the top.  Per digit: a histogram of the keys that match the digits fixed so far (LDS
  // atomics, one histogram per round so that no round waits for a reset), one barrier, then every wave finds,
  // with a prefix sum over the bins from the top, the largest digit d such that at least `need` matching keys have a
  // digit >= d; the keys above d are all in, the search goes on among those with digit d.  Keys are distinct,
  // so exactly `budget` candidates end up >= x.
  unsigned long long x = 0ull;  // digits fixed so far, in place (0: every candidate is kept)
  const unsigned lowest = lowest_s;
  if (budget > 0 && n_cand_s > budget) {
    int need = budget;
    int top = KEY_INDEX_BITS + (32 - __clz((int)((highest_s - lowest) | 1u)));  // bits that are not fixed yet
    for (int r = 0; r < N_ROUNDS; ++r) {
      const int shift = top > DIGIT_BITS ? top - DIGIT_BITS : 0;
      const unsigned mask = (1u << (top - shift)) - 1u;
      for (int i = tid; i < n; i += PR_THREADS) {
        const unsigned long long w = l_node[i];
        if (i >= 1 && node_ok(w)) {
          const unsigned long long k = order_key(order_bits(node_sum(w)) - lowest, i);
          if ((k >> top) == (x >> top)) atomicAdd(&hist[r][(unsigned)(k >> shift) & mask], 1);
        }
      }
      __syncthreads();
      const int4 c = reinterpret_cast<const int4*>(hist[r])[63 - lane];  // lane l looks at bins 252 - 4 l .. 255 - 4 l
      const int sum = c.x + c.y + c.z + c.w;
      const int incl = wave_prefix_sum(sum);  // matching keys in these bins and those above
      const int l_hit = __ffsll((long long)__ballot(incl >= need)) - 1;  // never empty: need <= matching keys
      int above = __builtin_amdgcn_readlane(incl - sum, l_hit);
      const int c3 = __builtin_amdgcn_readlane(c.w, l_hit), c2 = __builtin_amdgcn_readlane(c.z, l_hit);
      const int c1 = __builtin_amdgcn_readlane(c.y, l_hit), c0 = __builtin_amdgcn_readlane(c.x, l_hit);
      int digit = 255 - 4 * l_hit, here = c3;
      if (above + here < need) { above += here; here = c2; --digit; }
      if (above + here < need) { above += here; here = c1; --digit; }
      if (above + here < need) { above += here; here = c0; --digit; }
      need -= above;
      x |= (unsigned long long)(unsigned)digit << shift;
      // all of them are wanted: the digits fixed so far, followed by zeros, already separate the kept
      // keys from the others (the same values in every thread: the workgroup leaves the loop together)
      if (here == need || shift == 0) break;
      top = shift;
    }
  }

  // ---- positions of the kept nodes: a ballot to a run of 64, a prefix sum over the runs
  auto kept = [&](int i, unsigned long long w) {
    return i == 0 || (node_ok(w) && (x == 0ull || order_key(order_bits(node_sum(w)) - lowest, i) >= x));
  };
  for (int i0 = wave * 64; i0 < n; i0 += PR_THREADS) {
    const int i = i0 + lane;
    const unsigned long long who = __ballot(i < n && kept(i, l_node[i < n ? i : 0]));
    if (lane == 0) run_count[i0 >> 6] = __popcll(who);
    if (i < n) l_new[i] = (who >> lane) & 1ull ? __popcll(who & ((1ull << lane) - 1ull)) : -1;  // (inside its run)
  }
  __syncthreads();
  const int run = run_count[lane];
  const int run_incl = wave_prefix_sum(run);
  const int total = __builtin_amdgcn_readlane(run_incl, 63);
  // (a node's new row; its run's first row comes from the lane that holds the run)
  auto new_row = [&](int i) {
    const int in_run = l_new[i];
    const int first = __shfl(run_incl - run, i >> 6);
    return in_run < 0 ? -1 : first + in_run;
  };
  if (tid == 0) {
    a.ws_count[s] = total;
    if (emit) {
      a.out_offsets[0] = 0;
      a.out_offsets[1] = total;
    }
  }
  for (int i0 = wave * 64; i0 < n; i0 += PR_THREADS) {
    const int i = i0 + lane < n ? i0 + lane : n - 1;  // (all lanes take part in new_row's exchange)
    const unsigned long long w = l_node[i];
    const int p = l_par[i];
    const int row = new_row(i);
    const int up = new_row(p >= 0 && p < n ? p : 0);
    if (i0 + lane >= n) continue;
    a.keep[o + i] = row >= 0 ? 1 : 0;
    a.depth[o + i] = node_depth(w);
    a.cumlogp[o + i] = node_sum(w);
    if (emit) {
      if (row >= 0) {
        a.out_src[row] = i;
        a.out_parent[row] = i == 0 ? -1 : up;
      }
    } else {
      a.ws_pos[o + i] = row;
      a.ws_parent[o + i] = i == 0 ? -1 : up;
    }
  }
  if (emit)  // the unused tail of the output arrays: rows that hang off the root and repeat it
    for (int i = total + tid; i < a.NN; i += PR_THREADS) {
      a.out_src[i] = 0;
      a.out_parent[i] = 0;
    }
}

constexpr int PE_THREADS = 256;
__global__ __launch_bounds__(PE_THREADS) void k_prune_emit(PruneArgs a) {
  __shared__ int red[PE_THREADS / 64];
  const int s = blockIdx.x, tid = threadIdx.x;
  // (the counts, the offsets and the first nodes' rows are not waited for one after the other)
  const int o = a.node_offsets[s];
  const int n = a.node_counts != nullptr ? a.node_counts[s] : a.node_offsets[s + 1] - o;
  const int here = a.ws_count[s];
  int mine = 0;
  for (int t = tid; t < s; t += PE_THREADS) mine += a.ws_count[t];
  constexpr int AT = 4;
  int row[AT], up[AT];
#pragma unroll
  for (int k = 0; k < AT; ++k) {
    const int i = tid + k * PE_THREADS;
    row[k] = i < n ? a.ws_pos[o + i] : -1;
    up[k] = i < n ? a.ws_parent[o + i] : 0;
  }
  mine = __builtin_amdgcn_readlane(wave_prefix_sum(mine), 63);
  if ((tid & 63) == 0) red[tid >> 6] = mine;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int w = 0; w < PE_THREADS / 64; ++w) base += red[w];
  if (tid == 0) {
    a.out_offsets[s] = base;
    if (s == a.B - 1) a.out_offsets[a.B] = base + here;
  }
#pragma unroll
  for (int k = 0; k < AT; ++k)
    if (row[k] >= 0) {
      a.out_src[base + row[k]] = tid + k * PE_THREADS;
      a.out_parent[base + row[k]] = up[k];
    }
  for (int i = tid + AT * PE_THREADS; i < n; i += PE_THREADS) {
    const int p = a.ws_pos[o + i];
    if (p >= 0) {
      a.out_src[base + p] = i;
      a.out_parent[base + p] = a.ws_parent[o + i];
    }
  }
  // the unused tail of the output arrays (last workgroup): rows that hang off a root and repeat it
  if (s == a.B - 1)
    for (int i = base + here + tid; i < a.NN; i += PE_THREADS) {
      a.out_src[i] = 0;
      a.out_parent[i] = 0;
    }
}

}  // namespace hs

extern "C" size_t hs_tree_prune_workspace(int32_t B, int32_t NN) {
  if (B <= 0 || NN < 0) return 0;
  return 2 * hs::align_up((size_t)(NN > 0 ? NN : 1) * sizeof(int32_t), 256) +
         hs::align_up((size_t)B * sizeof(int32_t), 256);
}

// Validation and the two launches; `workspace` is the caller's buffer or this library's static one.
static hs_status prune_impl(const char* who, const int32_t* parent, const float* logc, const int32_t* node_offsets,
                            const int32_t* node_counts, int32_t B, int32_t NN, const int32_t* d_max,
                            const float* theta, const int32_t* max_nodes, int32_t* depth, float* cumlogp,
                            uint8_t* keep, int32_t* out_offsets, int32_t* out_src, int32_t* out_parent,
                            void* workspace, hs_stream stream) {
  (void)who;
  hs::Carver c(workspace);
  int32_t* ws_pos = c.take<int32_t>(NN > 0 ? NN : 1);
  int32_t* ws_parent = c.take<int32_t>(NN > 0 ? NN : 1);
  int32_t* ws_count = c.take<int32_t>(B);
  hipStream_t st = static_cast<hipStream_t>(stream);
  const hs::PruneArgs a{parent, node_offsets, node_counts, d_max, max_nodes, logc, theta, depth, cumlogp, keep,
                        ws_pos, ws_parent, ws_count, out_offsets, out_src, out_parent, B, NN};
  // (16 trees of 311 to 911 nodes: 11.3 us in workgroups of 512, 8.8 of 1024)
  if (NN > (int64_t)hs::PR_SMALL * B) hipLaunchKernelGGL(hs::k_prune_select<hs::PR_BIG>, dim3(B), dim3(hs::PR_BIG), 0, st, a);
  else hipLaunchKernelGGL(hs::k_prune_select<hs::PR_SMALL>, dim3(B), dim3(hs::PR_SMALL), 0, st, a);
  hs_status r = hs::launch_status("prune select");
  if (r != HS_OK) return r;
  // a single tree that fits LDS was emitted by the selecting workgroup itself
  if (B == 1 && NN <= hs::PR_LDS_NODES) return r;
  hipLaunchKernelGGL(hs::k_prune_emit, dim3(B), dim3(hs::PE_THREADS), 0, st, a);
  return hs::launch_status("prune emit");
}

#define HS_PRUNE_CHECK_ARGS(who)                                                                                      \
  HS_REQUIRE(B >= 0 && NN >= 0, HS_ERR_SHAPE, who ": B=%d NN=%d", B, NN);                                             \
  if (B == 0) return HS_OK;                                                                                           \
  HS_REQUIRE(node_offsets && d_max && theta && max_nodes && out_offsets, HS_ERR_NULL, who ": NULL argument");         \
  HS_REQUIRE(NN == 0 || (parent && logc && depth && cumlogp && keep && out_src && out_parent), HS_ERR_NULL,           \
             who ": NULL node array")

extern "C" hs_status hs_tree_prune_counted(const int32_t* parent, const float* logc, const int32_t* node_offsets,
                                           const int32_t* node_counts, int32_t B, int32_t NN, const int32_t* d_max,
                                           const float* theta, const int32_t* max_nodes, int32_t* depth,
                                           float* cumlogp, uint8_t* keep, int32_t* out_offsets, int32_t* out_src,
                                           int32_t* out_parent, void* workspace, size_t workspace_bytes,
                                           hs_stream stream) {
  hs::clear_error();
  HS_PRUNE_CHECK_ARGS("hs_tree_prune");
  const size_t need = hs_tree_prune_workspace(B, NN);
  HS_REQUIRE(workspace && workspace_bytes >= need && reinterpret_cast<uintptr_t>(workspace) % 256 == 0,
             HS_ERR_WORKSPACE, "hs_tree_prune: workspace needs %zu bytes, 256-byte aligned (got %zu)", need,
             workspace_bytes);
  return prune_impl("hs_tree_prune", parent, logc, node_offsets, node_counts, B, NN, d_max, theta, max_nodes, depth,
                    cumlogp, keep, out_offsets, out_src, out_parent, workspace, stream);
}

extern "C" hs_status hs_tree_prune(const int32_t* parent, const float* logc, const int32_t* node_offsets, int32_t B,
                                   int32_t NN, const int32_t* d_max, const float* theta, const int32_t* max_nodes,
                                   int32_t* depth, float* cumlogp, uint8_t* keep, int32_t* out_offsets,
                                   int32_t* out_src, int32_t* out_parent, void* workspace, size_t workspace_bytes,
                                   hs_stream stream) {
  return hs_tree_prune_counted(parent, logc, node_offsets, nullptr, B, NN, d_max, theta, max_nodes, depth, cumlogp,
                               keep, out_offsets, out_src, out_parent, workspace, workspace_bytes, stream);
}

// ---- hs_tree_prune_static: the same call for callers that cannot allocate (code under HIP graph
// capture, serving loops, harnesses that forbid hipMalloc).  Its scratch is a device array of this
// library, one copy per GPU, resolved once per device with hipGetSymbolAddress; every call on a GPU
// uses that GPU's copy, so calls that overlap on one GPU race.  Nothing in it has to start at zero:
// both kernels write every scratch entry they later read.
namespace {
constexpr int PRUNE_STATIC_MAX_NN = HS_PRUNE_STATIC_MAX_NODES;
constexpr int PRUNE_STATIC_MAX_B = HS_PRUNE_STATIC_MAX_SEQS;
constexpr size_t PRUNE_STATIC_BYTES = 2 * ((size_t)PRUNE_STATIC_MAX_NN * 4) + (size_t)PRUNE_STATIC_MAX_B * 4;  // 540672
constexpr int PRUNE_MAX_DEVICES = 64;
}  // namespace
static __device__ __align__(256) unsigned char scratch[PRUNE_STATIC_BYTES];
static void* scratch_of_device[PRUNE_MAX_DEVICES];  // the array's address on each GPU, once resolved

// The address of `scratch` on the current device (in host code the array's name is only a handle).
static hs_status static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= PRUNE_MAX_DEVICES)
    return hs::fail(HS_ERR_RUNTIME, "hs_tree_prune_static: no current device (%s)", hipGetErrorString(e));
  void* p = __atomic_load_n(&scratch_of_device[dev], __ATOMIC_ACQUIRE);
  if (p == nullptr) {
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      return hs::fail(HS_ERR_RUNTIME, "hs_tree_prune_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
    __atomic_store_n(&scratch_of_device[dev], p, __ATOMIC_RELEASE);  // (two threads may both resolve it: same value)
  }
  *out = p;
  return HS_OK;
}

extern "C" hs_status hs_tree_prune_static(const int32_t* parent, const float* logc, const int32_t* node_offsets,
                                          int32_t B, int32_t NN, const int32_t* d_max, const float* theta,
                                          const int32_t* max_nodes, int32_t* depth, float* cumlogp, uint8_t* keep,
                                          int32_t* out_offsets, int32_t* out_src, int32_t* out_parent,
                                          hs_stream stream) {
  hs::clear_error();
  HS_PRUNE_CHECK_ARGS("hs_tree_prune_static");
  HS_REQUIRE(B <= PRUNE_STATIC_MAX_B && NN <= PRUNE_STATIC_MAX_NN, HS_ERR_UNSUPPORTED,
             "hs_tree_prune_static: B=%d NN=%d exceed the static scratch (at most %d sequences, %d nodes); "
             "use hs_tree_prune with a workspace", B, NN, PRUNE_STATIC_MAX_B, PRUNE_STATIC_MAX_NN);
  static_assert(PRUNE_STATIC_MAX_NN % 64 == 0 && PRUNE_STATIC_MAX_B % 64 == 0, "the carved pieces stay 256-byte aligned");
  void* ws = nullptr;
  hs_status r = static_scratch(&ws);
  if (r != HS_OK) return r;
  return prune_impl("hs_tree_prune_static", parent, logc, node_offsets, nullptr, B, NN, d_max, theta, max_nodes, depth,
                    cumlogp, keep, out_offsets, out_src, out_parent, ws, stream);
}
