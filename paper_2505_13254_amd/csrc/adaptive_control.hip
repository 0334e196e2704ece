// hs_adaptive_control: complexity quantification of a draft tree and the decision that follows it
// (Section 4.1: cumulative meta-path Top-K entropy Phi of the operational path P*, Eq. 1;
// Section 4.2: entropy bins; Section 4.3: depth extension d' and node budget N').
//
// Nothing to stream: a few hundred nodes per sequence, one workgroup per sequence, no workspace.
// The tree is staged in LDS (up to 8192 rows; of larger ones the parents alone, or nothing).  A walk from each node
// to the root gives its depth and value (the float32 add per node of the reranking step, so the choice of P* is taken on
// the same numbers as the pruning that follows); one 64-bit (depth, value, row) key per node and a workgroup
// maximum pick P*; the first wave then sums the path's entropies root-first in float32 and looks up the bin.
// What bounds it is the chain of trips to memory and of barriers.  (Two walks from every node for
// the depths, the deepest nodes' values and the path's entropies from global memory: 511 rows 7.4 us, now 4.3.)
#include <limits.h>

#include "tree_settle.h"

namespace hs {

constexpr int CTL_THREADS = 512;
constexpr int CTL_MAX_BINS = 64;
constexpr int CTL_MAX_LOW = 8;
// Rows whose tree lies in LDS, at 16 bytes a row.  A compute unit holds one workgroup of the larger kernel, so calls of
// more sequences than there are compute units take the smaller one, of which it holds four; trees that outgrow that have their
// parents in the same 32 KB.  (1024 sequences of 61 / 511 / 1500 rows 10.6 / 12.4 / 19.2 us by the larger one, 4.4 / 5.8 / 10.1 by the
// smaller; with the parents in LDS alone, whatever the size, 7.8 / 7.8 / 13.1, and one sequence 8.3 / 7.9 / 12.0, now 3.7 / 3.8 / 5.6.)
constexpr int CTL_LDS_NODES = 8192, CTL_LDS_NODES_MANY = 2048;
constexpr int CTL_CUS = 256;

struct ControlArgs {
  const int32_t* parent;
  const float* logc;
  const float* ent;
  const int32_t* node_offsets;
  const int32_t* node_counts;
  int n_edges, n_low, alpha, d_base, n_default, mode;
  float edges[CTL_MAX_BINS - 1];
  float gamma[CTL_MAX_LOW];
  float* phi;
  int32_t* pstar;
  int32_t* bin;
  int32_t* d_prime;
  int32_t* n_prime;
};

// What bin b means (Section 4.3): depth extension and node budget.  One definition for the kernel and
// for the host query hs_adaptive_policy.
__host__ __device__ inline void bin_policy(int b, int n_low, int alpha, int d_base, int n_default, const float* gamma,
                                           int* d_prime, int* n_prime) {
  int delta = 0, budget = n_default;
  if (b < n_low) {
    delta = alpha - b > 0 ? alpha - b : 0;
    budget = (int)floor((double)gamma[b] * (double)n_default + 0.5) + delta;
  }
  *d_prime = d_base + delta;
  *n_prime = budget;
}

// (value, row) as one key: larger key = larger value, then lower row; never 0 for a real node.
__device__ __forceinline__ unsigned long long control_key(float v, int i) {
  return ((unsigned long long)order_bits(v) << 32) | (unsigned)(0x7fffffff - i);
}

// The ancestor of node i that is `up` levels above it.
template <typename IP>
__device__ __forceinline__ int ancestor(IP par, int i, int up) {
  for (; up > 0; --up) i = par[i];
  return i;
}

// The workgroup's largest key, in every thread (red_k: 0 before a barrier).
__device__ __forceinline__ unsigned long long best_key(unsigned long long best, unsigned long long* red_k) {
  best = wave_max_u64(best);
  if ((threadIdx.x & 63) == 0) atomicMax(red_k, best);
  __syncthreads();
  return *red_k;
}

// The decision, given P* = p at depth D (first wave): Eq. 1 along the path to P*, i.e. over the rows of its strict
// ancestors, root first.  The lanes fetch 64 path entries at a time side by side (one round trip instead of one
// per level); the float32 sum still takes them one by one in path order.
template <typename IP>
__device__ __forceinline__ void decide(const ControlArgs& a, int s, int p, int D, IP par, const float* __restrict__ ent) {
  const int lane = threadIdx.x;
  float acc = 0.f;
  for (int t0 = 0; t0 < D; t0 += 64) {
    const int t = t0 + lane;
    const float e = t < D ? ent[ancestor(par, p, D - t)] : 0.f;
    const int m = D - t0 < 64 ? D - t0 : 64;
    for (int l = 0; l < m; ++l) acc = acc + __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, e), l));
  }
  // (the boundaries are the lanes': one to each)
  const int b = __popcll(__ballot(lane < a.n_edges && acc >= a.edges[lane < a.n_edges ? lane : 0]));
  if (lane != 0) return;
  int dp, np_;
  bin_policy(b, a.n_low, a.alpha, a.d_base, a.n_default, a.gamma, &dp, &np_);
  a.phi[s] = acc;
  a.pstar[s] = p;
  a.bin[s] = b;
  a.d_prime[s] = dp;
  a.n_prime[s] = np_;
}

// Trees that do not fit LDS; `par` may.
template <typename IP>
__device__ __forceinline__ void control_large(const ControlArgs& a, int s, int o, int n, IP par, unsigned long long* red_k) {
  __shared__ int deepest;
  const int tid = threadIdx.x;
  const float* lc = a.logc + o;
  auto depth_of = [&](int i) {
    int d = 0;
    for (int j = par[i]; j >= 0; j = par[j]) ++d;
    return d;
  };
  if (tid == 0) {
    deepest = 0;
    *red_k = 0ull;
  }
  __syncthreads();
  int my_max = 0;
  for (int i = tid; i < n; i += CTL_THREADS) my_max = max(my_max, depth_of(i));
  my_max = (int)wave_max_u32((unsigned)my_max);
  if ((tid & 63) == 0) atomicMax(&deepest, my_max);
  __syncthreads();
  const int D = deepest;
  unsigned long long best = 0ull;
  for (int i = tid; i < n; i += CTL_THREADS) {
    if (depth_of(i) != D) continue;
    float v = 0.f;
    if (a.mode == 0)  // value of the root, then one float32 add per level, root first
      for (int t = 1; t <= D; ++t) v = v + fminf(lc[ancestor(par, i, D - t)], 0.f);
    else if (i != 0)
      v = fminf(lc[i], 0.f);
    const unsigned long long k = control_key(v, i);
    best = k > best ? k : best;
  }
  best = best_key(best, red_k);
  if (tid < 64) decide(a, s, 0x7fffffff - (int)(unsigned)(best & 0xffffffffull), D, par, a.ent + o);
}

template <int NODES>
__global__ __launch_bounds__(CTL_THREADS) void k_adaptive_control(ControlArgs a) {
  __shared__ unsigned long long red_k;
  __shared__ unsigned long long pool[2 * NODES];
  int* const l_par = reinterpret_cast<int*>(pool);
  float* const l_logc = reinterpret_cast<float*>(l_par + NODES);
  unsigned long long* const l_node = pool + NODES;  // deep trees: the nodes' words; else the entropies
  __shared__ int unsettled[3];
  const int s = blockIdx.x, tid = threadIdx.x;
  const int o = a.node_offsets[s];
  const int n = a.node_counts != nullptr ? a.node_counts[s] : a.node_offsets[s + 1] - o;
  if (n <= 0) {
    if (tid == 0) {
      a.phi[s] = 0.f;
      a.pstar[s] = -1;
      a.bin[s] = 0;
      a.d_prime[s] = a.d_base;
      a.n_prime[s] = a.n_default;
    }
    return;
  }
  if (n > NODES) {
    if (n <= 4 * NODES) {
      for (int i = tid; i < n; i += CTL_THREADS) l_par[i] = a.parent[o + i];
      control_large(a, s, o, n, (const int*)l_par, &red_k);  // (its first barrier comes before it looks at them)
    } else {
      control_large(a, s, o, n, a.parent + o, &red_k);
    }
    return;
  }
  float* const l_ent = reinterpret_cast<float*>(l_node);
  for (int i = tid; i < n; i += CTL_THREADS) {
    l_par[i] = a.parent[o + i];
    l_logc[i] = a.logc[o + i];
    l_ent[i] = a.ent[o + i];
  }
  if (tid < 3) unsettled[tid] = 0;
  if (tid == 0) red_k = 0ull;
  __syncthreads();
  // the best node of the deepest level: (depth, value, row) as one key
  static_assert(NODES <= 1 << 13, "13 bits of depth, 32 of value, 13 of row");
  auto key_of = [&](int i, unsigned long long w) {
    const float v = a.mode == 0 ? node_sum(w) : i == 0 ? 0.f : fminf(l_logc[i], 0.f);
    return ((unsigned long long)(unsigned)node_depth(w) << 45) | ((unsigned long long)order_bits(v) << 13) | (unsigned)(8191 - i);
  };
  auto any = [](bool, float, int) { return true; };
  unsigned long long best = 0ull;
  bool deep = false;
  for (int i = tid; i < n; i += CTL_THREADS) {
    const unsigned long long w = walk_node(l_par, l_logc, i, n, any);
    deep = deep || w == 0ull;
    best = max(best, key_of(i, w));
  }
  const float* ent = l_ent;
  if (__syncthreads_or(deep ? 1 : 0)) {
    ent = a.ent + o;
    for (int i = tid; i < n; i += CTL_THREADS) l_node[i] = i == 0 ? node_word(0.f, 0, true) : 0ull;
    __syncthreads();
    settle_nodes<CTL_THREADS, NODES>(l_par, l_logc, l_node, unsettled, n, any);
    best = 0ull;
    for (int i = tid; i < n; i += CTL_THREADS)
      if (l_node[i] != 0ull) best = max(best, key_of(i, l_node[i]));  // (0: not settled, a malformed tree)
  }
  best = best_key(best, &red_k);
  if (tid < 64) decide(a, s, 8191 - (int)(best & 8191ull), (int)(best >> 45), (const int*)l_par, ent);
}

}  // namespace hs

using namespace hs;

extern "C" hs_status hs_adaptive_control(const int32_t* parent, const float* logc, const float* ent,
                                         const int32_t* node_offsets, const int32_t* node_counts, int32_t B,
                                         int32_t NN, const float* host_bin_edges, int32_t n_bins, const float* host_gamma,
                                         int32_t n_low, int32_t alpha, int32_t d_base, int32_t n_default,
                                         hs_pstar_mode mode, float* phi, int32_t* pstar, int32_t* bin,
                                         int32_t* d_prime, int32_t* n_prime, hs_stream stream) {
  clear_error();
  HS_REQUIRE(B >= 0 && NN >= 0, HS_ERR_SHAPE, "hs_adaptive_control: B=%d NN=%d", B, NN);
  HS_REQUIRE(n_bins >= 1 && n_bins <= CTL_MAX_BINS, HS_ERR_SHAPE, "hs_adaptive_control: n_bins=%d must be in 1..%d",
             n_bins, CTL_MAX_BINS);
  HS_REQUIRE(n_low >= 0 && n_low <= CTL_MAX_LOW && n_low <= n_bins, HS_ERR_SHAPE,
             "hs_adaptive_control: n_low=%d must be in 0..min(%d, n_bins)", n_low, CTL_MAX_LOW);
  HS_REQUIRE(mode == HS_PSTAR_CUMULATIVE || mode == HS_PSTAR_LOCAL, HS_ERR_SHAPE, "hs_adaptive_control: mode %d",
             (int)mode);
  HS_REQUIRE(d_base >= 0 && n_default >= 0, HS_ERR_SHAPE, "hs_adaptive_control: d_base=%d n_default=%d", d_base,
             n_default);
  HS_REQUIRE((n_bins == 1 || host_bin_edges) && (n_low == 0 || host_gamma), HS_ERR_NULL,
             "hs_adaptive_control: NULL bin boundaries or gamma");
  for (int e = 0; e + 2 < n_bins; ++e)
    HS_REQUIRE(host_bin_edges[e] <= host_bin_edges[e + 1], HS_ERR_SHAPE,
               "hs_adaptive_control: bin boundaries must not decrease (entry %d)", e + 1);
  if (B == 0) return HS_OK;
  HS_REQUIRE(node_offsets && phi && pstar && bin && d_prime && n_prime, HS_ERR_NULL, "hs_adaptive_control: NULL argument");
  HS_REQUIRE(NN == 0 || (parent && logc && ent), HS_ERR_NULL, "hs_adaptive_control: NULL tree");
  ControlArgs a;
  a.parent = parent; a.logc = logc; a.ent = ent; a.node_offsets = node_offsets; a.node_counts = node_counts;
  a.n_edges = n_bins - 1; a.n_low = n_low; a.alpha = alpha; a.d_base = d_base; a.n_default = n_default;
  a.mode = (int)mode;
  for (int e = 0; e < CTL_MAX_BINS - 1; ++e) a.edges[e] = e < n_bins - 1 ? host_bin_edges[e] : 0.f;
  for (int e = 0; e < CTL_MAX_LOW; ++e) a.gamma[e] = e < n_low ? host_gamma[e] : 0.f;
  a.phi = phi; a.pstar = pstar; a.bin = bin; a.d_prime = d_prime; a.n_prime = n_prime;
  const dim3 grid((unsigned)B), block(CTL_THREADS);
  if (B > CTL_CUS && NN <= (int64_t)CTL_LDS_NODES_MANY * B)
    hipLaunchKernelGGL(k_adaptive_control<CTL_LDS_NODES_MANY>, grid, block, 0, static_cast<hipStream_t>(stream), a);
  else
    hipLaunchKernelGGL(k_adaptive_control<CTL_LDS_NODES>, grid, block, 0, static_cast<hipStream_t>(stream), a);
  return launch_status("adaptive control");
}

extern "C" hs_status hs_adaptive_policy(int32_t bin, const float* host_gamma, int32_t n_low, int32_t alpha,
                                        int32_t d_base, int32_t n_default, int32_t* host_d_prime,
                                        int32_t* host_n_prime) {
  clear_error();
  HS_REQUIRE(bin >= 0 && n_low >= 0 && n_low <= CTL_MAX_LOW && d_base >= 0 && n_default >= 0, HS_ERR_SHAPE,
             "hs_adaptive_policy: bin=%d n_low=%d d_base=%d n_default=%d", bin, n_low, d_base, n_default);
  HS_REQUIRE(host_d_prime && host_n_prime && (n_low == 0 || host_gamma), HS_ERR_NULL, "hs_adaptive_policy: NULL argument");
  int dp, np_;
  bin_policy(bin, n_low, alpha, d_base, n_default, host_gamma, &dp, &np_);
  *host_d_prime = dp;
  *host_n_prime = np_;
  return HS_OK;
}
