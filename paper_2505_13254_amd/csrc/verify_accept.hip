// hs_verify_accept: the accept walk over a verified draft tree (Section 2.1 acceptance rule, applied
// to the children of each node in turn).
//
// Stage A (all rows in parallel, HBM-bound): the row scan finds every target row's argmax and
// softmax normaliser (and every draft row's normaliser in the stochastic modes).
// Stage B (one workgroup per sequence, latency-bound):
//   greedy      every node checks in parallel whether its whole root path is confirmed by the
//               target's argmax; the deepest confirmed node is the end of the accepted path.
//   stochastic  the walk is serial by nature, but what a node's children face is not: the state
//               after j rejections at a node depends on the node and j alone, not on the path that
//               led there.  The residual itself is never materialised: after j rejections it is
//               max(p(v) - beta_j q(v), 0) for every token not yet rejected (beta_j a scalar that
//               accumulates Z_i / (1 - sum of rejected q)), and frozen at its value of the time
//               for a rejected token; only its normaliser is needed per rejection.  Whether a child is accepted
//               when its turn comes is thus known without the walk: a node's chain of rejections ends with its first
//               accepted child, for most nodes the first one, for which two probabilities are compared and nothing is
//               summed.  Of a node whose first child is rejected the tokens with p > q are sorted by p / q into buckets
//               with their sums (one kernel on the whole chip), after which every normaliser of its chain is two
//               suffix sums plus, from the second rejection on, the tokens of one bucket.  One
//               workgroup per node with children runs that node's chain, all nodes in parallel (k_accept_chain), and
//               leaves the accepted child; the walk is a chase through them, made by every workgroup of the kernel that
//               sums the row where it ends and draws the bonus token there (k_bonus_rows): an inverse-CDF search
//               done as row sums of 64 tokens, a scan of the row sums, and a scan inside the one row that is hit.
#include <limits.h>

#include <algorithm>

#include "tree_settle.h"

namespace hs {

constexpr int GR_THREADS = 256;
constexpr int GR_LDS_ROWS = 1024;  // tree rows that the greedy walk stages in LDS
constexpr int AC_THREADS = 1024;
constexpr int AC_WAVES = AC_THREADS / 64;
constexpr int AC_MAX_KIDS = 256;    // children tried per node
constexpr int AC_MAX_ROWS = 8192;   // 64-token rows of the CDF search held in LDS (V <= 524288)
constexpr int BR_SLICES = 64, BR_WGS = 1024;  // workgroups per sequence, and in all, that sum the row a bonus token is drawn from
constexpr int BR_THREADS = 512;
constexpr int BR_TRIP_ROWS = BR_THREADS / 64 * 4;  // 64-token rows that such a workgroup sums in a trip
constexpr int BR_FEW_ROWS = 2048;    // 64-token rows that most vocabularies have (V <= 131072)
constexpr int BK_NODES = 4096;      // calls with up to this many tree rows get the sorted residual (below)
constexpr int BK_SLICES = 16;       // vocabulary slices per row, each sorted by itself
constexpr int BK_N = 256;           // buckets of the ratio p / q: BK_PER_OCTAVE per factor of two, from 1 upwards
constexpr int BK_THREADS = 256;     // (one thread per bucket)
constexpr float BK_PER_OCTAVE = 32.f;
constexpr float FIX_SCALE = 0x1p62f;   // probabilities are summed as 64-bit integers in units of 2^-62:
constexpr double FIX_UNIT = 0x1p-62;   // the sums do not depend on the order of their terms

// ----------------------------------------------------------------------------------- greedy
// With n_slices > 1 the target rows' argmax arrives as one pair per row slice (the row scan's merge
// launch is folded into this kernel): the slice's largest key is the row's argmax, stored in `arg` for
// the walk.
__global__ __launch_bounds__(GR_THREADS) void k_accept_greedy(int32_t* __restrict__ arg,
                                                              const unsigned long long* __restrict__ slice_key, int n_slices,
                                                              const int32_t* __restrict__ token,
                                                              const int32_t* __restrict__ parent,
                                                              const int32_t* __restrict__ node_offsets,
                                                              int max_depth, int32_t* __restrict__ accept_len,
                                                              int32_t* __restrict__ accept_path,
                                                              int32_t* __restrict__ bonus_token) {
  __shared__ long long red[GR_THREADS / 64];
  const int s = blockIdx.x, tid = threadIdx.x;
  const int o = node_offsets[s];
  const int n = node_offsets[s + 1] - o;
  int32_t* path = accept_path + (int64_t)s * max_depth;
  for (int d = tid; d < max_depth; d += GR_THREADS) path[d] = -1;
  if (n <= 0) {
    if (tid == 0) {
      accept_len[s] = 0;
      bonus_token[s] = -1;
    }
    return;
  }
  // Trees of up to GR_LDS_ROWS rows are staged in LDS (parents, tokens, the rows' argmax), all of their
  // global reads in one trip: the walks below are chains of dependent reads, one per tree level.
  __shared__ int l_par[GR_LDS_ROWS], l_tok[GR_LDS_ROWS], l_arg[GR_LDS_ROWS];
  const bool staged = n <= GR_LDS_ROWS;
  if (staged) {
    for (int i = tid; i < n; i += GR_THREADS) {
      l_par[i] = parent[o + i];
      l_tok[i] = token[o + i];
    }
  }
  if (n_slices > 1) {
    for (int i = tid; i < n; i += GR_THREADS) {
      const int64_t base = (int64_t)(o + i) * n_slices;
      unsigned long long best = 0ull;
      for (int q = 0; q < n_slices; ++q) best = max(best, slice_key[base + q]);
      const int bi = best != 0ull ? (int)(0xffffffffu - (unsigned)best) : INT_MAX;
      arg[o + i] = bi;
      if (staged) l_arg[i] = bi;
    }
  } else if (staged) {
    for (int i = tid; i < n; i += GR_THREADS) l_arg[i] = arg[o + i];
  }
  __syncthreads();  // every row's argmax is visible to the workgroup
  // key = depth of a fully confirmed node (higher wins), then lower index
  long long best = ((long long)0 << 32) | (unsigned)(INT_MAX - 0);  // the root: depth 0
  for (int i = tid; i < n; i += GR_THREADS) {
    bool ok = true;
    int d = 0;
    if (staged) {
      for (int j = i; j > 0;) {
        const int p = l_par[j];
        ok = ok && (l_tok[j] == l_arg[p]);
        j = p;
        ++d;
      }
    } else {
      for (int j = i; j > 0;) {
        const int p = parent[o + j];
        ok = ok && (token[o + j] == arg[o + p]);
        j = p;
        ++d;
      }
    }
    if (ok && d <= max_depth) {
      long long key = ((long long)d << 32) | (unsigned)(INT_MAX - i);
      best = key > best ? key : best;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    long long other = __shfl_xor(best, off);
    best = other > best ? other : best;
  }
  if ((tid & 63) == 0) red[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < GR_THREADS / 64; ++w) best = red[w] > best ? red[w] : best;
    const int d = (int)(best >> 32);
    int node = INT_MAX - (int)(best & 0xffffffffll);
    accept_len[s] = d;
    bonus_token[s] = staged ? l_arg[node] : arg[o + node];
    for (int k = d - 1; k >= 0; --k) {
      path[k] = node;
      node = staged ? l_par[node] : parent[o + node];
    }
  }
}

// The greedy walk on its own, for calls of many rows: one workgroup to a sequence reads the rows of the path it
// takes and no others.  A level is one row streamed by one compute unit, which bounds it (128256 logits in 7.2 us, 71 GB/s;
// 32000 in 2.8), so a path costs levels, where the scan of every row costs bytes: see greedy_by_path.
//
// Nodes of a level that are confirmed (their root path is what the target's argmax says) are listed; usually there is
// one, several when siblings carry the same token.  Each gets its row's argmax, its children that carry it make up
// the next list, and the lowest row of the last list that is not empty ends the path, as in k_accept_greedy.
constexpr int GP_THREADS = 1024;
constexpr int GP_WAVES = GP_THREADS / 64;
constexpr int GP_LDS_ROWS = 4096;   // tree rows in LDS; of larger trees the lists and the argmax are in the workspace
constexpr int GP_AHEAD = 16;        // 16-byte loads that a lane has in flight
__global__ __launch_bounds__(GP_THREADS) void k_greedy_path(const float* __restrict__ target, int64_t row_stride, int V, int NN,
                                                            const int32_t* __restrict__ token,
                                                            const int32_t* __restrict__ parent,
                                                            const int32_t* __restrict__ node_offsets, int max_depth,
                                                            int32_t* __restrict__ ws_arg, int32_t* __restrict__ ws_list,
                                                            int32_t* __restrict__ accept_len,
                                                            int32_t* __restrict__ accept_path,
                                                            int32_t* __restrict__ bonus_token) {
  __shared__ int l_par[GP_LDS_ROWS], l_tok[GP_LDS_ROWS], l_arg[GP_LDS_ROWS];
  __shared__ int l_list[2][GP_LDS_ROWS];
  __shared__ int n_list[2];
  __shared__ unsigned long long wave_key[2][GP_WAVES];
  const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int o = node_offsets[s];
  const int n = node_offsets[s + 1] - o;
  int32_t* path = accept_path + (int64_t)s * max_depth;
  for (int d = tid; d < max_depth; d += GP_THREADS) path[d] = -1;
  if (n <= 0) {
    if (tid == 0) {
      accept_len[s] = 0;
      bonus_token[s] = -1;
    }
    return;
  }
  const bool staged = n <= GP_LDS_ROWS;
  if (staged)
    for (int i = tid; i < n; i += GP_THREADS) {
      l_par[i] = parent[o + i];
      l_tok[i] = token[o + i];
    }
  auto par_of = [&](int i) { return staged ? l_par[i] : parent[o + i]; };
  auto tok_of = [&](int i) { return staged ? l_tok[i] : token[o + i]; };
  auto put = [&](int which, int at, int node) {
    if (staged) l_list[which][at] = node;
    else ws_list[(int64_t)which * NN + o + at] = node;
  };
  auto get = [&](int which, int at) { return staged ? l_list[which][at] : ws_list[(int64_t)which * NN + o + at]; };
  if (tid == 0) {
    n_list[0] = 1;
    put(0, 0, 0);
  }
  __syncthreads();

  // The row's largest value with the lowest index, in every thread.  Chunk k is the row's elements 4096 k .. 4096 k + 4095,
  // four to a thread; a wave keeps its largest value so far and, per lane, the last four values that were above it: an
  // equal value of a later chunk has a higher index.
  constexpr int CHUNK = 4 * GP_THREADS;
  int turn = 0;
  auto row_argmax = [&](int node) {
    const float* __restrict__ x = target + (int64_t)(o + node) * row_stride;
    float thr = -HS_INF;
    float4 best = make_float4(-HS_INF, -HS_INF, -HS_INF, -HS_INF);
    int best_chunk = 0;
    auto take = [&](const float4 f, int k) {
      const float m = fmaxf(fmaxf(f.x, f.y), fmaxf(f.z, f.w));
      if (__ballot(m > thr) != 0ull) {
        if (m > thr) {
          best = f;
          best_chunk = k;
        }
        thr = wave_max(fmaxf(m, thr));
      }
    };
    // whole chunks by loads without conditions, the rest of the row by one that is requested first and looked at last
    const int n_full = V / CHUNK;
    float4 tail = make_float4(-HS_INF, -HS_INF, -HS_INF, -HS_INF);
    {
      const int i0 = n_full * CHUNK + tid * 4;
      if (i0 + 3 < V) {
        tail = load_float4(x + i0);
      } else {
        if (i0 < V) tail.x = x[i0];
        if (i0 + 1 < V) tail.y = x[i0 + 1];
        if (i0 + 2 < V) tail.z = x[i0 + 2];
        if (i0 + 3 < V) tail.w = x[i0 + 3];
      }
    }
    const float* __restrict__ src = x + tid * 4;
    auto load = [&](int k) { return load_float4(src + (int64_t)k * CHUNK); };
    float4 f[GP_AHEAD];
    int k = 0;
    if (n_full >= GP_AHEAD) {
#pragma unroll
      for (int u = 0; u < GP_AHEAD; ++u) f[u] = load(u);
      for (; k + 2 * GP_AHEAD <= n_full; k += GP_AHEAD)
#pragma unroll
        for (int u = 0; u < GP_AHEAD; ++u) {
          take(f[u], k + u);
          f[u] = load(k + u + GP_AHEAD);
        }
#pragma unroll
      for (int u = 0; u < GP_AHEAD; ++u) {
        take(f[u], k + u);
        if (k + u + GP_AHEAD < n_full) f[u] = load(k + u + GP_AHEAD);
      }
      k += GP_AHEAD;
    } else {
#pragma unroll
      for (int u = 0; u < GP_AHEAD; ++u)
        if (u < n_full) f[u] = load(u);
    }
#pragma unroll
    for (int u = 0; u < GP_AHEAD; ++u)
      if (k + u < n_full) take(f[u], k + u);
    take(tail, n_full);
    // the lane's best pair: of its four values the first that is the wave's largest
    const float m = fmaxf(fmaxf(best.x, best.y), fmaxf(best.z, best.w));
    const int e = best.x == m ? 0 : best.y == m ? 1 : best.z == m ? 2 : 3;
    const unsigned at = (unsigned)(best_chunk * CHUNK + tid * 4 + e);
    unsigned long long key = ((unsigned long long)order_bits(m + 0.f) << 32) | (0xffffffffu - at);
    key = wave_max_u64(key);
    unsigned long long* const keys = wave_key[turn & 1];  // (the other one may still be read)
    ++turn;
    if (lane == 0) keys[wave] = key;
    __syncthreads();
    key = wave_max_u64(lane < GP_WAVES ? keys[lane] : 0ull);
    return (int)(0xffffffffu - (unsigned)key);
  };

  int depth = 0, cur = 0;
  for (;;) {
    const int count = n_list[cur];
    if (tid == 0) n_list[cur ^ 1] = 0;
    __syncthreads();
    for (int c = 0; c < count; ++c) {
      const int node = get(cur, c);
      const int arg = row_argmax(node);
      if (tid == 0) {
        if (staged) l_arg[node] = arg;
        else ws_arg[o + node] = arg;
      }
      if (depth < max_depth)
        for (int i = 1 + tid; i < n; i += GP_THREADS)
          if (par_of(i) == node && tok_of(i) == arg) put(cur ^ 1, atomicAdd(&n_list[cur ^ 1], 1), i);
    }
    __syncthreads();
    if (n_list[cur ^ 1] == 0) break;
    cur ^= 1;
    ++depth;
  }
  // ---- the lowest row of the last list ends the path
  if (wave == 0) {
    unsigned best = 0u;
    for (int c = lane; c < n_list[cur]; c += 64) best = max(best, 0x7fffffffu - (unsigned)get(cur, c));
    int node = (int)(0x7fffffffu - wave_max_u32(best));
    if (lane == 0) {
      accept_len[s] = depth;
      bonus_token[s] = staged ? l_arg[node] : ws_arg[o + node];
      for (int k = depth - 1; k >= 0; --k) {
        path[k] = node;
        node = par_of(node);
      }
    }
  }
}

// Which of the two a greedy call takes: the scan of every row, or the rows of the paths alone, one after the other.  The
// longest path that the call allows decides, so that a tree whose path is as long as that is no slower than by the scan; sibling
// tokens differ, as everywhere (a level with several confirmed nodes is read row by row, right but slower).  Sequences of 61
// rows, paths of 1, 5 and 11 rows of a longest 11, whole calls of 12 to 13 us at least: 16 of 128256 tokens 91 us by the scan,
// 12.7, 41 and 86 by the paths; 64 of them 339 and 13, 43, 140; 64 of 32000 tokens 92 and 12.5, 21, 41; 200 of 8000 75 and
// 12.5, 14, 29.  (16 sequences of 8 to 128 nodes on 128256 tokens, the whole step: 382 us, 303.)  Looking for children in
// trees beyond LDS is priced on neither side: 3 us a level and 20000 rows here, but more in the walk that follows the scan
// (one tree of 60000 rows on 600 tokens, depth limit 10, all children of the root or at random depths: 258 and 826 us by the
// scan, 119 and 113 by the paths; of 9000 rows on 2000 tokens, limit 4, 45 and 111, 19 and 18).
static bool greedy_by_path(int B, int NN, int V, int max_depth) {
  const double row_bytes = 4.0 * V;
  const double scan_us = 6.0 + (double)NN * row_bytes / 6.0e6;
  const double row_us = fmax(2.0 + row_bytes / 1.0e5, (double)B * row_bytes / 2.2e6);
  return 6.0 + row_us * ((double)max_depth + 1.0) < scan_us;
}

// ----------------------------------------------------------------------------------- stochastic
// A row of logits as probabilities: p(v) = exp((x[v] - m) / T + lz) with m the row's maximum and
// lz = -ln(sum exp((x - m) / T)), evaluated as exp2((x[v] - m) * c1 + c2): a subtraction, a fused
// multiply-add and the exponential instruction per token.
struct RowView {
  const float* x;  // logits row
  float m;         // its maximum
  float c1;        // log2(e) / T
  float c2;        // log2(e) * lz
  __device__ __forceinline__ RowView(const float* row, float max_logit, float lz, float inv_t)
      : x(row), m(max_logit), c1(inv_t * 1.4426950408889634f), c2(lz * 1.4426950408889634f) {}
  __device__ __forceinline__ float arg(float logit) const { return fmaf(logit - m, c1, c2); }  // log2 p
  __device__ __forceinline__ float of(float logit) const { return exp2_fast(arg(logit)); }
  __device__ __forceinline__ float prob(int v) const { return of(x[v]); }
  __device__ __forceinline__ float4 of4(const float4 f) const { return make_float4(of(f.x), of(f.y), of(f.z), of(f.w)); }
  // tokens 4 i .. 4 i + 3 with one 16-byte load
  __device__ __forceinline__ float4 prob4(int i) const { return of4(load_float4(x + 4 * i)); }
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Sum over each row of 16 lanes; the row's last lane holds it.  DPP moves of the two halves of the
// double: a lane without a source takes 0.
__device__ __forceinline__ double row16_sum(double x) {
#define HS_DPP_ADD(ctrl, banks)                                                                              \
  x += __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), ctrl, 0xf, banks, false),          \
                        __builtin_amdgcn_update_dpp(0, __double2loint(x), ctrl, 0xf, banks, false))
  HS_DPP_ADD(0x111, 0xf);  // row_shr:1
  HS_DPP_ADD(0x112, 0xf);  // row_shr:2
  HS_DPP_ADD(0x114, 0xe);  // row_shr:4
  HS_DPP_ADD(0x118, 0xc);  // row_shr:8
#undef HS_DPP_ADD
  return x;
}

// Sum over the lanes of a wave, in every lane, by DPP moves.
__device__ __forceinline__ double wave_sum_dpp(double x) {
  x = row16_sum(x);  // lanes 15, 31, 47, 63
  const int lo = __double2loint(x), hi = __double2hiint(x);
  double t = __hiloint2double(__builtin_amdgcn_readlane(hi, 15), __builtin_amdgcn_readlane(lo, 15));
#pragma unroll
  for (int l = 31; l < 64; l += 16) t += __hiloint2double(__builtin_amdgcn_readlane(hi, l), __builtin_amdgcn_readlane(lo, l));
  return t;
}

// Inclusive prefix sums over the lanes of a wave: DPP moves inside the rows of 16 lanes, then the totals of the rows before.
__device__ __forceinline__ double wave_incl_scan(double v, int lane) {
  v = row16_sum(v);  // (each step adds what lies 1, 2, 4, 8 lanes to the left: every lane ends up with its prefix)
  const int lo = __double2loint(v), hi = __double2hiint(v);
  double before = 0.0;
#pragma unroll
  for (int l = 15; l < 63; l += 16) {
    const double t = __hiloint2double(__builtin_amdgcn_readlane(hi, l), __builtin_amdgcn_readlane(lo, l));
    before += lane > l ? t : 0.0;
  }
  return v + before;
}

// Sum of max(p(v) - beta q(v), 0) over the vocabulary, all threads of the workgroup; the result is
// the same in every thread.  Terms are formed in float32 (relative error 2^-24 of p(v)), summed in
// four float32 partial sums per thread over about V / (4 * threads) terms each, then in float64.
__device__ __forceinline__ double residual_mass(const RowView& p, const RowView& q, double beta, int V, double* red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float bf = (float)beta;
  float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
  // 16-byte loads, four of each row in flight per thread: a single compute unit streams the two
  // rows, so what is in flight bounds the pass
  const int n4 = V >> 2;
#pragma unroll 4
  for (int i = tid; i < n4; i += AC_THREADS) {
    const float4 pp = p.prob4(i), qq = q.prob4(i);
    a0 += fmaxf(fmaf(-bf, qq.x, pp.x), 0.f);
    a1 += fmaxf(fmaf(-bf, qq.y, pp.y), 0.f);
    a2 += fmaxf(fmaf(-bf, qq.z, pp.z), 0.f);
    a3 += fmaxf(fmaf(-bf, qq.w, pp.w), 0.f);
  }
  for (int v = (n4 << 2) + tid; v < V; v += AC_THREADS) a0 += fmaxf(fmaf(-bf, q.prob(v), p.prob(v)), 0.f);
  double acc = wave_sum(((double)a0 + (double)a1) + ((double)a2 + (double)a3));
  __syncthreads();  // red is free
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  double F = 0.0;
  for (int w = 0; w < AC_WAVES; ++w) F += red[w];
  return F;
}

// The same term for one token, as residual_mass forms it (used to take a frozen token's live term
// out of the sum again).
__device__ __forceinline__ double residual_term(const RowView& p, const RowView& q, double beta, int v) {
  return (double)fmaxf(fmaf(-(float)beta, q.prob(v), p.prob(v)), 0.f);
}
// Weight of token v in the distribution the bonus token is drawn from (frozen tokens aside).
__device__ __forceinline__ double token_weight(const RowView& p, const RowView& q, bool use_q, double beta, int v) {
  return use_q ? residual_term(p, q, beta, v) : (double)p.prob(v);
}

// Children of local row `cur` of a sequence of n rows, ascending, into kids_sorted; returns their
// number (at most AC_MAX_KIDS: of a node with more children the AC_MAX_KIDS lowest rows are taken,
// whatever order the threads arrive in).  Called by all threads; ends with a barrier.
template <int THREADS>
__device__ __forceinline__ int gather_children(const int* parent, int o, int n, int cur, bool any,
                                               int* kids, int* kids_sorted, int* n_kids) {
  const int tid = threadIdx.x;
  if (tid == 0) *n_kids = 0;
  __syncthreads();
  if (any)
    for (int i = 1 + tid; i < n; i += THREADS)
      if (parent[o + i] == cur) {
        int pos = atomicAdd(n_kids, 1);
        if (pos < AC_MAX_KIDS) kids[pos] = i;
      }
  __syncthreads();
  if (*n_kids > AC_MAX_KIDS) {
    // more children than the lists hold (never with Top-k expansion): which of them the atomic
    // counter let in depends on arrival order, so the lists are made again by rank, each child
    // counting the children before it; the first AC_MAX_KIDS stay
    for (int i = 1 + tid; i < n; i += THREADS)
      if (parent[o + i] == cur) {
        int r = 0;
        for (int j = 1; j < i && r < AC_MAX_KIDS; ++j) r += parent[o + j] == cur ? 1 : 0;
        if (r < AC_MAX_KIDS) kids_sorted[r] = i;
      }
    __syncthreads();
    return AC_MAX_KIDS;
  }
  const int nk = *n_kids;
  if (tid < nk) {
    int me = kids[tid], r = 0;
    for (int j = 0; j < nk; ++j) r += kids[j] < me ? 1 : 0;
    kids_sorted[r] = me;
  }
  __syncthreads();
  return nk;
}

// What the tree says about each row (k_tree_rows), and what the walk needs from a node's chain of rejections.
struct ChainOut {
  int32_t* n_tried;      // [NN] number of children the node's chain tries (0: the node's residual is p itself)
  int32_t* first;        // [NN] the first of them
  int32_t* kid_tok;      // [NN] its token
  float* kid_u;          // [NN] its uniform
  int32_t* accepted;     // [NN] the child that the chain ends with (a local row), -1: none is accepted
  double* child_frozen;  // [NN] where none is: the child's weight in the residual after its own rejection
  double* node_beta;     // [NN] and beta and normaliser after all of the node's children were rejected
  double* node_Z;
  double* bonus_rows;    // [NN][ceil(V / 64)] row sums of the distribution that the bonus token is drawn from, of the
                         // row where a sequence's walk ends (NULL: k_accept_walk makes them itself)
};

// The test of a child under the ratio rule: current target and draft probability of its token.
__device__ __forceinline__ bool ratio_accepts(double pc, double qc, float u) { return pc >= qc || (double)u * qc < pc; }

// ------------------------------------------------------------------ the sorted residual
// Along a node's chain of rejections only beta changes: F(beta) = sum_v max(p(v) - beta q(v), 0),
// taken at an increasing sequence of beta >= 1 that is not known in advance, but for the first:
// 1.  A token contributes p - beta q while its ratio p / q exceeds beta and nothing afterwards.  So, for
// every node with at least two children (of long rows: with one), a kernel that runs on the whole chip sorts the tokens with p > q of each
// vocabulary slice by their ratio into BK_N buckets (a counting sort inside a workgroup: count, then place) and keeps,
// per bucket, the sums of p and of q.  F(1) is the sum of all of them, F(beta)
//     sum over the buckets well above beta of (P_b - beta Q_b)      two suffix sums, read once
//   + sum over the tokens of beta's bucket (and of the next one where beta is near its edge) of max(p - beta q, 0)
// which is what k_accept_chain evaluates per rejection: about a thousand pairs instead of two
// vocabulary rows.  (Sorted across slices, with a scan and a second pass over the rows in launches of
// their own: 23.6 us for a 61-row tree; slice by slice, read twice, 15.7; kept in registers for the second pass, now, 11.7.)
// A token's bucket is floor(BK_PER_OCTAVE * log2(p / q)), taken from the two
// exponent arguments (p = exp2(a_p)): the rounding of that difference is many orders below a
// bucket's width, and where beta lies near the edge of a bucket the next one is treated token by token as well, so
// no token is ever taken for live or dead by its bucket alone when it is not.  All sums are 64-bit
// integers in units of 2^-62 (LDS and per-slice partial sums), so neither the order in which the
// lanes' atomic additions arrive nor the order of the tokens inside a bucket changes a result.
// (A chain of one rejection needs the sums alone: no pairs are written for it.)
// Nodes with one child are sorted where rows are long.  Their own workgroup of k_accept_chain makes the one sum
// in a pass over both rows as well, 3 us of 32000 tokens and 10 of 128256, all nodes side by side, while the sort reads the rows of every
// node with the whole chip before it knows that a first child is accepted.  Whole calls, chains of single children all rejected, without the sort and
// with it: one tree of 9 rows of 128256 tokens 41.6 us and 35.2, of 31 47.4 and 40.8, 4 trees of 9 48.8 and 47.1, 16 of 9 84.9 and 90.0; one
// of 9 of 65536 tokens 34.2 and 31.8, of 50257 33.0 and 31.8, of 32000 29.2 and 29.7; but 16 of 9 of 50257 tokens 51.0 and 59.1, of 32000 41.9 and 50.2, of 8192 31.7 and
// 36.8, of 4096 28.1 and 34.5.  Trees that branch, 33 to 640 rows: within 2 % of each other on 32000 tokens, on 128256 up to 6 % faster with the sort.
constexpr int BK_SINGLE_V = 65536;
__device__ __forceinline__ int sorted_from(int V) { return V >= BK_SINGLE_V ? 1 : 2; }  // children of a node that is sorted
struct BucketWs {
  uint32_t* start;            // [NN][BK_SLICES][BK_N + 1] first position in `pairs` of a slice's buckets (ascending ratio)
  unsigned long long* psum;   // [NN][BK_SLICES][BK_N] sum of p over a slice's bucket
  unsigned long long* qsum;   // [NN][BK_SLICES][BK_N] sum of q over it
  float2* pairs;              // [NN][V] (p, q) of the live tokens, slice by slice, bucket by bucket
};

__device__ __forceinline__ int bucket_of(float ap, float aq) {
  return (int)fminf(fmaxf((ap - aq) * BK_PER_OCTAVE, 0.f), (float)(BK_N - 1));
}
__device__ __forceinline__ unsigned long long to_fixed(float x) { return (unsigned long long)(x * FIX_SCALE); }

// grid (BK_SLICES, NN): sorts slice blockIdx.x of row blockIdx.y, if the row has children and the first is rejected.
__global__ __launch_bounds__(BK_THREADS) void k_bucket_sort(const float* __restrict__ target, const float* __restrict__ draft,
                                                            int64_t row_stride, int V, float inv_t,
                                                            ChainOut chain, const int32_t* __restrict__ t_arg,
                                                            const float* __restrict__ t_lz, const int32_t* __restrict__ d_arg,
                                                            const float* __restrict__ d_lz, BucketWs ws) {
  static_assert(BK_THREADS == BK_N, "a thread per bucket");
  __shared__ unsigned cnt[BK_N];  // tokens of a bucket; then its next free position
  __shared__ unsigned long long ps[BK_N], qs[BK_N];
  __shared__ unsigned wave_total[BK_N / 64];
  const int slice = blockIdx.x, g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // (one trip for what the row's statistics say, one for the slice and the two maxima)
  const int nk = chain.n_tried[g], p_arg = t_arg[g], q_arg = d_arg[g], x0 = chain.kid_tok[g];
  const float p_lz = t_lz[g], q_lz = d_lz[g], u0 = chain.kid_u[g];
  if (nk < sorted_from(V)) return;
  cnt[tid] = 0u;
  ps[tid] = 0ull;
  qs[tid] = 0ull;
  const float* p_row = target + (int64_t)g * row_stride;
  const float* q_row = draft + (int64_t)g * row_stride;
  const int n4 = V >> 2;
  const int per = (n4 + BK_SLICES - 1) / BK_SLICES;
  const int i0 = min(n4, slice * per), i1 = min(n4, i0 + per);
  const int tail = slice == BK_SLICES - 1 ? V & 3 : 0;  // the last V % 4 tokens are the last slice's
  auto px = [&](int i) { return load_float4(p_row + 4 * i); };
  auto qx = [&](int i) { return load_float4(q_row + 4 * i); };
  // A thread's tokens stay in its registers for both passes where they fit, requested all at once.  (Read twice, two at a
  // time: 61 rows of 128256 tokens 15.7 us, 12.1 so; 97 rows 28.7 and 19.8.)
  constexpr int KEEP = 8;
  const bool kept = i1 - i0 <= KEEP * BK_THREADS;
  float4 fp[KEEP], fq[KEEP];
  if (kept) {
#pragma unroll
    for (int u = 0; u < KEEP; ++u) {
      const int i = i0 + tid + u * BK_THREADS;
      const bool mine = i < i1;  // (p = q = 0 elsewhere: not live)
      fp[u] = mine ? px(i) : make_float4(-HS_INF, -HS_INF, -HS_INF, -HS_INF);
      fq[u] = mine ? qx(i) : make_float4(-HS_INF, -HS_INF, -HS_INF, -HS_INF);
    }
  }
  const RowView p(p_row, p_row[p_arg], p_lz, inv_t);
  const RowView q(q_row, q_row[q_arg], q_lz, inv_t);
  if (ratio_accepts((double)p.prob(x0), (double)q.prob(x0), u0)) return;  // (the chain ends with its first child)
  auto each_token = [&](auto token) {
    auto four = [&](const float4 a, const float4 b) {
      token(a.x, b.x);
      token(a.y, b.y);
      token(a.z, b.z);
      token(a.w, b.w);
    };
    if (kept) {
#pragma unroll
      for (int u = 0; u < KEEP; ++u)
        if (i0 + tid + u * BK_THREADS < i1) four(fp[u], fq[u]);
    } else {
#pragma unroll 2
      for (int i = i0 + tid; i < i1; i += BK_THREADS) four(px(i), qx(i));
    }
    if (tid < tail) token(p_row[(n4 << 2) + tid], q_row[(n4 << 2) + tid]);
  };
  __syncthreads();
  each_token([&](float xp, float xq) {
    const float ap = p.arg(xp), aq = q.arg(xq);
    const float pv = exp2_fast(ap), qv = exp2_fast(aq);
    if (pv > qv) {  // live at beta = 1, where every chain starts
      const int b = bucket_of(ap, aq);
      atomicAdd(&cnt[b], 1u);
      atomicAdd(&ps[b], to_fixed(pv));
      atomicAdd(&qs[b], to_fixed(qv));
    }
  });
  __syncthreads();
  const int64_t slot = (int64_t)g * BK_SLICES + slice;
  ws.psum[slot * BK_N + tid] = ps[tid];
  ws.qsum[slot * BK_N + tid] = qs[tid];
  if (nk == 1) return;  // (nothing comes behind the first rejection, which needs the sums alone)
  const unsigned mine = cnt[tid];
  const unsigned incl = (unsigned)wave_prefix_sum((int)mine);
  if (lane == 63) wave_total[wave] = incl;
  __syncthreads();
  unsigned first = (unsigned)i0 * 4u + incl - mine;
  for (int w = 0; w < wave; ++w) first += wave_total[w];
  ws.start[slot * (BK_N + 1) + tid] = first;
  if (tid == BK_N - 1) ws.start[slot * (BK_N + 1) + BK_N] = first + mine;
  cnt[tid] = first;
  __syncthreads();
  float2* __restrict__ pairs = ws.pairs + (int64_t)g * V;
  each_token([&](float xp, float xq) {
    const float ap = p.arg(xp), aq = q.arg(xq);
    const float pv = exp2_fast(ap), qv = exp2_fast(aq);
    if (pv > qv) pairs[atomicAdd(&cnt[bucket_of(ap, aq)], 1u)] = make_float2(pv, qv);
  });
}

// Sums of 64-bit integers over the lanes of a wave by DPP moves of their halves: inclusive prefix sums ...
__device__ __forceinline__ unsigned long long wave_prefix_sum(unsigned long long x) {
#define HS_DPP_STEP(ctrl, rows, banks)                                                                                       \
  x += ((unsigned long long)(unsigned)__builtin_amdgcn_update_dpp(0, (int)(x >> 32), ctrl, rows, banks, false) << 32) |     \
       (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, banks, false)
  HS_DPP_STEP(0x111, 0xf, 0xf);  // row_shr:1
  HS_DPP_STEP(0x112, 0xf, 0xf);  // row_shr:2
  HS_DPP_STEP(0x114, 0xf, 0xe);  // row_shr:4
  HS_DPP_STEP(0x118, 0xf, 0xc);  // row_shr:8
  HS_DPP_STEP(0x142, 0xa, 0xf);  // row_bcast:15
  HS_DPP_STEP(0x143, 0xc, 0xf);  // row_bcast:31
#undef HS_DPP_STEP
  return x;
}
// ... and the last lane's, in every lane: the sum.
__device__ __forceinline__ unsigned long long wave_total(unsigned long long x) {
  x = wave_prefix_sum(x);
  return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(x >> 32), 63) << 32) |
         (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}

// A row's bucket tables in LDS, made once per chain from the slices' (the chain is serial: what it reads
// per rejection should not be a round trip to memory).
struct BucketTables {
  unsigned start[BK_SLICES][BK_N + 1];
  unsigned long long sp[BK_N + 1], sq[BK_N + 1];  // sums of p and of q over the buckets >= b
};
// What a thread requests of them, ahead of everything that the tree says ...
constexpr int BT_PARTS = AC_THREADS / BK_N, BT_PER = BK_SLICES / BT_PARTS;
static_assert(BT_PARTS * BK_N == AC_THREADS && BT_PER * BT_PARTS == BK_SLICES, "a thread per bucket and group of slices");
constexpr int BT_STARTS = (BK_SLICES * (BK_N + 1) + AC_THREADS - 1) / AC_THREADS;
struct BucketLoads {
  unsigned long long p[BT_PER], q[BT_PER];
  unsigned start[BT_STARTS];
};
__device__ __forceinline__ void request_bucket_tables(const BucketWs& ws, int g, BucketLoads& l) {
  const int tid = threadIdx.x, b = tid % BK_N, part = tid / BK_N;
  const int64_t first = (int64_t)g * BK_SLICES;
#pragma unroll
  for (int k = 0; k < BT_PER; ++k) {
    l.p[k] = ws.psum[(first + part * BT_PER + k) * BK_N + b];
    l.q[k] = ws.qsum[(first + part * BT_PER + k) * BK_N + b];
  }
#pragma unroll
  for (int k = 0; k < BT_STARTS; ++k) {
    const int e = tid + k * AC_THREADS;
    l.start[k] = ws.start[first * (BK_N + 1) + (e < BK_SLICES * (BK_N + 1) ? e : 0)];
  }
}
// ... and what becomes of it (all AC_THREADS threads; no barrier at the end).
__device__ __forceinline__ void make_bucket_tables(const BucketLoads& l, BucketTables& t) {
  __shared__ unsigned long long part_p[BT_PARTS][BK_N], part_q[BT_PARTS][BK_N], wave_p[BK_N / 64], wave_q[BK_N / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  {
    const int b = tid % BK_N, part = tid / BK_N;
    unsigned long long tp = 0ull, tq = 0ull;
#pragma unroll
    for (int k = 0; k < BT_PER; ++k) {
      tp += l.p[k];
      tq += l.q[k];
    }
    part_p[part][b] = tp;
    part_q[part][b] = tq;
  }
#pragma unroll
  for (int k = 0; k < BT_STARTS; ++k) {
    const int e = tid + k * AC_THREADS;
    if (e < BK_SLICES * (BK_N + 1)) (&t.start[0][0])[e] = l.start[k];
  }
  __syncthreads();
  unsigned long long ip = 0ull, iq = 0ull;
  const int b = BK_N - 1 - tid;  // (from the top: prefix sums over the threads are suffix sums over the buckets)
  if (tid < BK_N) {
#pragma unroll
    for (int k = 0; k < BT_PARTS; ++k) {
      ip += part_p[k][b];
      iq += part_q[k][b];
    }
    ip = wave_prefix_sum(ip);
    iq = wave_prefix_sum(iq);
    if (lane == 63) {
      wave_p[tid >> 6] = ip;
      wave_q[tid >> 6] = iq;
    }
  }
  __syncthreads();
  if (tid < BK_N) {
    for (int w = 0; w < (tid >> 6); ++w) {
      ip += wave_p[w];
      iq += wave_q[w];
    }
    t.sp[b] = ip;
    t.sq[b] = iq;
    if (tid == 0) t.sp[BK_N] = t.sq[BK_N] = 0ull;
  }
}

// What the first wave hands to the others for one rejection, and what they hand back.
struct BucketStep {
  int stop;                            // the chain has ended: a child was accepted
  double beta;
  int b_lo, b_hi;                      // buckets whose tokens are taken one by one
  unsigned long long part[AC_WAVES];   // their terms, summed per wave
};

// beta's own bucket, with the next one on the side where beta lies within a hundredth of a bucket of the edge: [b_lo,
// b_hi).  NaN and infinity end up at valid indices as well; float32 is enough to pick the bucket, as it is for the tokens'
// buckets: the difference of two exponent arguments below 2^7, times 32, is off by 1e-3 of a bucket at most, and so
// is beta's place, so tokens beyond are live, or not, as a bucket.  (One bucket to either side always: three times the
// pairs, 2.3 us a step instead of 2.0.)
__device__ __forceinline__ void near_buckets(double beta, int& b_lo, int& b_hi) {
  const float place = fminf(fmaxf(__log2f((float)beta) * BK_PER_OCTAVE, 0.f), (float)(BK_N - 1));
  const int own = (int)place;
  const float inside = place - (float)own;
  b_lo = own > 0 && !(inside > 0.01f) ? own - 1 : own;
  b_hi = own + 1 < BK_N && !(inside < 0.99f) ? own + 2 : own + 1;
}

// The terms max(p - beta q, 0) of the pairs in buckets [b_lo, b_hi), a slice to a wave, summed per wave
// into step.part.  They are formed in float64 and summed as integers in units of 2^-52 (the fraction
// bits of 1 + term, term < 1): the order of the pairs inside a bucket, which the sort's atomic
// additions decide, does not reach the result.
__device__ __forceinline__ void near_terms(const float2* __restrict__ pairs, const BucketTables& t, BucketStep& step) {
  static_assert(AC_WAVES == BK_SLICES, "a slice to a wave");
  constexpr int AHEAD = 8;  // pairs a lane requests together: one trip to memory for about 500 pairs of a slice
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double beta = step.beta;
  const int lo = (int)t.start[wave][step.b_lo], hi = (int)t.start[wave][step.b_hi];
  unsigned long long acc = 0ull;
  for (int i = lo + lane; i < hi; i += 64 * AHEAD) {
    float2 e[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) e[u] = i + 64 * u < hi ? pairs[i + 64 * u] : make_float2(0.f, 0.f);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const double term = fmin(fmax((double)e[u].x - beta * (double)e[u].y, 0.0), 0x1.fffffffffffffp-1);
      acc += (unsigned long long)__double_as_longlong(1.0 + term) & 0xfffffffffffffull;
    }
  }
  acc = wave_total(acc);
  if (lane == 0) step.part[wave] = acc;
}

// One workgroup per sequence, ahead of everything else: what the tree says about each row.
//   wanted    the rows the scan of [target rows ; draft rows] has to read: every target row
//             (wanted[row] = 1) and the draft rows of the rows that are somebody's parent
//             (wanted[NN + row]; nobody reads the draft row of a row without children)
//   n_tried   children that the row's chain tries: none below the last level that may be accepted
//   first     the first of them (a local row), kid_tok and kid_u its token and uniform: what later kernels need
//             to tell whether there is a chain at all
//   tickets   the scan's counters of these rows, cleared (its slices are merged by its own launch)
// (Every later kernel used to walk from its row to the root for the depth, a chain of global reads.)
__global__ __launch_bounds__(GR_THREADS) void k_tree_rows(const int32_t* __restrict__ parent,
                                                          const int32_t* __restrict__ node_offsets,
                                                          const int32_t* __restrict__ token, const float* __restrict__ uniforms,
                                                          int NN, int max_depth, uint8_t* __restrict__ wanted, ChainOut chain,
                                                          unsigned* __restrict__ tickets) {
  __shared__ int l_par[GR_LDS_ROWS], l_kids[GR_LDS_ROWS], l_first[GR_LDS_ROWS], l_tok[GR_LDS_ROWS];
  __shared__ float l_u[GR_LDS_ROWS];
  int32_t* const n_tried = chain.n_tried;
  const int s = blockIdx.x, tid = threadIdx.x;
  const int o = node_offsets[s];
  const int n = node_offsets[s + 1] - o;
  const bool staged = n <= GR_LDS_ROWS;
  if (s == (int)gridDim.x - 1)
    for (int g = o + n + tid; g < NN; g += GR_THREADS) {  // rows behind the last sequence: nobody's
      wanted[g] = 0;
      wanted[NN + g] = 0;
      n_tried[g] = 0;
      tickets[g] = 0u;
      tickets[NN + g] = 0u;
    }
  for (int i = tid; i < n; i += GR_THREADS) {
    wanted[o + i] = 1;
    tickets[o + i] = 0u;
    tickets[NN + o + i] = 0u;
    if (staged) {
      l_par[i] = parent[o + i];
      l_tok[i] = token[o + i];
      l_u[i] = uniforms[o + i];
      l_kids[i] = 0;
      l_first[i] = INT_MAX;
    } else {
      n_tried[o + i] = 0;
      chain.first[o + i] = INT_MAX;
    }
  }
  __syncthreads();
  for (int i = 1 + tid; i < n; i += GR_THREADS) {
    if (staged) {
      atomicAdd(&l_kids[l_par[i]], 1);
      atomicMin(&l_first[l_par[i]], i);
    } else {
      atomicAdd(&n_tried[o + parent[o + i]], 1);
      atomicMin(&chain.first[o + parent[o + i]], i);
    }
  }
  __syncthreads();
  for (int i = tid; i < n; i += GR_THREADS) {
    int depth = 0;
    if (staged)
      for (int j = l_par[i]; j >= 0; j = l_par[j]) ++depth;
    else
      for (int j = parent[o + i]; j >= 0; j = parent[o + j]) ++depth;
    const int kids = staged ? l_kids[i] : __hip_atomic_load(&n_tried[o + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (kids > 0) {
      const int c = staged ? l_first[i] : __hip_atomic_load(&chain.first[o + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (staged) chain.first[o + i] = c;
      chain.kid_tok[o + i] = staged ? l_tok[c] : token[o + c];
      chain.kid_u[o + i] = staged ? l_u[c] : uniforms[o + c];
    }
    wanted[NN + o + i] = kids > 0 ? 1 : 0;
    n_tried[o + i] = depth < max_depth ? min(kids, AC_MAX_KIDS) : 0;
  }
}

// Sums of the bonus distribution's weights over rows of 64 tokens, rows [r_begin, r_end) of a node,
// by all waves of the workgroup: dst[r] for each of them.  A lane takes four tokens, 16 lanes a row, a
// wave four rows per trip; the loads of four trips are requested together (lanes past the last row
// re-read it), and a row's 16 partial sums meet in its last lane by DPP moves.  Rows that are not
// whole are summed a token per lane.  A row's sum
// does not depend on who computes it: the walk and k_bonus_rows give the same bits.  SHARED: another workgroup of the launch
// reads them.
template <bool SHARED>
__device__ __forceinline__ void bonus_row_sums(const RowView& p, const RowView& q, bool sub_q, double beta, int V,
                                               int r_begin, int r_end, double* __restrict__ dst) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n_waves = blockDim.x >> 6;
  auto put = [&](int r, double w) {
    if (SHARED) st_dev(reinterpret_cast<unsigned long long*>(dst) + r, __builtin_bit_cast(unsigned long long, w));
    else dst[r] = w;
  };
  int first_row = r_begin;  // rows below it were summed with 16-byte loads
  if (V >= 64) {
    constexpr int TRIPS = 4;
    const int full_end = min(V >> 6, r_end);
    const int sub = lane >> 4, l16 = lane & 15;
    const float bf = (float)beta;
    for (int r0 = r_begin + wave * 4; r0 < full_end; r0 += n_waves * 4 * TRIPS) {
      float4 fp[TRIPS], fq[TRIPS];
#pragma unroll
      for (int u = 0; u < TRIPS; ++u) {
        const int r = min(r0 + u * n_waves * 4 + sub, full_end - 1);
        fp[u] = load_float4(p.x + r * 64 + l16 * 4);
        fq[u] = sub_q ? load_float4(q.x + r * 64 + l16 * 4) : fp[u];
      }
#pragma unroll
      for (int u = 0; u < TRIPS; ++u) {
        const int r = r0 + u * n_waves * 4 + sub;
        const float4 pp = p.of4(fp[u]);
        double w;
        if (sub_q) {
          const float4 qq = q.of4(fq[u]);
          w = ((double)fmaxf(fmaf(-bf, qq.x, pp.x), 0.f) + (double)fmaxf(fmaf(-bf, qq.y, pp.y), 0.f)) +
              ((double)fmaxf(fmaf(-bf, qq.z, pp.z), 0.f) + (double)fmaxf(fmaf(-bf, qq.w, pp.w), 0.f));
        } else {
          w = ((double)pp.x + (double)pp.y) + ((double)pp.z + (double)pp.w);
        }
        w = row16_sum(w);
        if (l16 == 15 && r < full_end) put(r, w);
      }
    }
    first_row = max(full_end, r_begin);
  }
  for (int r = first_row + wave; r < r_end; r += n_waves) {
    const int v = r * 64 + lane;
    double w = v < V ? token_weight(p, q, sub_q, beta, v) : 0.0;
    w = wave_sum(w);
    if (lane == 0) put(r, w);
  }
}

// One workgroup per tree row that has children (others leave at once): the chain of rejections at that node under the
// ratio rule.  Whether a child is accepted when its turn comes depends on the node, its uniform and the rejections before it, so the
// chain ends with the first accepted child, usually the first child, before anything but its two probabilities has
// been looked at.  (With every child rejected in turn, whatever the uniforms, and the rows of p summed here for every row
// without children: 22.4 us for the 61 rows of 128256 tokens of the 8B step, now 14.4; with all chains run to their ends the same as before.)
__global__ __launch_bounds__(AC_THREADS) void k_accept_chain(
    const float* __restrict__ target, const float* __restrict__ draft, int64_t row_stride,
    const int32_t* __restrict__ token, const int32_t* __restrict__ parent, const int32_t* __restrict__ node_offsets,
    int B, int V, float inv_t, const float* __restrict__ uniforms, const int32_t* __restrict__ t_arg, const float* __restrict__ t_lz,
    const int32_t* __restrict__ d_arg, const float* __restrict__ d_lz, ChainOut out, BucketWs bk) {
  __shared__ int kids[AC_MAX_KIDS];
  __shared__ int kids_sorted[AC_MAX_KIDS];
  __shared__ int n_kids;
  __shared__ double rej_w[AC_MAX_KIDS];
  __shared__ float kid_p[AC_MAX_KIDS], kid_q[AC_MAX_KIDS], kid_u[AC_MAX_KIDS];  // p(x), q(x) of each child's token, its uniform
  __shared__ double red[AC_WAVES];
  __shared__ BucketTables tables;
  __shared__ BucketStep step;
  const int g = blockIdx.x, tid = threadIdx.x;
  // (row statistics first: these loads do not depend on the tree)
  const float p_lz = t_lz[g], q_lz = d_lz[g], u0 = out.kid_u[g];
  const int p_arg = t_arg[g], q_arg = d_arg[g], x0 = out.kid_tok[g], first = out.first[g];
  const int nk = out.n_tried[g];
  int lo = 0, hi = B;  // sequence of this row: last s with node_offsets[s] <= g
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (node_offsets[mid] <= g) lo = mid; else hi = mid;
  }
  const int o = node_offsets[lo];
  const int n = node_offsets[lo + 1] - o;
  const int cur = g - o;
  if (cur >= n) return;  // (a row behind the last sequence)
  if (nk == 0) {
    if (tid == 0) out.accepted[g] = -1;
    return;
  }
  const float* p_row = target + (int64_t)g * row_stride;
  const float* q_row = draft + (int64_t)g * row_stride;
  const RowView p(p_row, p_row[p_arg], p_lz, inv_t);
  const RowView q(q_row, q_row[q_arg], q_lz, inv_t);
  if (ratio_accepts((double)p.prob(x0), (double)q.prob(x0), u0)) {
    if (tid == 0) out.accepted[g] = first;
    return;
  }
  const bool sorted = bk.pairs != nullptr && nk >= sorted_from(V);  // there is a sorted residual
  // Everything is requested side by side: the tables, the children and their tokens, then the tokens' logits; the chain
  // below is serial, and a round trip to memory per step would dominate it.
  BucketLoads loads;
  if (sorted) request_bucket_tables(bk, g, loads);
  gather_children<AC_THREADS>(parent, o, n, cur, true, kids, kids_sorted, &n_kids);
  float xp = 0.f, xq = 0.f;
  if (tid < nk) {
    const int c = o + kids_sorted[tid];
    const int x = token[c];
    kid_u[tid] = uniforms[c];
    xp = p_row[x];
    xq = q_row[x];
  }
  if (sorted) make_bucket_tables(loads, tables);
  if (tid < nk) {
    kid_p[tid] = p.of(xp);
    kid_q[tid] = q.of(xq);
  }
  __syncthreads();
  const float2* __restrict__ pairs = sorted ? bk.pairs + (int64_t)g * V : nullptr;
  double beta = 0.0, Z = 1.0, sumq = 0.0;
  int acc = -1;  // the accepted child's place among the children
  if (sorted) {
    // The first wave keeps the chain's scalars; the others only help with the tokens around beta.
    // (Sixteen waves that all repeat the scalar part take issue slots from one another: 4 us a step.)
    // A step is a chain of its own, two divisions, two barriers and a trip to memory, so whatever is not
    // part of it is left for later or for other lanes: the rejected tokens' corrections are a lane each, sums travel by DPP
    // moves.  (61 rows, chains of ten: 2.0 us a step, most of it the trip to memory, and 0.6 for the first; 2.6 and a
    // trip before.)
    const bool lead = tid < 64;
    const int lane = tid & 63;
    for (int j = 0; j < nk; ++j) {
      int b_hi = 0;
      if (lead && acc < 0) {
        const double px = (double)kid_p[j], qx = (double)kid_q[j];
        const double rem = 1.0 - sumq;
        // (current p(x) and q(x); the first child was rejected above)
        if (j > 0 && ratio_accepts(fmax(px - beta * qx, 0.0) / Z, qx / rem, kid_u[j])) {
          acc = j;
        } else {
          // rejected: p <- norm(max(p - q, 0)), q(x) <- 0, q <- norm(q)
          beta += Z / rem;
          sumq += qx;
          rej_w[j] = fmax(px - beta * qx, 0.0);  // (every lane of the wave stores the same value; LDS keeps a wave's order)
          if (j > 0) {
            int b_lo;
            near_buckets(beta, b_lo, b_hi);
            if (tid == 0) {
              step.beta = beta;
              step.b_lo = b_lo;
              step.b_hi = b_hi;
            }
          }
        }
      }
      if (j > 0) {  // (beta = 1 at the first rejection: every sorted token is live)
        if (tid == 0) step.stop = acc >= 0 ? 1 : 0;
        __syncthreads();
        if (step.stop != 0) break;
        near_terms(pairs, tables, step);
        __syncthreads();
      }
      if (lead) {
        double F;
        if (j == 0) {
          F = (double)(tables.sp[0] - tables.sq[0]) * FIX_UNIT;
        } else {
          const unsigned long long near = wave_total(lane < AC_WAVES ? step.part[lane] : 0ull);
          F = ((double)tables.sp[b_hi] - beta * (double)tables.sq[b_hi]) * FIX_UNIT + (double)near * 0x1p-52;
        }
        // a rejected token's weight is frozen: its live term leaves the sum
        double fix = 0.0;
        for (int i = lane; i <= j; i += 64) fix += rej_w[i] - fmax((double)kid_p[i] - beta * (double)kid_q[i], 0.0);
        Z = F + wave_sum_dpp(fix);
      }
    }
    if (!lead) return;
  } else {
    for (int j = 0; j < nk; ++j) {
      const double px = (double)kid_p[j];
      const double qx = (double)kid_q[j];
      if (j > 0 && ratio_accepts(fmax(px - beta * qx, 0.0) / Z, qx / (1.0 - sumq), kid_u[j])) {
        acc = j;
        break;
      }
      beta += Z / (1.0 - sumq);
      sumq += qx;
      if (tid == 0) rej_w[j] = fmax(px - beta * qx, 0.0);
      double F = residual_mass(p, q, beta, V, red);  // (its barriers also publish rej_w)
      // a rejected token's weight is frozen: its live term, as the pass formed it, leaves the sum
      const float bf = (float)beta;
      for (int i = 0; i <= j; ++i) F += rej_w[i] - (double)fmaxf(fmaf(-bf, kid_q[i], kid_p[i]), 0.f);
      Z = F;
    }
    if (tid >= 64) return;
  }
  // (the first wave, for which its own stores to LDS are in order; rej_w is tid 0's or the wave's own)
  if (acc < 0)
    for (int i = tid; i < nk; i += 64) out.child_frozen[o + kids_sorted[i]] = rej_w[i];
  if (tid == 0) {
    out.accepted[g] = acc >= 0 ? kids_sorted[acc] : -1;
    out.node_beta[g] = beta;
    out.node_Z[g] = Z;
  }
}

// Where a sequence's walk ends under the ratio rule: from its root from one accepted child to the next.  Called by all
// threads; `next` has room for the path's rows when they are wanted (NULL: not).
__device__ __forceinline__ int chase(const int32_t* __restrict__ accepted, int o, int n, int max_depth, int* l_acc, int* len, int32_t* path) {
  const bool staged = n <= GR_LDS_ROWS;
  if (staged)
    for (int i = threadIdx.x; i < n; i += blockDim.x) l_acc[i] = accepted[o + i];
  __syncthreads();
  int cur = 0, l = 0;
  for (int c; l < max_depth && (c = staged ? l_acc[cur] : accepted[o + cur]) >= 0; ++l) {
    if (path != nullptr && threadIdx.x == 0) path[l] = c;
    cur = c;
  }
  if (path != nullptr)
    for (int d = l + threadIdx.x; d < max_depth; d += blockDim.x) path[d] = -1;
  *len = l;
  return cur;
}

// Draws a sequence's bonus token: the first one at which the running sum of the weights passes `goal`.  rowsum: the weights'
// sums over rows of 64 tokens, all tokens taken as live (LDS); rej_tok, rej_w: the n_rej rejected tokens and their frozen weights.  Called
// by all threads, after a barrier.
template <int THREADS>
__device__ __forceinline__ void draw_bonus(const RowView& p, const RowView& q, bool sub_q, double beta, double goal, int V, int n_rej,
                                           const int* rej_tok, const double* rej_w, double* rowsum, int s, int len,
                                           int32_t* __restrict__ accept_len, int32_t* __restrict__ bonus_token) {
  __shared__ double rej_fix[AC_MAX_KIDS];         // what a rejected token's frozen weight changes in its row sum
  __shared__ double chunk_tot[AC_MAX_ROWS / 64];  // sums of 64 rows
  __shared__ int chunk_last[AC_MAX_ROWS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_rows = (V + 63) / 64;
  // (every rejected token's correction by a thread of its own: one trip to memory for all of them)
  if (tid < n_rej) rej_fix[tid] = rej_w[tid] - token_weight(p, q, sub_q, beta, rej_tok[tid]);
  __syncthreads();
  if (tid == 0)
    for (int i = 0; i < n_rej; ++i) rowsum[rej_tok[i] >> 6] += rej_fix[i];
  __syncthreads();
  // two levels: the waves sum chunks of 64 rows side by side, one wave then looks for the
  // chunk, the row inside it and the token inside the row
  const int n_chunks = (n_rows + 63) >> 6;
  for (int c = wave; c < n_chunks; c += THREADS / 64) {
    const int r = c * 64 + lane;
    const double val = r < n_rows ? rowsum[r] : 0.0;
    const double tot = wave_sum_dpp(val);
    const unsigned long long pos = __ballot(r < n_rows && val > 0.0);
    if (lane == 0) {
      chunk_tot[c] = tot;
      chunk_last[c] = pos != 0ull ? c * 64 + 63 - __clzll((long long)pos) : -1;  // its last row with mass
    }
  }
  __syncthreads();
  if (wave == 0) {
    double carry = 0.0, chunk_excl = 0.0;
    int chunk = -1, last_pos = -1;
    for (int cb = 0; cb < n_chunks && chunk < 0; cb += 64) {
      const int c = cb + lane;
      const double val = c < n_chunks ? chunk_tot[c] : 0.0;
      const int lp = c < n_chunks ? chunk_last[c] : -1;
      const double incl = wave_incl_scan(val, lane) + carry;
      const unsigned long long hit = __ballot(c < n_chunks && incl > goal);
      if (hit != 0ull) {
        const int l = __ffsll((long long)hit) - 1;
        chunk = cb + l;
        chunk_excl = __shfl(incl - val, l);
      } else {
        const unsigned long long pos = __ballot(lp >= 0);
        if (pos != 0ull) last_pos = __shfl(lp, 63 - __clzll((long long)pos));
        carry = __shfl(incl, 63);
      }
    }
    int row = -1;
    double excl = 0.0;
    if (chunk >= 0) {
      const int r = chunk * 64 + lane;
      const double val = r < n_rows ? rowsum[r] : 0.0;
      const double incl = wave_incl_scan(val, lane) + chunk_excl;
      const unsigned long long hit = __ballot(r < n_rows && incl > goal);
      if (hit != 0ull) {
        const int l = __ffsll((long long)hit) - 1;
        row = chunk * 64 + l;
        excl = __shfl(incl - val, l);
      } else {
        last_pos = chunk_last[chunk];  // (the two orders of summation differ by a rounding: the chunk's last row with mass)
      }
    }
    double row_goal = goal - excl;
    if (row < 0) {  // rounding left the goal at or above the total: take the last token with mass
      row = last_pos < 0 ? 0 : last_pos;
      row_goal = HS_INF;
    }
    const int v = row * 64 + lane;
    double w = v < V ? token_weight(p, q, sub_q, beta, v) : 0.0;
    for (int i = 0; i < n_rej; ++i)
      if (rej_tok[i] == v) w = rej_w[i];
    const double incl = wave_incl_scan(w, lane);
    const unsigned long long hit = __ballot(incl > row_goal);
    const unsigned long long pos = __ballot(w > 0.0);
    int l;
    if (hit != 0ull)
      l = __ffsll((long long)hit) - 1;
    else
      l = pos != 0ull ? 63 - __clzll((long long)pos) : 0;
    if (lane == 0) {
      accept_len[s] = len;
      int tok = row * 64 + l;
      bonus_token[s] = tok < V ? tok : V - 1;
    }
  }
}

// grid (B, slices), after the chains: every workgroup finds where its sequence's walk ends and sums its slice of that
// row; one compute unit alone would take 15 us for a row of the vocabulary.  The
// distribution is max(p - beta q, 0) with the chain's final beta where all children were rejected, p itself where none is
// tried; the rejected tokens' frozen weights are the draw's corrections.  The first slice's workgroup writes the path, and the one that
// draws the last ticket of its sequence (a counter of the scan's, zero before and cleared by each call's k_tree_rows) draws the bonus token.
// ROWS: rows of 64 tokens that LDS has room for.  (The draw by a launch of its own: 4.9 and 6.1 us for 61 rows
// of 128256 tokens, 8.4 in one now; the whole step 151.1 us, now 149.1, on 32000 tokens 133.7 and 131.0.)
template <int ROWS>
__global__ __launch_bounds__(BR_THREADS) void k_bonus_rows(const float* __restrict__ target,
                                                           const float* __restrict__ draft, int64_t row_stride,
                                                           const int32_t* __restrict__ token,
                                                           const int32_t* __restrict__ parent,
                                                           const int32_t* __restrict__ node_offsets, int NN, int V,
                                                           float inv_t, const float* __restrict__ uniforms, int max_depth,
                                                           int slices, const int32_t* __restrict__ t_arg,
                                                           const float* __restrict__ t_lz,
                                                           const int32_t* __restrict__ d_arg,
                                                           const float* __restrict__ d_lz, ChainOut chain,
                                                           unsigned* __restrict__ tickets, int32_t* __restrict__ accept_len,
                                                           int32_t* __restrict__ accept_path, int32_t* __restrict__ bonus_token) {
  __shared__ double rowsum[ROWS];
  __shared__ int l_acc[GR_LDS_ROWS];
  __shared__ int kids[AC_MAX_KIDS];
  __shared__ int kids_sorted[AC_MAX_KIDS];
  __shared__ int n_kids, is_last;
  __shared__ int rej_tok[AC_MAX_KIDS];
  __shared__ double rej_w[AC_MAX_KIDS];
  const int s = blockIdx.x, slice = blockIdx.y, tid = threadIdx.x;
  const int o = node_offsets[s];
  const int n = node_offsets[s + 1] - o;
  int32_t* const path = accept_path + (int64_t)s * max_depth;
  if (n <= 0) {
    if (slice == 0) {
      for (int d = tid; d < max_depth; d += BR_THREADS) path[d] = -1;
      if (tid == 0) {
        accept_len[s] = 0;
        bonus_token[s] = -1;
      }
    }
    return;
  }
  int len;
  const int cur = chase(chain.accepted, o, n, max_depth, l_acc, &len, slice == 0 ? path : nullptr);
  const int n_rows = (V + 63) / 64;
  const int per = (n_rows + slices - 1) / slices;
  const int r_begin = slice * per, r_end = min(n_rows, r_begin + per);
  if (r_begin >= r_end) return;
  const int g = o + cur;
  const bool sub_q = chain.n_tried[g] > 0;
  const float* p_row = target + (int64_t)g * row_stride;
  const RowView p(p_row, p_row[t_arg[g]], t_lz[g], inv_t);
  RowView q = p;
  double beta = 0.0, Z = 1.0;
  if (sub_q) {
    const float* q_row = draft + (int64_t)g * row_stride;
    q = RowView(q_row, q_row[d_arg[g]], d_lz[g], inv_t);
    beta = chain.node_beta[g];
    Z = chain.node_Z[g];
  }
  double* const sums = chain.bonus_rows + (int64_t)g * n_rows;
  bonus_row_sums<true>(p, q, sub_q, beta, V, r_begin, r_end, sums);
  // (what the draw needs besides is looked up while the sums are on their way)
  const double goal = (double)uniforms[NN + s] * Z;
  const int n_rej = gather_children<BR_THREADS>(parent, o, n, cur, len < max_depth, kids, kids_sorted, &n_kids);
  if (tid < n_rej) {
    const int c = o + kids_sorted[tid];
    rej_tok[tid] = token[c];
    rej_w[tid] = chain.child_frozen[c];
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0)
    is_last = __hip_atomic_fetch_add(&tickets[o], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)((n_rows + per - 1) / per - 1) ? 1 : 0;
  __syncthreads();
  if (!is_last) return;
  constexpr int PER = 4;  // sums of a thread that are requested together
  for (int r0 = tid; r0 < n_rows; r0 += PER * BR_THREADS) {
    unsigned long long v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) v[k] = ld_dev(reinterpret_cast<const unsigned long long*>(sums) + min(r0 + k * BR_THREADS, n_rows - 1));
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (r0 + k * BR_THREADS < n_rows) rowsum[r0 + k * BR_THREADS] = __builtin_bit_cast(double, v[k]);
  }
  draw_bonus<BR_THREADS>(p, q, sub_q && n_rej > 0, beta, goal, V, n_rej, rej_tok, rej_w, rowsum, s, len, accept_len, bonus_token);
}

// The walk of the point-mass rule, and the end of the ratio rule's for trees beyond BK_NODES rows.
__global__ __launch_bounds__(AC_THREADS) void k_accept_walk(
    const float* __restrict__ target, const float* __restrict__ draft, int64_t row_stride,
    const int32_t* __restrict__ token, const int32_t* __restrict__ parent, const int32_t* __restrict__ node_offsets,
    int NN, int V, int mode, float inv_t, const float* __restrict__ uniforms, int max_depth,
    const int32_t* __restrict__ t_arg, const float* __restrict__ t_lz, const int32_t* __restrict__ d_arg,
    const float* __restrict__ d_lz, ChainOut chain, int32_t* __restrict__ accept_len,
    int32_t* __restrict__ accept_path, int32_t* __restrict__ bonus_token) {
  // Every wave reads these while it tries a level's children, at its own pace: they are written between the
  // barriers ahead of that loop only.  A next level's writes come behind the barriers of gather_children, and
  // what is made after the loop, the corrections of a bonus draw, has an array of its own.
  __shared__ int kids[AC_MAX_KIDS];
  __shared__ int kids_sorted[AC_MAX_KIDS];
  __shared__ int n_kids;
  __shared__ int rej_tok[AC_MAX_KIDS];
  __shared__ double rej_w[AC_MAX_KIDS];  // frozen weight of each rejected token
  __shared__ float kid_u[AC_MAX_KIDS];    // the child's uniform
  __shared__ double kid_p[AC_MAX_KIDS];   // its p(x)
  __shared__ double rowsum[AC_MAX_ROWS];

  const int s = blockIdx.x, tid = threadIdx.x;
  const int o = node_offsets[s];
  const int n = node_offsets[s + 1] - o;
  int32_t* path = accept_path + (int64_t)s * max_depth;
  const bool ratio_mode = mode == HS_ACCEPT_STOCHASTIC;
  if (n <= 0 || !ratio_mode)
    for (int d = tid; d < max_depth; d += AC_THREADS) path[d] = -1;
  if (n <= 0) {
    if (tid == 0) {
      accept_len[s] = 0;
      bonus_token[s] = -1;
    }
    return;
  }
  // Under the ratio rule the chains have left every node's accepted child: the walk is a chase through them.
  // (Level by level, each a few trips to memory, 12.6 us for a 61-row tree and 22 for 97 rows.)
  int cur = 0, len = 0;
  const int n_rows = (V + 63) / 64;
  if (ratio_mode) {
    __shared__ int l_acc[GR_LDS_ROWS];
    cur = chase(chain.accepted, o, n, max_depth, l_acc, &len, path);
  }
  for (;;) {
    const int nk = gather_children<AC_THREADS>(parent, o, n, cur, len < max_depth, kids, kids_sorted, &n_kids);

    const float* p_row = target + (int64_t)(o + cur) * row_stride;
    const RowView p(p_row, p_row[t_arg[o + cur]], t_lz[o + cur], inv_t);
    RowView q = p;
    const bool use_q = ratio_mode && nk > 0;
    if (use_q) {
      const float* q_row = draft + (int64_t)(o + cur) * row_stride;
      q = RowView(q_row, q_row[d_arg[o + cur]], d_lz[o + cur], inv_t);
    }

    // ---- what the tests of the children need, fetched side by side (a round trip to memory per
    // child would dominate the walk).  The rejected children are a prefix of the list, so entry i of
    // rej_tok / rej_w belongs to child i.
    if (tid < nk) {
      const int c = kids_sorted[tid];
      const int x = token[o + c];
      rej_tok[tid] = x;
      if (ratio_mode) {  // (all of them were rejected: k_accept_chain)
        rej_w[tid] = chain.child_frozen[o + c];
      } else {
        kid_u[tid] = uniforms[o + c];
        kid_p[tid] = (double)p.prob(x);
        rej_w[tid] = 0.0;
      }
    }
    __syncthreads();
    // ---- point-mass rule: try the children in order (every thread runs the same scalar logic)
    double beta = 0.0, Z = 1.0, rem = 1.0;
    int n_rej = 0, accepted = -1;
    if (ratio_mode) {
      n_rej = nk;
      if (nk > 0) {
        beta = chain.node_beta[o + cur];
        Z = chain.node_Z[o + cur];
      }
    } else {
      for (; n_rej < nk; ++n_rej) {
        const double px = kid_p[n_rej];
        if ((double)kid_u[n_rej] * rem < px) {  // u < p(x) / rem
          accepted = kids_sorted[n_rej];
          break;
        }
        rem -= px;
      }
    }
    if (accepted >= 0) {
      if (tid == 0) path[len] = accepted;
      ++len;
      cur = accepted;
      continue;
    }

    // ---- no child accepted: draw the bonus token from the current distribution
    const bool sub_q = use_q && n_rej > 0;
    const double total = ratio_mode ? Z : rem;
    const double goal = (double)uniforms[NN + s] * total;
    bonus_row_sums<false>(p, q, sub_q, beta, V, 0, n_rows, rowsum);
    draw_bonus<AC_THREADS>(p, q, sub_q, beta, goal, V, n_rej, rej_tok, rej_w, rowsum, s, len, accept_len, bonus_token);
    return;
  }
}

// Bytes of the sorted residual's arrays for NN rows (0 beyond BK_NODES rows); with a carver, also
// takes them.
static size_t bucket_workspace(int NN, int V, Carver* c, BucketWs* ws) {
  if (NN > BK_NODES) return 0;
  const size_t n_sb = (size_t)NN * BK_SLICES * BK_N, n_st = (size_t)NN * BK_SLICES * (BK_N + 1);
  if (c != nullptr) {
    ws->start = c->take<uint32_t>(n_st);
    ws->psum = c->take<unsigned long long>(n_sb);
    ws->qsum = c->take<unsigned long long>(n_sb);
    ws->pairs = c->take<float2>((size_t)NN * V);
  }
  return align_up(n_st * 4, 256) + 2 * align_up(n_sb * 8, 256) + align_up((size_t)NN * V * sizeof(float2), 256);
}

// Bytes of the row sums of k_bonus_rows, which has a place for every tree row and uses one a sequence (0 beyond BK_NODES rows: the walk then sums
// the rows of its stop node itself).
static size_t bonus_rows_bytes(int NN, int V) {
  return NN <= BK_NODES ? align_up((size_t)NN * ((V + 63) / 64) * sizeof(double), 256) : 0;
}

// Bytes of a call besides the scan's workspace, which comes last.
static size_t accept_arrays_bytes(int NN, int V, bool ratio) {
  // per row: argmax, -ln Z and an unused Top-1 entropy, for the target and for the draft rows (the
  // two sets back to back: the ratio rule scans [target rows ; draft rows] in one launch)
  const size_t sets = 3 * align_up((size_t)2 * NN * sizeof(float), 256);
  // five doubles per row: what the rejection chains hand to the walk; two bytes per row: rows to scan
  const size_t chain = 5 * align_up((size_t)NN * sizeof(double), 256) + align_up((size_t)2 * NN, 256);
  // the sorted residual belongs to the ratio rule alone, and so do the children counts and the bonus
  // distribution's row sums of every tree row
  const size_t sorted = ratio ? bucket_workspace(NN, V, nullptr, nullptr) + align_up((size_t)NN * sizeof(int32_t), 256) + bonus_rows_bytes(NN, V) : 0;
  return sets + chain + sorted;
}

}  // namespace hs

extern "C" size_t hs_verify_accept_workspace_mode(int32_t B, int32_t NN, int32_t V, hs_accept_mode mode) {
  if (B <= 0 || NN <= 0 || V <= 0) return 0;
  const bool ratio = mode == HS_ACCEPT_STOCHASTIC;  // (it scans twice the rows)
  return hs::accept_arrays_bytes(NN, V, ratio) + hs::row_topk_workspace(ratio ? 2 * NN : NN, V, 1, ratio);
}

extern "C" size_t hs_verify_accept_workspace(int32_t B, int32_t NN, int32_t V) {
  return hs_verify_accept_workspace_mode(B, NN, V, HS_ACCEPT_STOCHASTIC);  // the largest of the three
}

extern "C" hs_status hs_verify_accept(const float* target_logits, const float* draft_logits, int64_t row_stride,
                                      const int32_t* token, const int32_t* parent, const int32_t* node_offsets,
                                      int32_t B, int32_t NN, int32_t V, hs_accept_mode mode, float temperature,
                                      const float* uniforms, int32_t max_depth, int32_t* accept_len,
                                      int32_t* accept_path, int32_t* bonus_token, void* workspace,
                                      size_t workspace_bytes, hs_stream stream) {
  hs::clear_error();
  HS_REQUIRE(B >= 0 && NN >= 0 && V >= 1, HS_ERR_SHAPE, "hs_verify_accept: B=%d NN=%d V=%d", B, NN, V);
  HS_REQUIRE(max_depth >= 1, HS_ERR_SHAPE, "hs_verify_accept: max_depth=%d must be at least 1", max_depth);
  HS_REQUIRE(row_stride >= V, HS_ERR_SHAPE, "hs_verify_accept: row_stride=%lld < V=%d", (long long)row_stride, V);
  HS_REQUIRE(mode == HS_ACCEPT_GREEDY || mode == HS_ACCEPT_STOCHASTIC || mode == HS_ACCEPT_STOCHASTIC_POINTMASS,
             HS_ERR_SHAPE, "hs_verify_accept: unknown mode %d", (int)mode);
  if (B == 0) return HS_OK;
  HS_REQUIRE(node_offsets && accept_len && accept_path && bonus_token, HS_ERR_NULL, "hs_verify_accept: NULL argument");
  const bool stochastic = mode != HS_ACCEPT_GREEDY;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (NN > 0) {
    HS_REQUIRE(target_logits && token && parent, HS_ERR_NULL, "hs_verify_accept: NULL node array");
    if (stochastic) {
      HS_REQUIRE(uniforms, HS_ERR_NULL, "hs_verify_accept: uniforms are required in the stochastic modes");
      HS_REQUIRE(mode != HS_ACCEPT_STOCHASTIC || draft_logits, HS_ERR_NULL,
                 "hs_verify_accept: draft_logits are required in mode HS_ACCEPT_STOCHASTIC");
      HS_REQUIRE(temperature > 0.f, HS_ERR_SHAPE, "hs_verify_accept: temperature must be positive");
      HS_REQUIRE((V + 63) / 64 <= hs::AC_MAX_ROWS, HS_ERR_UNSUPPORTED,
                 "hs_verify_accept: stochastic modes support V <= %d", hs::AC_MAX_ROWS * 64);
    }
  }
  // (what this call's scan needs; the query gives what any call of up to NN rows can need)
  const bool ratio = mode == HS_ACCEPT_STOCHASTIC;
  const hs::ScanRows rows{hs::scan_aligned(target_logits, ratio ? draft_logits : nullptr, row_stride), ratio, !stochastic};
  const size_t need = NN > 0 ? hs::accept_arrays_bytes(NN, V, ratio) + hs::row_topk_need(ratio ? 2 * NN : NN, V, 1, rows) : 0;
  HS_REQUIRE(need == 0 || (workspace && workspace_bytes >= need && reinterpret_cast<uintptr_t>(workspace) % 256 == 0),
             HS_ERR_WORKSPACE, "hs_verify_accept: workspace needs %zu bytes, 256-byte aligned (got %zu)", need,
             workspace_bytes);
  // (for every call, whichever way it takes, and before anything is launched)
  const int64_t scanned = ratio ? 2 * (int64_t)NN : NN;
  HS_REQUIRE(scanned <= hs::ROW_SCAN_MAX, HS_ERR_UNSUPPORTED, "hs_verify_accept: NN=%d, %lld rows to scan in one call (at most %d)",
             NN, (long long)scanned, hs::ROW_SCAN_MAX);
  int32_t *t_arg = nullptr, *d_arg = nullptr;
  float *t_lz = nullptr, *d_lz = nullptr;
  hs::ScanSlices slices{nullptr, 1};
  slices.pairs_only = true;  // (the greedy walk needs the rows' argmax and nothing else)
  hs::ChainOut chain{};
  hs::BucketWs bk{};  // (all NULL: no sorted residual)
  unsigned* tickets = nullptr;  // the scan's counters
  if (NN > 0) {
    hs::Carver c(workspace);
    t_arg = c.take<int32_t>(2 * (size_t)NN);
    t_lz = c.take<float>(2 * (size_t)NN);
    float* t_ent = c.take<float>(2 * (size_t)NN);
    d_arg = t_arg + NN;  // (the draft rows' results follow the target rows')
    d_lz = t_lz + NN;
    chain.first = c.take<int32_t>(2 * (size_t)NN);
    chain.kid_tok = chain.first + NN;
    chain.kid_u = c.take<float>(2 * (size_t)NN);
    chain.accepted = reinterpret_cast<int32_t*>(chain.kid_u + NN);
    chain.child_frozen = c.take<double>(NN);
    chain.node_beta = c.take<double>(NN);
    chain.node_Z = c.take<double>(NN);
    uint8_t* wanted = c.take<uint8_t>(2 * (size_t)NN);
    if (mode == HS_ACCEPT_STOCHASTIC) {
      hs::bucket_workspace(NN, V, &c, &bk);
      chain.n_tried = c.take<int32_t>(NN);
      if (hs::bonus_rows_bytes(NN, V) > 0) chain.bonus_rows = c.take<double>((size_t)NN * ((V + 63) / 64));
    }
    void* scan_ws = c.take<char>(0);
    tickets = static_cast<unsigned*>(scan_ws);
    const float T = stochastic ? temperature : 1.0f;
    hs_status r;
    if (!stochastic && hs::greedy_by_path(B, NN, V, max_depth)) {
      int32_t* list = reinterpret_cast<int32_t*>(t_lz);  // (2 NN words that the scan would fill)
      hipLaunchKernelGGL(hs::k_greedy_path, dim3(B), dim3(hs::GP_THREADS), 0, st, target_logits, row_stride, V, NN, token, parent,
                         node_offsets, max_depth, t_arg, list, accept_len, accept_path, bonus_token);
      return hs::launch_status("accept (greedy path)");
    }
    if (mode == HS_ACCEPT_STOCHASTIC) {
      // one scan over [target rows ; draft rows]; draft rows are read where a row has children, and
      // nowhere else
      hipLaunchKernelGGL(hs::k_tree_rows, dim3(B), dim3(hs::GR_THREADS), 0, st, parent, node_offsets, token, uniforms, NN,
                         max_depth, wanted, chain, tickets);
      r = hs::launch_status("accept (tree rows)");
      if (r != HS_OK) return r;
      // (the rows' counters are clear: the scan merges its slices itself)
      r = hs::row_topk_launch(target_logits, row_stride, 2 * NN, V, 1, T, t_arg, t_lz, t_ent, nullptr, nullptr,
                              scan_ws, st, nullptr, wanted, nullptr, draft_logits, NN, true);
    } else {
      // greedy: the merge of the row slices is done by the accept kernel (one launch less)
      r = hs::row_topk_launch(target_logits, row_stride, NN, V, 1, T, t_arg, t_lz, t_ent, nullptr, nullptr, scan_ws,
                              st, stochastic ? nullptr : &slices);
    }
    if (r != HS_OK) return r;
  }
  if (!stochastic) {
    hipLaunchKernelGGL(hs::k_accept_greedy, dim3(B), dim3(hs::GR_THREADS), 0, st, t_arg, slices.key,
                       slices.count, token, parent, node_offsets, max_depth, accept_len, accept_path, bonus_token);
    return hs::launch_status("accept (greedy)");
  }
  if (mode == HS_ACCEPT_STOCHASTIC && NN > 0) {
    // the sorted residual pays from a few thousand tokens on
    const bool sorted = bk.pairs != nullptr && V >= 4096;  // (its rows need no alignment: load_float4)
    if (sorted) {
      hipLaunchKernelGGL(hs::k_bucket_sort, dim3(hs::BK_SLICES, NN), dim3(hs::BK_THREADS), 0, st, target_logits, draft_logits,
                         row_stride, V, 1.0f / temperature, chain, t_arg, t_lz, d_arg, d_lz, bk);
      hs_status r = hs::launch_status("accept (sorted residual)");
      if (r != HS_OK) return r;
    } else {
      bk.pairs = nullptr;
    }
    hipLaunchKernelGGL(hs::k_accept_chain, dim3(NN), dim3(hs::AC_THREADS), 0, st, target_logits, draft_logits,
                       row_stride, token, parent, node_offsets, B, V, 1.0f / temperature, uniforms, t_arg, t_lz, d_arg,
                       d_lz, chain, bk);
    hs_status r = hs::launch_status("accept (rejection chains)");
    if (r != HS_OK) return r;
    if (chain.bonus_rows != nullptr) {
      // (no fewer rows to a workgroup than its waves take in a trip: more would only queue for the counters, which of short trees share a
      // cache line.  Trees of the root alone, 64 workgroups each and so: 16 of 32000 tokens 32.4 us, now 23.9, 8 of 8000 22.1 and 17.0; one of 61 rows 34.7 and 34.6)
      const int trips = ((V + 63) / 64 + hs::BR_TRIP_ROWS - 1) / hs::BR_TRIP_ROWS;
      const unsigned slices = (unsigned)std::max(1, std::min({hs::BR_SLICES, hs::BR_WGS / B, trips}));
#define BR_LAUNCH(ROWS)                                                                                                    \
  hipLaunchKernelGGL(hs::k_bonus_rows<ROWS>, dim3(B, slices), dim3(hs::BR_THREADS), 0, st, target_logits, draft_logits, row_stride, \
                     token, parent, node_offsets, NN, V, 1.0f / temperature, uniforms, max_depth, (int)slices, t_arg, t_lz,  \
                     d_arg, d_lz, chain, tickets, accept_len, accept_path, bonus_token)
      // (16 KB of sums leave room for four workgroups to a compute unit, 64 KB for two)
      if ((V + 63) / 64 <= hs::BR_FEW_ROWS) BR_LAUNCH(hs::BR_FEW_ROWS);
      else BR_LAUNCH(hs::AC_MAX_ROWS);
#undef BR_LAUNCH
      return hs::launch_status("accept (bonus rows)");
    }
  }
  hipLaunchKernelGGL(hs::k_accept_walk, dim3(B), dim3(hs::AC_THREADS), 0, st, target_logits, draft_logits, row_stride,
                     token, parent, node_offsets, NN, V, (int)mode, 1.0f / temperature, uniforms, max_depth, t_arg,
                     t_lz, d_arg, d_lz, chain, accept_len, accept_path, bonus_token);
  return hs::launch_status("accept (stochastic)");
}
