// hs_tree_attention: tree-masked attention of the kept tree rows over the prefix KV cache
// (Section 2.2: the pruned tree is verified in one pass with tree-mask attention).
//
// This file holds the entry point, the launch planning, the float32 / any-shape kernel
// (k_attn_generic: float32 matrix instructions, 16 rows per workgroup, keys shared out to its waves)
// and the split combine (k_attn_combine).  bfloat16 with head dimension 128, or 64 and an even number of
// KV heads, goes to the kernel in tree_attention_mfma.hip (16-byte aligned tensors, G * rows < 65536).
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <vector>

#include "attn_common.h"

namespace hs {

hs_status attn_mfma_launch(const AttnArgs& a, int max_tree_rows, hipStream_t stream, hipEvent_t ev_start,
                           hipEvent_t ev_stop);
bool attn_mfma_supported(int D, hs_dtype dt, int max_tree_rows, float scale);
size_t attn_mfma_table_bytes(int max_tree_rows, int64_t NN);

constexpr int GEN_THREADS = 512;
constexpr int GEN_WAVES = GEN_THREADS / 64;
constexpr int GEN_ROWS = 16;  // rows per workgroup
constexpr int gen_groups(int D) { return D == 64 ? 2 : 1; }  // key groups of a wave's trip
// Whether a split of so many keys and a tree of max_M rows are one trip of the workgroup's waves at most.
static inline bool generic_short(int64_t keys, int max_M, int D) {
  return (keys + 15) / 16 + (max_M + 15) / 16 <= GEN_WAVES * gen_groups(D);
}
constexpr int GEN_TILE = 64;  // tokens of a page
constexpr int MAX_TREE_ROWS = 1024;

// ---- float32, and every bfloat16 call that the matrix-core kernel of the other file does not take.
//
// One workgroup = 16 query rows of one (sequence, KV head, key split); its eight waves share out the
// split's keys in groups of 16 (GPI groups to a wave and trip) and their partial softmaxes meet in LDS at
// the end.  What bounds these calls is latency: there are few rows, so a workgroup's own chain of trips
// counts, and keys are spread over waves before they are spread over workgroups, which would need the
// combine launch.  Both products run on the float32 matrix instruction (v_mfma_f32_16x16x4_f32: full
// float32 multiply-adds), transposed so that a lane holds scores of one row:
//     S^T[key, row] = K[key, :] . Q[row, :]      A = K, B = Q: lane (i = l % 16, h = l / 16) holds row i,
//                                                elements 4 (4 c + h) + e of step 4 c + e
//     O^T[d, row] += V^T[d, key] P^T[key, row]   B = P: score register v of lane (i, h) is key 4 h + v of
//                                                row i, which is the B operand of step v as it stands
// The contraction order is free, so K, Q and V go from global memory into operand registers 16 bytes at
// a time and nothing is staged in LDS; output column block b holds columns i * D / 16 + b.
// (One row group of four rows per wave on the vector ALUs, K and V staged through LDS, five LDS reads to
// four multiply-adds: three sequences of 100 to 1500 tokens, 8 heads of 64, 17 to 40 rows: 84 us a call, 23 then and 17 now;
// one of 16384 tokens, 32 heads of 128 on 8, 61 rows: 2048 us a call, now 210.)
// SHORT: no workgroup of the launch has more keys than one trip takes (generic_short), so that waves may have none.  These then
// request none; in longer launches the branch would cost the loop its register allocation.  (77 sequences of one row, 8 heads of
// 64, without a prefix: 11.0 us before the keys were requested ahead of the root paths, 13.4 with it, 11.2 now; 16 heads, 22
// tokens 21.0, 24.2, 20.5; 4 sequences of 250 tokens, 20 rows, 8 heads of 128: 15.2, 14.6, and 15.1 to 15.7 with the branch.)
template <typename T, int D, bool SHORT>
__global__ __launch_bounds__(GEN_THREADS) void k_attn_generic(AttnArgs a) {
  constexpr int NQ = D / 16;            // 16-byte (float32) pieces of a lane's part of a K, Q or V row group
  constexpr int GPI = gen_groups(D);
  constexpr int DPL = D / 16;           // output columns of a lane's row (and column blocks)
  constexpr int ANC_WORDS = MAX_TREE_ROWS / 32;
  __shared__ int par[MAX_TREE_ROWS];
  __shared__ unsigned anc[GEN_ROWS][ANC_WORDS + 1];
  __shared__ float o_part[GEN_WAVES][GEN_ROWS][D + 4];
  __shared__ float m_part[GEN_WAVES][GEN_ROWS], l_part[GEN_WAVES][GEN_ROWS];

  const int s = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = a.node_offsets[s];
  const int M = a.node_offsets[s + 1] - n0;
  const bool paged = a.block_table != nullptr;  // prefix tiles are pages of GEN_TILE tokens
  const int64_t p0 = paged ? 0 : a.prefix_offsets[s];
  const int64_t L = prefix_len_of(a, s);
  if (M <= 0) return;
  const int G = a.G, Hkv = a.Hkv, Hq = a.Hq;
  const int R = G * M;
  const int n_rb = (R + GEN_ROWS - 1) / GEN_ROWS;
  const int n_sp = splits_of(L, a.split_len);
  int x = blockIdx.x;
  const int g = x % Hkv;
  x /= Hkv;
  const int rb = x % a.n_rb_max;
  const int sp = x / a.n_rb_max;
  if (rb >= n_rb || sp >= n_sp) return;

  const T* q = static_cast<const T*>(a.q);
  const T* kp = static_cast<const T*>(a.k_prefix) + (p0 * Hkv + g) * D;
  const T* vp = static_cast<const T*>(a.v_prefix) + (p0 * Hkv + g) * D;
  const T* kt = static_cast<const T*>(a.k_tree) + ((int64_t)n0 * Hkv + g) * D;
  const T* vt = static_cast<const T*>(a.v_tree) + ((int64_t)n0 * Hkv + g) * D;
  const int64_t tok = (int64_t)Hkv * D;  // elements from one token's row of this head to the next one's

  const bool last_split = sp == n_sp - 1;
  const int64_t k_lo = (int64_t)sp * a.split_len;
  const int64_t k_hi = last_split ? L : k_lo + a.split_len;
  const int n_pg = (int)((k_hi - k_lo + 15) >> 4);      // groups of 16 prefix keys, the last one may be short
  const int n_groups = n_pg + (last_split ? (M + 15) >> 4 : 0);

  const int i16 = lane & 15, h = lane >> 4;
  const int r0 = rb * GEN_ROWS;
  const int r = r0 + i16 < R ? r0 + i16 : R - 1;        // this lane's row (rows past the end repeat the last one)
  const int node = r / G;
  const int64_t qrow = (int64_t)(n0 + node) * Hq + g * G + (r - node * G);

  // a key group's operands: K pieces (key i16) and V pieces (keys 4 h + v, columns i16 * DPL ...)
  struct Frag {
    float4 k[NQ], v[NQ];
  };
  auto load_group = [&](int grp, Frag& f) {
    const bool tree = grp >= n_pg;
    const int64_t first = tree ? (int64_t)(grp - n_pg) * 16 : k_lo + (int64_t)grp * 16;
    const int rows = (int)((tree ? (int64_t)M : k_hi) - first);  // >= 1; keys past the end repeat the last one
    // where the group's first key lives: in place, or in the page the block table names
    const int64_t where = (!tree && paged) ? (int64_t)a.block_table[(int64_t)s * a.max_blocks + first / GEN_TILE] * GEN_TILE + first % GEN_TILE
                                           : first;
    const T* kb = (tree ? kt : kp) + where * tok;
    const T* vb = (tree ? vt : vp) + where * tok;
    const T* krow = kb + (i16 < rows ? i16 : rows - 1) * tok + 4 * h;
#pragma unroll
    for (int c = 0; c < NQ; ++c) f.k[c] = load4<T>(krow + 16 * c);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int key = 4 * h + v;
      const T* vrow = vb + (key < rows ? key : rows - 1) * tok + i16 * DPL;
#pragma unroll
      for (int c = 0; c < DPL / 4; ++c) f.v[v * (DPL / 4) + c] = load4<T>(vrow + 4 * c);
    }
  };

  // The parent pointers are requested first, and nothing behind them depends on a condition, so that the wait for them
  // counts the younger loads: the root paths are found while the first keys are on their way.
  constexpr int PAR_PER = MAX_TREE_ROWS / GEN_THREADS;
  int my_par[PAR_PER];
  const int32_t* parent = a.parent + (a.tree_shared ? 0 : n0);
#pragma unroll
  for (int k = 0; k < PAR_PER; ++k) my_par[k] = parent[min(tid + k * GEN_THREADS, M - 1)];
  asm volatile("" ::: "memory");  // (keeps the requests in this order)

  // ---- the rows' root paths as bit sets over the tree rows
  auto root_paths = [&]() {
    if (!last_split) return;
#pragma unroll
    for (int k = 0; k < PAR_PER; ++k)
      if (tid + k * GEN_THREADS < M) par[tid + k * GEN_THREADS] = my_par[k];
    for (int e = tid; e < GEN_ROWS * (ANC_WORDS + 1); e += GEN_THREADS) (&anc[0][0])[e] = 0u;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // (through LDS only: the keys stay on their way)
    if (tid < GEN_ROWS) {  // (lane tid of the first wave: its own row; nobody waits for the ORs)
      for (int j = node; j >= 0;) {
        atomicOr(&anc[tid][j >> 5], 1u << (j & 31));
        const int up = par[j];
        j = up < j ? up : -1;  // (a malformed tree cannot keep the walk from ending)
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  Frag cur[GPI], nxt[GPI];
  float4 qf[NQ];
  const int stride = GEN_WAVES * GPI;
  int grp = wave * GPI;
  if (!SHORT || grp < n_groups) {
#pragma unroll
    for (int u = 0; u < GPI; ++u) load_group(min(grp + u, n_groups - 1), cur[u]);
#pragma unroll
    for (int c = 0; c < NQ; ++c) qf[c] = load4<T>(q + qrow * D + 16 * c + 4 * h);
    root_paths();
  } else {  // (a wave without keys requests none; it meets the same barriers)
    root_paths();
  }

  floatx4 acc[DPL];
  float m_run = -HS_INF, l_run = 0.f;  // m_run: of the row (all four lanes of it); l_run: of this lane's keys
#pragma unroll
  for (int b = 0; b < DPL; ++b) acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};

  for (; grp < n_groups; grp += stride) {
#pragma unroll
    for (int u = 0; u < GPI; ++u)
      if (grp + stride + u < n_groups) load_group(grp + stride + u, nxt[u]);

    floatx4 S[GPI];
    float mx = -HS_INF;
#pragma unroll
    for (int u = 0; u < GPI; ++u) {
      if (GPI > 1 && grp + u >= n_groups) {
        S[u] = floatx4{-HS_INF, -HS_INF, -HS_INF, -HS_INF};
        continue;
      }
      // (two chains: consecutive instructions of one accumulator wait for each other)
      floatx4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
      for (int c = 0; c < NQ; ++c) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[u].k[c].x, qf[c].x, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[u].k[c].y, qf[c].y, s1, 0, 0, 0);
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[u].k[c].z, qf[c].z, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[u].k[c].w, qf[c].w, s1, 0, 0, 0);
      }
      const bool tree = grp + u >= n_pg;
      const int64_t first = tree ? (int64_t)(grp + u - n_pg) * 16 : k_lo + (int64_t)(grp + u) * 16;
      // bit v: key 4 h + v of the group counts for this lane's row
      unsigned ok = 0xfu;
      if (tree) ok = anc[i16][(int)first >> 5] >> (((int)first & 31) + 4 * h);  // (bits past the tree are zero)
      else if (first + 16 > k_hi) {
        const int left = (int)(k_hi - first) - 4 * h;
        ok = left >= 4 ? 0xfu : left > 0 ? (1u << left) - 1u : 0u;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        S[u][v] = ((ok >> v) & 1u) ? (s0[v] + s1[v]) * a.scale : -HS_INF;
        mx = fmaxf(mx, S[u][v]);
      }
    }
    // the row's maximum moves only when a score of this trip lies above it
    if (__ballot(mx > m_run) != 0ull) {
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mx);
      const float alpha = m_new == -HS_INF ? 1.f : __expf(m_run - m_new);  // 0 when nothing was seen before
      l_run *= alpha;
#pragma unroll
      for (int b = 0; b < DPL; ++b) acc[b] *= alpha;
      m_run = m_new;
    }
#pragma unroll
    for (int u = 0; u < GPI; ++u) {
      if (GPI > 1 && grp + u >= n_groups) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float p = S[u][v] == -HS_INF ? 0.f : __expf(S[u][v] - m_run);
        l_run += p;
#pragma unroll
        for (int c = 0; c < DPL / 4; ++c) {
          const float4 vv = cur[u].v[v * (DPL / 4) + c];
          acc[4 * c + 0] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv.x, p, acc[4 * c + 0], 0, 0, 0);
          acc[4 * c + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv.y, p, acc[4 * c + 1], 0, 0, 0);
          acc[4 * c + 2] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv.z, p, acc[4 * c + 2], 0, 0, 0);
          acc[4 * c + 3] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv.w, p, acc[4 * c + 3], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < GPI; ++u) cur[u] = nxt[u];
  }

  // ---- the waves' parts meet: register b of value vv is column (4 h + vv) * DPL + b of row i16
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (h == 0) {
    m_part[wave][i16] = m_run;
    l_part[wave][i16] = l_run;
  }
#pragma unroll
  for (int vv = 0; vv < 4; ++vv)
#pragma unroll
    for (int c = 0; c < DPL / 4; ++c)
      *reinterpret_cast<float4*>(&o_part[wave][i16][(4 * h + vv) * DPL + 4 * c]) =
          make_float4(acc[4 * c][vv], acc[4 * c + 1][vv], acc[4 * c + 2][vv], acc[4 * c + 3][vv]);
  __syncthreads();
  constexpr int PIECES = GEN_ROWS * D / 4;  // four columns to a thread
  for (int e = tid; e < PIECES; e += GEN_THREADS) {
    const int rr = e / (D / 4), d = (e - rr * (D / 4)) * 4;
    if (r0 + rr >= R) continue;
    float m = m_part[0][rr];
#pragma unroll
    for (int w = 1; w < GEN_WAVES; ++w) m = fmaxf(m, m_part[w][rr]);
    float l = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < GEN_WAVES; ++w) {
      const float mw = m_part[w][rr];
      const float f = mw == -HS_INF ? 0.f : __expf(mw - m);  // (a wave without a visible key: weight 0)
      const float4 ow = *reinterpret_cast<const float4*>(&o_part[w][rr][d]);
      l = fmaf(l_part[w][rr], f, l);
      o.x = fmaf(ow.x, f, o.x);
      o.y = fmaf(ow.y, f, o.y);
      o.z = fmaf(ow.z, f, o.z);
      o.w = fmaf(ow.w, f, o.w);
    }
    // the result (sequences with one split) or this split's partial record
    const int i = (r0 + rr) / G, gi = r0 + rr - i * G;
    const int64_t row = (int64_t)(n0 + i) * Hq + g * G + gi;
    if (n_sp == 1) {
      const float inv = 1.f / l;
      store4<T>(static_cast<T*>(a.o) + row * D + d, make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv));
      if (a.lse && d == 0) a.lse[row] = m + __logf(l);
    } else {
      float* rec = a.part + (row * a.sp_max + sp) * (D + ATTN_REC_PAD);
      *reinterpret_cast<float4*>(rec + d) = o;
      if (d == 0) {
        rec[D] = m;
        rec[D + 1] = l;
      }
    }
  }
}

// Merges the splits of a (node, head) row: weights exp(m_sp - max m), splits taken in rising order, eight at a time.
// D / 4 lanes to a row, four output elements each.  A workgroup has rows of one node, whose split count is a scalar,
// and of every CMB_UNITS-th KV head: workgroup x of a launch runs on XCD x % 8, so with a multiple of eight KV heads it
// merges records that its own XCD has written (all heads of a node spread over the XCDs: 4.2 us a launch became 6.3).
// The launch is a chain of trips to memory: the arguments, the table (a single entry's count is an argument), then
// everything of eight splits at once.
constexpr int CMB_UNITS = 8;
constexpr int CMB_THREADS = 256;  // at most
template <typename T, int D>
__global__ __launch_bounds__(CMB_THREADS) void k_attn_combine(AttnArgs a) {
  constexpr int LPR = D / 4;  // lanes of a row
  constexpr int REC = D + ATTN_REC_PAD;
  constexpr int AT_ONCE = 8;
  const int lane = threadIdx.x & 63;
  // (all in one batch, as in the matrix-core kernel)
  const int n_tbl = a.n_tbl, n_sp0 = a.tbl[0].n_sp, row0 = a.cmb_row0, Hkv = a.Hkv, G = a.G, Hq = a.Hq, sp_max = a.sp_max;
  const float* const part = a.part;
  void* const out = a.o;
  float* const lse = a.lse;
  asm volatile("" ::"s"(n_tbl), "s"(n_sp0), "s"(row0), "s"(Hkv), "s"(G), "s"(Hq), "s"(sp_max), "s"(part), "s"(out), "s"(lse), "s"(a.half));
  const int units = Hkv < CMB_UNITS ? Hkv : CMB_UNITS;
  const int node = row0 + (int)blockIdx.x / units, unit = (int)blockIdx.x % units;
  int n_sp = n_sp0;
  if (n_tbl > 1) {
    // the table entry whose row range holds this node
    n_sp = 1;
    for (int base = 0; base < n_tbl; base += 64) {
      const int idx = base + lane;
      const int at = idx < n_tbl ? idx : n_tbl - 1;
      const int n0 = a.tbl[at].n0, M = a.tbl[at].M, cnt = a.tbl[at].n_sp;
      const unsigned long long hit = __ballot((node >= n0) & (node < n0 + M));
      if (hit != 0ull) {
        n_sp = __builtin_amdgcn_readlane(cnt, __builtin_ctzll(hit));
        break;
      }
    }
  } else if (n_tbl == 0) {
    // sequence of this node: last s with node_offsets[s] <= node
    int lo = 0, hi = a.B;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (a.node_offsets[mid] <= node) lo = mid; else hi = mid;
    }
    n_sp = splits_of(prefix_len_of(a, lo), a.split_len);
  }
  if (n_sp == 1) return;  // written directly by the attention kernel
  const int d = (int)threadIdx.x % LPR * 4;
  const int rows = (Hkv - unit + CMB_UNITS - 1) / CMB_UNITS * G;  // of this workgroup
  for (int j = (int)threadIdx.x / LPR; j < rows; j += (int)blockDim.x / LPR) {
    const int64_t row = (int64_t)node * Hq + (unit + j / G * CMB_UNITS) * G + j % G;
    const float* rec = part + row * sp_max * REC;
    float m = -HS_INF, l = 0.f;
    float4 o = {0.f, 0.f, 0.f, 0.f};
    for (int sp0 = 0; sp0 < n_sp; sp0 += AT_ONCE, rec += AT_ONCE * REC) {
      float2 ml[AT_ONCE];  // reference maximum and denominator, the same for all lanes of the row
      float4 v[AT_ONCE];
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {
        ml[u] = make_float2(-HS_INF, 0.f);
        v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (sp0 + u < n_sp) {
          ml[u] = *reinterpret_cast<const float2*>(rec + u * REC + D);
          v[u] = *reinterpret_cast<const float4*>(rec + u * REC + d);
        }
      }
      float top = m;
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) top = fmaxf(top, ml[u].x);
      // (a split without a finite score, e.g. of keys masked by -inf, left -inf, 0 and zeros: no weight, first or not)
      const float ref = top == -HS_INF ? 0.f : top;
      const float f = __expf(m - ref);  // (0 at the first eight)
      m = top;
      l *= f;
      o = make_float4(o.x * f, o.y * f, o.z * f, o.w * f);
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {
        const float w = __expf(ml[u].x - ref);  // (0 beyond the last split)
        l = fmaf(ml[u].y, w, l);
        o.x = fmaf(v[u].x, w, o.x);
        o.y = fmaf(v[u].y, w, o.y);
        o.z = fmaf(v[u].z, w, o.z);
        o.w = fmaf(v[u].w, w, o.w);
      }
    }
    const float inv = 1.f / l;
    store4<T>(static_cast<T*>(out) + row * D + d, make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv));
    if (lse && d == 0) lse[row] = m + __logf(l);
  }
}

constexpr int PLAN_CUS = 256;

struct AttnPlan {
  int split_len, sp_max, n_rb_max, max_rows;
  int64_t max_L;
  bool ok;
};

// Splits of the float32 kernel: a workgroup's time is its chain of trips over its split's keys, 5 us and 0.014 (D = 64) or
// 0.028 us a key; beyond one workgroup to a compute unit they slow each other down, first by half, then in proportion
// (workgroups of the grid that have nothing to do get in the way as well: three in five of the grid's count at least); the merge
// launch takes 4 us.  Measured, whole calls, 8 KV heads, split into: D = 64, 3 sequences of 962 to 1319 tokens, 33 to
// 40 rows: 256 tokens (360 workgroups) 18.8 us, 384 (264) 20.3, 512 (192) 17.1, 1024 (120) 24.1; one of 2000, 20 rows: 256
// 13.4, 512 15.9, 1024 22.9, unsplit 33.2; 4 of 283 to 437: 256 13.3, unsplit 12.7; 8 of 866 to 1819: 512 (704) 39.4,
// unsplit (216) 32.0.  D = 128, one of 432, 55 rows: 128 13.5, 256 16.3, unsplit 19.1; one of 595: 128 14.2, 256 15.5,
// 512 22.6; one of 213: 128 14.1, unsplit 14.4.
// one_launch: by the rule without this estimate the call would be unsplit.  It stays so while its chain is no longer than what
// a second launch costs the host: calls one behind the other take 14.6 us at least with one launch and 18 with two (D = 128, 8
// KV heads, in splits of 128 and unsplit: one and two sequences of 300 tokens, 20 rows 17.9 and 15.5, 18.0 and 15.7; 4 of 110 to
// 355, 10 to 21 rows 18.2 and 16.1; 4 of 350, 16 rows 18.2 and 17.1; with 40 rows on 2 KV heads 18.6 both).
constexpr float PLAN_ONE_LAUNCH_US = 15.7f;
static int64_t plan_float_split(const int32_t* hno, const int64_t* hpo, const int64_t* hlens, int B, int G, int Hkv, int D,
                                int n_rb_max, int rows_per_wg, int64_t max_L, bool one_launch) {
  const float key_us = D == 64 ? 0.014f : 0.028f;
  const int64_t least = D == 64 ? 256 : 128;  // a trip's keys
  int64_t best = 0, last = 0;
  float best_us = 0.f;
  for (int64_t cut = 1; cut <= 64; ++cut) {
    const int64_t len = std::max(least, ((max_L + cut - 1) / cut + 127) / 128 * 128);
    if (len == last) continue;
    last = len;
    int64_t wgs = 0, keys = 0;
    for (int s = 0; s < B; ++s) {
      const int M = hno[s + 1] - hno[s];
      if (M <= 0) continue;
      const int64_t L = hlens != nullptr ? hlens[s] : hpo[s + 1] - hpo[s];
      const int n = splits_of(L, (int)len);
      wgs += (int64_t)Hkv * ((G * M + rows_per_wg - 1) / rows_per_wg) * n;
      keys = std::max(keys, std::max(n > 1 ? len : 0, L - (n - 1) * len + M));
    }
    const int sp_max = splits_of(max_L, (int)len);
    const float grid = (float)Hkv * n_rb_max * sp_max * B;
    const float w = std::max((float)wgs, 0.6f * grid) / PLAN_CUS;
    const float us = (5.f + key_us * keys) * (w <= 1.f ? 1.f : std::max(w, 1.f + 0.5f * w)) + (sp_max > 1 ? 4.f : 0.f);
    if (best == 0 || us < best_us) {
      best = len;
      best_us = us;
    }
    if (len == least || w > 4.f || (one_launch && sp_max == 1 && us <= PLAN_ONE_LAUNCH_US)) break;
  }
  return best;
}

// Chooses the split length from the host copies of the offsets: enough workgroups to fill the
// chip, but splits long enough that partial records stay small next to the K/V they summarise.
// rows_per_wg: of the float32 kernel, 0 for the matrix-core kernel.  lean: the plan for a workspace that does not hold the
// usual one's records.
static AttnPlan plan_attention(const int32_t* hno, const int64_t* hpo, const int64_t* hlens, int B, int Hq, int Hkv, int D,
                               int rows_per_wg, bool lean) {
  AttnPlan p{};
  int max_M = 0;
  int64_t max_L = 0, sum_L = 0;
  for (int s = 0; s < B; ++s) {
    const int M = hno[s + 1] - hno[s];
    const int64_t L = hlens != nullptr ? hlens[s] : hpo[s + 1] - hpo[s];
    if (M > max_M) max_M = M;
    if (M > 0) {
      if (L > max_L) max_L = L;
      sum_L += L;
    }
  }
  p.max_rows = max_M;
  p.max_L = max_L;
  const int G = Hq / Hkv;
  p.n_rb_max = rows_per_wg > 0 ? (G * max_M + rows_per_wg - 1) / rows_per_wg : 1;
  if (p.n_rb_max < 1) p.n_rb_max = 1;
  // workgroups without splitting: one per (sequence, head, row block); split until the target is met
  const int64_t base_wgs = (int64_t)B * Hkv * p.n_rb_max;
  int64_t want = base_wgs > 0 ? (PLAN_CUS + base_wgs - 1) / base_wgs : 1;  // splits per average sequence
  if (want < 1) want = 1;
  const int64_t mean_L = B > 0 ? sum_L / B : 0;
  int64_t len = (mean_L + want - 1) / want;
  len = (len + 255) / 256 * 256;   // multiple of 256 tokens
  if (len < 512) len = 512;        // never split finer than 512 tokens
  // (many rounds of workgroups, of which the estimate knows nothing, are left to the rule above)
  if (rows_per_wg > 0 && !lean && base_wgs <= 4 * PLAN_CUS && max_L < (int64_t)1 << 30)
    len = plan_float_split(hno, hpo, hlens, B, G, Hkv, D, p.n_rb_max, rows_per_wg, max_L, splits_of(max_L, (int)len) == 1);
  p.split_len = (int)len;
  p.sp_max = splits_of(max_L, p.split_len);
  p.ok = true;
  return p;
}

// ---- work-list plan for the matrix-core kernel.
// Every (sequence, split, row group, KV head) is one work item = one workgroup.  The hardware
// starts workgroups in index order as compute units free up, so listing the items by falling cost
// is longest-processing-time-first scheduling.  The cost model (microseconds, fitted to
// measurements on MI355X) only has to rank alternatives: an item costs a fixed part plus a
// per-tile part that grows with the number of waves that have rows.
constexpr float PLAN_ITEM_US = 10.f;
// Splits of at least 128 tokens (the workspace bound relies on it).  A launch of few workgroups is mostly an
// item's fixed cost: one layer of the 8B shape (32 tiles a head) takes 25.9 us cut into 4 x 8 tiles, 23.5 us
// into 8 x 4 or 16 x 2, combine launch included.
constexpr int PLAN_MIN_SPLIT_TILES = 2;
// A launch of at most half as many items as compute units can give each item two workgroups of up to 128 rows,
// in which two waves share a row block and take every other 32 keys ("narrow"): 0.65 us a tile instead of 1.05 on
// an otherwise idle chip for items of more than 128 rows (33 and 126 tiles a workgroup, 244 rows: 43.9 and 140 us
// -> 31.2 and 91 us).
// At most a quarter as many can be given four, of up to 64 rows each: four waves to a row block, half the sums to
// exchange and half the records to write for each of them.  Whole calls, one layer, 8 KV heads, best cut with two and with four: 61 rows on 500 /
// 1000 / 2048 / 4096 tokens 14.6 / 16.0 / 18.3 / 20.3 us and 13.9 / 15.1 / 16.7 / 19.5, D = 64 on 2048 13.3 and 12.9; 40
// heads, 129 rows on 400 tokens 18.3 and 16.4.  None gained by items of at most 128 rows (20 on 2048 14.9 and 15.3), nor by long
// prefixes, which want more splits than that leaves room for (9000 tokens 27.1 and 29.5).  Nor, with D = 128, by trees
// beyond 256 rows: 300 rows on 500 tokens, 16 heads one row each, 18.6 us with two and 21.4 with four, on 2000 25.2 and 25.1; 8 heads on 2, 260 rows
// on 400 18.4 and 19.8, 300 on 1000 21.1 and 22.3, 1024 on 2000 40.7 and 48.9.  With D = 64 they do: 8 heads on 4, 300 on 1000 17.7 and 16.8, 1024 on 200 24.4 and
// 23.9, 8 on 8, 300 on 2000 18.2 and 17.6; but 16 on 16, 300 on 1000 18.0 and 19.4.
constexpr int PLAN_NARROW_ITEMS = PLAN_CUS / 2, PLAN_QUARTER_ITEMS = PLAN_CUS / 4, PLAN_QUARTER_ROWS = 256;
// Launches that give every item a compute unit of its own, either way: the longest item decides.  A tile costs
// the more the more K/V streams are read at a time, and above 128 rows, where two waves share a SIMD, the matrix
// instructions' time at least; up to 128 rows two waves to a row block gain nothing, and cost more to start and
// to end.  Measured per tile with 28 / 115 / 180 / 230 streams: narrow 0.70, 0.87; else up to 128 rows 0.71, 0.82,
// 0.97, 1.11; 256 rows 1.1, 1.2, 1.6, 1.65, at D = 64 0.75 to 1.1.  The constants are those that chose the best of
// all cuts in 2499 random launches (1 to 48 entries, 60 to 12000 tokens, 1 to 300 rows, five head layouts, both head
// dimensions; 1.4 % above each launch's best cut on average), which makes them higher than the times: the estimates
// of fuller launches that they are compared with are high as well.  (Every launch of up to 128 items narrow, with
// flat costs a tile: 2.0 %; 3 entries of 2344 tokens, 66 rows, 40 heads 49.0 us, now and without narrow launches 39.4;
// one of 8945 tokens, 130 rows 68 and 55; without narrow launches 9.9 % on average.)
// (narrow: 0 to 2, as in AttnArgs)
static inline float plan_own_cu_us(int narrow, bool half, int waves, int tiles, float streams) {
  const float item = waves > 4 ? (narrow == 2 ? 10.4f : 12.f) : narrow && waves > 2 ? 8.4f : 6.5f;
  float tile = narrow ? 0.88f + 0.0029f * streams : 1.07f + 0.0018f * streams;
  if (!narrow && waves > 4) tile = std::max(tile, half ? 1.35f : 1.5f);
  return item + (float)tiles * tile;
}
// Waves share row blocks (AttnArgs::share) in launches of more than one round of the compute units.  Sequences of a
// single row group gain 3 to 5 % in launches that follow one another, but a launch that follows other kernels, as in a
// step, loses some in its first round: short items earn that back in the fifth round or so, long ones in the second.  Whole
// steps, a block to a wave and shared: 129 rows, 40 heads, 10 / 20 / 30 layers on 4096 tokens 224 / 376 / 539 us and 214 / 364 / 513, 20 layers on
// 2000 tokens 241 and 231, on 1000 161 and 163; 46 rows, 8 KV heads, 80 layers on 2048 205 and 200, on 1000 137 and 141, 40 layers (320
// items) on 2048 132 and 140.  With several groups there is no such loss: 73 rows, 20 and 40
// layers 138 and 197, shared 127 and 180.  Nor in ragged batches, whose workgroups drift apart (16 sequences, whole step 400 us,
// 395 with the sharing of several groups alone, 381 with both).
constexpr int PLAN_SHARE_ITEMS = 5 * PLAN_CUS;
constexpr int PLAN_SHARE_LONG_ITEMS = 3 * PLAN_CUS / 2, PLAN_SHARE_LONG = 24;  // (from so many tiles to an item)
constexpr int PLAN_MIN_SPLIT_TOKENS = PLAN_MIN_SPLIT_TILES * 64;
static inline float plan_tile_us(int waves) { return 1.25f + 0.04f * (float)waves; }

struct ListPlan {
  float est_us;
  int target;
  int tail, cuts;  // the last `tail` entries have each of their splits cut into `cuts` once more (0, 1: none)
  int narrow;      // 1: two workgroups to an item, 2: four
};

// Equal entries whose items do not fill whole rounds of the compute units: the entries that spill into the
// last round can be cut finer, so that their items fill the chip.  When do `q` items of cost c and, behind
// them, `m` items of cost s end?
static inline float plan_two_sizes(int64_t q, float c, int64_t m, float s) {
  const int64_t k = q / PLAN_CUS, r = q % PLAN_CUS;        // k whole rounds, then r compute units have one more
  const int64_t early = (PLAN_CUS - r) * (int64_t)(c / s);  // small items that end while they do
  const float full = (float)(k + (r > 0 ? 1 : 0)) * c;
  if (m <= early) {
    const float end = (float)k * c + (float)((m + PLAN_CUS - r - 1) / (PLAN_CUS - r)) * s;
    return end > full ? end : full;
  }
  return (float)(k + 1) * c + (float)((m - early + PLAN_CUS - 1) / PLAN_CUS) * s;
}

// Splits of a sequence of `tiles` prefix tiles when items should hold about `target` tiles.
static inline int plan_splits(int tiles, int target, int sp_cap, bool paged = false) {
  int n = (tiles + target / 2) / target;
  const int most = tiles / PLAN_MIN_SPLIT_TILES;
  if (n > most) n = most;
  if (n > sp_cap) n = sp_cap;
  if (paged && n < (tiles + 255) / 256) n = (tiles + 255) / 256;  // the kernel holds the pages of 256 tiles
  return n < 1 ? 1 : n;
}

// The cut itself: `per` tiles to a split, and as many splits as that takes (rounding `per` up can make
// the last of the splits asked for empty: they are dropped, every split starts inside the prefix).
static inline void plan_cut(int tiles, int target, int sp_cap, bool paged, int* nsp, int* per) {
  int n = plan_splits(tiles, target, sp_cap, paged);
  int p = (tiles + n - 1) / n;
  if (p < 1) p = 1;
  n = (tiles + p - 1) / p;
  *nsp = n < 1 ? 1 : n;
  *per = p;
}

// Fills a.tbl / a.n_tbl / a.n_items / a.sp_max.  Returns false when the batch does not fit the table.
// lean: the plan for a workspace that does not hold the usual one's records (fewer cuts, hence fewer
// records): no finer last round, no two workgroups to an item.
static bool plan_worklist(AttnArgs& a, const int32_t* hno, const int64_t* hpo, const int64_t* hlens, int B,
                          int sp_cap, bool lean) {
  struct Seq {
    int s, M, tiles, rg, waves0, waves_last, ttiles;
    float tile_us;  // of its largest group if that were full: what the entries are ordered by
  };
  Seq seqs[ATTN_TBL];
  int n = 0, max_rows = 0;
  for (int s = 0; s < B; ++s) {
    const int M = hno[s + 1] - hno[s];
    const int64_t L = hlens != nullptr ? hlens[s] : hpo[s + 1] - hpo[s];
    if (M <= 0) continue;
    if (n == ATTN_TBL || L >= (int64_t)1 << 30) return false;
    const int blocks = row_blocks(a.G, a.half, M);
    Seq q;
    q.s = s;
    q.M = M;
    max_rows = std::max(max_rows, M);
    q.tiles = (int)((L + 63) / 64);
    q.tile_us = plan_tile_us(std::min(8, (a.G * M + 31) / 32));
    q.rg = row_groups(blocks);
    int first;
    row_group(blocks, 0, &first, &q.waves0);
    row_group(blocks, q.rg - 1, &first, &q.waves_last);
    q.ttiles = (M + 63) / 64;
    seqs[n++] = q;
  }
  if (n == 0) return false;
  // Unequal items (a ragged batch): the makespan of each candidate is found by replaying the
  // hardware's dispatch, which hands the next workgroup in index order to the first compute unit
  // that falls free (list scheduling).  Equal items (the layers of one step) run in whole rounds.
  static const int targets[] = {1 << 20, 192, 160, 128, 112, 96, 80, 72, 64, 56, 48, 40, 32, 24, 16, 12, 8, 6, 4, 2};
  // Cuts finer than eight tiles are candidates only while eight-tile items would leave compute units idle
  // (a launch of one or two layers): such an item is mostly its fixed cost.
  int64_t coarse_items = 0;
  for (int i = 0; i < n; ++i) coarse_items += (int64_t)a.Hkv * seqs[i].rg * (seqs[i].tiles / 8 > 0 ? seqs[i].tiles / 8 : 1);
  const int n_targets = (int)(sizeof(targets) / sizeof(targets[0])) - (coarse_items < PLAN_CUS ? 0 : 3);
  bool equal = true;  // entries of one size
  for (int i = 1; i < n; ++i) equal = equal && seqs[i].M == seqs[0].M && seqs[i].tiles == seqs[0].tiles;
  ListPlan best{0.f, 0, 0, 1, 0};
  static thread_local std::vector<float> item_cost, cu_free;  // (kept between calls: no allocation in the steady state)
  for (int ti = 0; ti < n_targets; ++ti) {
    const int target = targets[ti];
    if (lean && (target == 12 || target == 6)) continue;
    double total = 0.0, rec_bytes = 0.0;
    float mx = 0.f, mn = 1e30f;
    int64_t items = 0;
    int ord[ATTN_TBL];
    float seq_cost[ATTN_TBL];
    for (int i = 0; i < n; ++i) {
      const Seq& q = seqs[i];
      int nsp, per;
      plan_cut(q.tiles, target, sp_cap, a.block_table != nullptr, &nsp, &per);
      const float big = PLAN_ITEM_US + (float)(per + q.ttiles) * plan_tile_us(q.waves0);
      const float one = PLAN_ITEM_US + (float)per * plan_tile_us(q.waves0);
      const float one_last = PLAN_ITEM_US + (float)per * plan_tile_us(q.waves_last);
      total += (double)a.Hkv * nsp * ((q.rg - 1) * one + one_last);
      items += (int64_t)a.Hkv * nsp * q.rg;
      if (big > mx) mx = big;
      if (one_last < mn) mn = one_last;
      if (nsp > 1) rec_bytes += (double)q.M * a.Hq * nsp * ((a.half ? 64 : 128) + ATTN_REC_PAD) * 4 * 2;  // written, then read
      ord[i] = i;
      seq_cost[i] = (float)per * q.tile_us;
    }
    const float combine_us = rec_bytes > 0.0 ? 4.f + (float)(rec_bytes / 2.5e6) : 0.f;  // the combine launch, ~2.5 TB/s
    if (items <= PLAN_CUS && !lean) {  // every item has a compute unit of its own
      int longest = 0;     // tiles of an item
      double streamed = 0.0;  // tiles of all items, row groups of the same keys as one
      for (int i = 0; i < n; ++i) {
        const Seq& q = seqs[i];
        int nsp, per;
        plan_cut(q.tiles, target, sp_cap, a.block_table != nullptr, &nsp, &per);
        longest = std::max(longest, per + q.ttiles);
        streamed += (double)a.Hkv * nsp * (per + q.ttiles);
      }
      const float streams = (float)(streamed / longest);  // read at a time while the longest item runs
      const bool quarter = items <= PLAN_QUARTER_ITEMS && (a.half != 0 || max_rows <= PLAN_QUARTER_ROWS);
      for (int narrow = 0; narrow <= (quarter ? 2 : items <= PLAN_NARROW_ITEMS ? 1 : 0); ++narrow) {
        float est = 0.f;
        for (int i = 0; i < n; ++i) {
          const Seq& q = seqs[i];
          int nsp, per;
          plan_cut(q.tiles, target, sp_cap, a.block_table != nullptr, &nsp, &per);
          est = std::max(est, plan_own_cu_us(narrow, a.half != 0, q.waves0, per + q.ttiles, streams));
        }
        est += combine_us;
        if (best.target == 0 || est < best.est_us) best = ListPlan{est, target, 0, 1, narrow};
      }
      continue;
    }
    // Equal entries, a last round that is not full: its entries cut finer.  (Layers of
    // the 8B head layout in one call: 33 of 2048 tokens and 61 rows, 264 items for 256 compute units, 112 us
    // uncut and 91 with the last layer in eight; 38 of 6000 tokens and 33 rows 242 and 189; 129 rows on 4096
    // tokens, 40 layers and heads, 730 and 707.)
    if (equal && !lean && n > 1 && items > PLAN_CUS && items % PLAN_CUS != 0) {
      const Seq& q = seqs[0];
      int nsp, per;
      plan_cut(q.tiles, target, sp_cap, a.block_table != nullptr, &nsp, &per);
      const int64_t entry_items = items / n;
      const int tail = (int)((items % PLAN_CUS + entry_items - 1) / entry_items);
      for (int cuts = 2; cuts <= 8 && tail < n; cuts *= 2) {
        const int per2 = (per + cuts - 1) / cuts;
        const int nsp2 = (q.tiles + per2 - 1) / per2;
        if (per2 < 2 * PLAN_MIN_SPLIT_TILES || nsp2 > sp_cap) break;
        const float c = PLAN_ITEM_US + (float)(per + q.ttiles) * plan_tile_us(q.waves0);
        const float small = PLAN_ITEM_US + (float)(per2 + q.ttiles) * plan_tile_us(q.waves0);
        const double rec = (double)q.M * a.Hq * ((a.half ? 64 : 128) + ATTN_REC_PAD) * 4 * 2 *
                           ((double)tail * nsp2 + (nsp > 1 ? (double)(n - tail) * nsp : 0.0));
        const float est = plan_two_sizes(entry_items * (n - tail), c, entry_items / nsp * nsp2 * tail, small) +
                          4.f + (float)(rec / 2.5e6);
        if (best.target == 0 || est < best.est_us) best = ListPlan{est, target, tail, cuts, 0};
      }
    }
    // (no schedule ends before the work divided by the compute units, nor before its longest item: a
    // candidate whose bound is no better than the best estimate so far needs no replay)
    {
      const float floor_us = (float)(total / PLAN_CUS) > mx ? (float)(total / PLAN_CUS) : mx;
      if (best.target != 0 && floor_us + combine_us >= best.est_us) continue;
    }
    float est;
    if (mx - mn <= 0.1f * mx || items > 8192) {
      est = (float)(total / PLAN_CUS) + 0.15f * mx;
      if (mx > est) est = mx;
      if (mx - mn <= 0.1f * mx) {  // equal items run in whole rounds
        const float rounds = (float)((items + PLAN_CUS - 1) / PLAN_CUS) * (float)(total / (double)items);
        if (rounds > est) est = rounds;
      }
    } else {
      // the items in dispatch order (as the table below lists them), then the replay
      std::stable_sort(ord, ord + n, [&](int x, int y) { return seq_cost[x] > seq_cost[y]; });
      item_cost.clear();
      for (int k = 0; k < n; ++k) {
        const Seq& q = seqs[ord[k]];
        int nsp, per;
        plan_cut(q.tiles, target, sp_cap, a.block_table != nullptr, &nsp, &per);
        for (int sp = 0; sp < nsp; ++sp) {
          int t = q.tiles - sp * per;
          t = t > per ? per : (t < 0 ? 0 : t);
          if (sp == nsp - 1) t += q.ttiles;
          for (int rg = 0; rg < q.rg; ++rg) {
            const float c = PLAN_ITEM_US + (float)t * plan_tile_us(rg == q.rg - 1 ? q.waves_last : q.waves0);
            for (int h = 0; h < a.Hkv; ++h) item_cost.push_back(c);
          }
        }
      }
      cu_free.assign(PLAN_CUS, 0.f);
      std::make_heap(cu_free.begin(), cu_free.end(), std::greater<float>());
      float end = 0.f;
      for (float c : item_cost) {
        std::pop_heap(cu_free.begin(), cu_free.end(), std::greater<float>());
        const float done = cu_free.back() + c;
        cu_free.back() = done;
        std::push_heap(cu_free.begin(), cu_free.end(), std::greater<float>());
        if (done > end) end = done;
      }
      est = end;
    }
    est += combine_us;
    if (best.target == 0 || est < best.est_us) best = ListPlan{est, target, 0, 1, 0};
  }
  // the table: sequences by falling cost of an item
  int order[ATTN_TBL];
  float cost[ATTN_TBL];
  int nsp_of[ATTN_TBL], per_of[ATTN_TBL];
  for (int i = 0; i < n; ++i) {
    const Seq& q = seqs[i];
    plan_cut(q.tiles, best.target, sp_cap, a.block_table != nullptr, &nsp_of[i], &per_of[i]);
    if (i >= n - best.tail) {
      per_of[i] = (per_of[i] + best.cuts - 1) / best.cuts;
      nsp_of[i] = (q.tiles + per_of[i] - 1) / per_of[i];
    }
    cost[i] = (float)per_of[i] * q.tile_us;
    order[i] = i;
  }
  std::stable_sort(order, order + n, [&](int x, int y) { return cost[x] > cost[y]; });
  int64_t first = 0;
  int sp_max = 1;
  for (int k = 0; k < n; ++k) {
    const int i = order[k];
    const Seq& q = seqs[i];
    SeqEntry& e = a.tbl[k];
    e.first_item = (int)first;
    e.n0 = hno[q.s];
    e.M = q.M;
    e.L = (int)(hlens != nullptr ? hlens[q.s] : hpo[q.s + 1] - hpo[q.s]);
    e.p0 = a.block_table != nullptr ? (long long)q.s * a.max_blocks : hpo[q.s];
    e.tiles_per_split = per_of[i];
    e.n_sp = (short)nsp_of[i];
    e.n_rg = (short)q.rg;
    first += (int64_t)a.Hkv * nsp_of[i] * q.rg;
    if (nsp_of[i] > sp_max) sp_max = nsp_of[i];
    if (first >= (int64_t)1 << 30) return false;
  }
  a.cmb_row0 = hno[seqs[n - 1].s + 1];  // (rows before the first entry with several splits need no merge)
  for (int i = n - 1; i >= 0; --i)
    if (nsp_of[i] > 1) a.cmb_row0 = hno[seqs[i].s];
  a.n_tbl = n;
  a.n_items = (int)first;
  a.narrow = best.narrow;
  a.share = first <= PLAN_CUS ? 0 : !equal || first > (per_of[0] >= PLAN_SHARE_LONG ? PLAN_SHARE_LONG_ITEMS : PLAN_SHARE_ITEMS) ? 2 : 1;
  a.sp_max = sp_max;
  return true;
}

// The plan depends on the host arrays and the head layout alone, and a model calls the attention of all its
// layers with the same ones: the last few plans are kept per thread.  (Planning a ragged batch of 16 sequences
// replays some twenty candidate cuts over hundreds of items each, a few hundred microseconds on the host:
// more than the launch itself takes on the GPU.)
struct PlanMemo {
  std::vector<int64_t> key;  // everything the plan is a function of; empty: unused slot
  bool ok;
  int n_tbl, n_items, narrow, share, sp_max, cmb_row0;
  SeqEntry tbl[ATTN_TBL];
};
constexpr int PLAN_MEMO_SLOTS = 4;
constexpr int PLAN_MEMO_MAX_B = 1024;  // larger batches (at most 96 of their entries non-empty) are planned every time

static bool plan_worklist_memo(AttnArgs& a, const int32_t* hno, const int64_t* hpo, const int64_t* hlens, int B,
                               int sp_cap, bool lean) {
  if (B > PLAN_MEMO_MAX_B) return plan_worklist(a, hno, hpo, hlens, B, sp_cap, lean);
  static thread_local PlanMemo memo[PLAN_MEMO_SLOTS];
  static thread_local unsigned next_slot = 0;
  static thread_local std::vector<int64_t> key;
  key.clear();
  key.push_back(B);
  key.push_back(sp_cap);
  key.push_back(lean ? 1 : 0);
  key.push_back(a.G);
  key.push_back(a.Hkv);
  key.push_back(a.half);
  key.push_back(a.block_table != nullptr ? 1 + (int64_t)a.max_blocks : 0);  // (paged: an entry's p0 is s * max_blocks)
  key.push_back((hpo != nullptr ? 1 : 0) + (hlens != nullptr ? 2 : 0));
  for (int s = 0; s <= B; ++s) key.push_back(hno[s]);
  if (hpo != nullptr)
    for (int s = 0; s <= B; ++s) key.push_back(hpo[s]);
  if (hlens != nullptr)
    for (int s = 0; s < B; ++s) key.push_back(hlens[s]);
  for (PlanMemo& m : memo)
    if (m.key == key) {
      if (m.ok) {
        a.n_tbl = m.n_tbl;
        a.n_items = m.n_items;
        a.narrow = m.narrow;
        a.share = m.share;
        a.sp_max = m.sp_max;
        a.cmb_row0 = m.cmb_row0;
        memcpy(a.tbl, m.tbl, sizeof(SeqEntry) * (size_t)m.n_tbl);
      }
      return m.ok;
    }
  PlanMemo& m = memo[next_slot++ % PLAN_MEMO_SLOTS];
  m.ok = plan_worklist(a, hno, hpo, hlens, B, sp_cap, lean);
  m.key = key;
  if (m.ok) {
    m.n_tbl = a.n_tbl;
    m.n_items = a.n_items;
    m.narrow = a.narrow;
    m.share = a.share;
    m.sp_max = a.sp_max;
    m.cmb_row0 = a.cmb_row0;
    memcpy(m.tbl, a.tbl, sizeof(SeqEntry) * (size_t)a.n_tbl);
  }
  return m.ok;
}

}  // namespace hs

using namespace hs;

static size_t part_bytes(int64_t NN, int Hq, int D, int sp_max) {
  if (sp_max <= 1) return 0;
  return align_up((size_t)NN * Hq * sp_max * (D + ATTN_REC_PAD) * sizeof(float), 256);
}

extern "C" size_t hs_tree_attention_workspace(int32_t B, int32_t NN, int64_t total_prefix, int32_t Hq, int32_t Hkv,
                                              int32_t D, hs_dtype dt) {
  (void)dt;
  if (B <= 0 || NN <= 0 || Hq <= 0 || Hkv <= 0 || D <= 0 || total_prefix < 0) return 0;
  // upper bound over every plan the launch may choose: splits are at least PLAN_MIN_SPLIT_TOKENS long
  const int64_t sp_bound = total_prefix / PLAN_MIN_SPLIT_TOKENS + 1;
  // (+ what trees of more than 256 rows ask for besides: such a tree needs NN > 256)
  return part_bytes(NN, Hq, D, (int)(sp_bound < 2 ? 2 : sp_bound > 64 ? 64 : sp_bound)) +
         align_up(attn_mfma_table_bytes(NN < MAX_TREE_ROWS ? NN : MAX_TREE_ROWS, NN), 256);
}

extern "C" hs_status hs_tree_attention(const void* q, const void* k_prefix, const void* v_prefix, const void* k_tree,
                                       const void* v_tree, const int32_t* parent, const int32_t* node_offsets,
                                       const int64_t* prefix_offsets, const int32_t* host_node_offsets,
                                       const int64_t* host_prefix_offsets, int32_t B, int32_t Hq, int32_t Hkv,
                                       int32_t D, hs_dtype dt, float scale, void* o, float* lse, void* workspace,
                                       size_t workspace_bytes, hs_stream stream) {
  return hs_tree_attention_lens(q, k_prefix, v_prefix, k_tree, v_tree, parent, node_offsets, prefix_offsets,
                                host_node_offsets, host_prefix_offsets, nullptr, nullptr, B, Hq, Hkv, D, dt, scale, o,
                                lse, workspace, workspace_bytes, stream);
}

// Events that hs_time_next_attention left for this thread's next attention call.
static thread_local hipEvent_t timing_start = nullptr, timing_stop = nullptr;
// Kernel that this thread's last attention call launched (hs_tree_attention_last_kernel).
static thread_local int last_kernel = 0;

extern "C" int32_t hs_tree_attention_last_kernel(void) { return last_kernel; }

// How its row blocks went to workgroups and waves, or would have (hs_tree_attention_last_form).
static thread_local int last_form = 0;

extern "C" int32_t hs_tree_attention_last_form(void) { return last_form; }

extern "C" hs_status hs_time_next_attention(void* start_event, void* stop_event) {
  clear_error();
  HS_REQUIRE((start_event == nullptr) == (stop_event == nullptr), HS_ERR_NULL,
             "hs_time_next_attention: give both events or neither");
  timing_start = static_cast<hipEvent_t>(start_event);
  timing_stop = static_cast<hipEvent_t>(stop_event);
  return HS_OK;
}

// What hs_tree_attention_plan reports (host memory; per_seq may be NULL).
struct PlanReport {
  int64_t* totals;   // [6]
  int32_t* per_seq;  // [B][4]
};

// The three entry points in one: dense prefix regions (prefix_lens NULL), regions with spare
// capacity (prefix_lens given), pages (block_table given: k_prefix / v_prefix are the page pools,
// the offset arrays are absent).
static hs_status attention_impl(const void* q, const void* k_prefix, const void* v_prefix, const void* k_tree,
                                const void* v_tree, const int32_t* parent, const int32_t* node_offsets,
                                const int64_t* prefix_offsets, const int32_t* host_node_offsets,
                                const int64_t* host_prefix_offsets, const int64_t* prefix_lens,
                                const int64_t* host_prefix_lens, const int32_t* block_table, int32_t max_blocks,
                                int32_t B, int32_t Hq, int32_t Hkv, int32_t D, hs_dtype dt, float scale, void* o,
                                float* lse, void* workspace, size_t workspace_bytes, hs_stream stream,
                                bool tree_shared = false, const PlanReport* report = nullptr) {
  // report != NULL: plan only.  The host arrays are read and checked as in a real call, the device
  // pointers may be NULL, nothing is launched; the report says how the launch would be cut.
  const bool plan_only = report != nullptr;
  if (plan_only)
    for (int k = 0; k < 6; ++k) report->totals[k] = 0;
  const bool paged = block_table != nullptr;
  hipEvent_t ev_start = nullptr, ev_stop = nullptr;
  last_form = 0;
  if (!plan_only) {
    ev_start = timing_start;  // one-shot, whatever this call comes to
    ev_stop = timing_stop;
    timing_start = timing_stop = nullptr;
    last_kernel = 0;
  }
  HS_REQUIRE(B >= 0, HS_ERR_SHAPE, "hs_tree_attention: B=%d", B);
  HS_REQUIRE(Hq >= 1 && Hkv >= 1 && Hq % Hkv == 0, HS_ERR_SHAPE, "hs_tree_attention: Hq=%d must be a multiple of Hkv=%d",
             Hq, Hkv);
  HS_REQUIRE(D == 64 || D == 128, HS_ERR_UNSUPPORTED, "hs_tree_attention: head dimension %d (64 and 128 are built)", D);
  HS_REQUIRE(dt == HS_F32 || dt == HS_BF16, HS_ERR_SHAPE, "hs_tree_attention: unknown dtype %d", (int)dt);
  if (B == 0) return HS_OK;
  HS_REQUIRE(host_node_offsets && (paged || host_prefix_offsets) &&
                 (plan_only || (node_offsets && (paged || prefix_offsets))),
             HS_ERR_NULL, "hs_tree_attention: offset arrays (device and host copies) are required");
  HS_REQUIRE(host_node_offsets[0] == 0 && (paged || host_prefix_offsets[0] == 0), HS_ERR_SHAPE,
             "hs_tree_attention: offsets must start at 0");
  HS_REQUIRE(!paged || ((plan_only || prefix_lens) && host_prefix_lens && max_blocks >= 0), HS_ERR_NULL,
             "hs_tree_attention_paged: prefix lengths (device and host) are required");
  int64_t total_used = 0;
  for (int s = 0; s < B; ++s) {
    const int M = host_node_offsets[s + 1] - host_node_offsets[s];
    if (paged) {
      HS_REQUIRE(M >= 0, HS_ERR_SHAPE, "hs_tree_attention: offsets decrease at sequence %d", s);
      HS_REQUIRE(host_prefix_lens[s] >= 0 && host_prefix_lens[s] <= (int64_t)max_blocks * 64, HS_ERR_SHAPE,
                 "hs_tree_attention_paged: prefix length of sequence %d exceeds its %d blocks", s, max_blocks);
      // (a key split holds the pages of at most 256 tiles, a sequence has at most 64 splits)
      HS_REQUIRE(host_prefix_lens[s] <= (int64_t)64 * 256 * 64, HS_ERR_UNSUPPORTED,
                 "hs_tree_attention_paged: prefix of sequence %d is longer than %d tokens", s, 64 * 256 * 64);
      total_used += host_prefix_lens[s];
      HS_REQUIRE(M <= MAX_TREE_ROWS, HS_ERR_UNSUPPORTED, "hs_tree_attention: sequence %d has %d tree rows (limit %d)",
                 s, M, MAX_TREE_ROWS);
      continue;
    }
    HS_REQUIRE(M >= 0 && host_prefix_offsets[s + 1] >= host_prefix_offsets[s], HS_ERR_SHAPE,
               "hs_tree_attention: offsets decrease at sequence %d", s);
    HS_REQUIRE(M <= MAX_TREE_ROWS, HS_ERR_UNSUPPORTED, "hs_tree_attention: sequence %d has %d tree rows (limit %d)", s,
               M, MAX_TREE_ROWS);
    HS_REQUIRE(host_prefix_lens == nullptr ||
                   (host_prefix_lens[s] >= 0 && host_prefix_lens[s] <= host_prefix_offsets[s + 1] - host_prefix_offsets[s]),
               HS_ERR_SHAPE, "hs_tree_attention: prefix length of sequence %d exceeds its region", s);
  }
  HS_REQUIRE(plan_only || (prefix_lens == nullptr) == (host_prefix_lens == nullptr), HS_ERR_NULL,
             "hs_tree_attention: prefix_lens and host_prefix_lens go together");
  const int NN = host_node_offsets[B];
  const int64_t total_prefix = paged ? total_used : host_prefix_offsets[B];
  if (NN == 0) return HS_OK;
  HS_REQUIRE(plan_only || (q && k_tree && v_tree && parent && o), HS_ERR_NULL, "hs_tree_attention: NULL tensor");
  HS_REQUIRE(plan_only || total_prefix == 0 || (k_prefix && v_prefix), HS_ERR_NULL, "hs_tree_attention: NULL prefix cache");

  int max_M = 0;
  for (int s = 0; s < B; ++s) max_M = std::max(max_M, host_node_offsets[s + 1] - host_node_offsets[s]);
  auto aligned16 = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  // (head-count limits: the matrix-core kernel numbers rows and lane offsets in narrow types)
  // D = 64: the matrix-core kernel takes the KV heads in pairs (their number must be even); a pair
  // then has twice the query heads
  const bool pairs = D == 64;
  const int kv_units = pairs ? Hkv / 2 : Hkv, g_unit = pairs ? 2 * (Hq / Hkv) : Hq / Hkv;
  const bool mfma = attn_mfma_supported(D, dt, max_M, scale) && (!pairs || Hkv % 2 == 0) && g_unit <= 128 &&
                    (int64_t)g_unit * max_M < 65536 && Hkv <= 4096 && aligned16(q) &&
                    aligned16(k_prefix) && aligned16(v_prefix) && aligned16(k_tree) && aligned16(v_tree) &&
                    aligned16(o);
  AttnArgs a;
  a.q = q; a.k_prefix = k_prefix; a.v_prefix = v_prefix; a.k_tree = k_tree; a.v_tree = v_tree;
  a.parent = parent; a.tree_shared = tree_shared ? 1 : 0; a.node_offsets = node_offsets; a.prefix_offsets = prefix_offsets; a.prefix_lens = prefix_lens;
  a.block_table = block_table; a.max_blocks = max_blocks;
  a.B = B; a.Hq = Hq; a.Hkv = mfma ? kv_units : Hkv; a.G = mfma ? g_unit : Hq / Hkv; a.half = mfma && pairs ? 1 : 0; a.scale = scale;
  a.o = o; a.lse = lse; a.part = static_cast<float*>(workspace);
  a.n_tbl = 0; a.n_items = 0; a.narrow = 0; a.share = 0; a.cmb_row0 = 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the workspace query bounds the splits of a sequence the same way
  const int64_t sp_bound = total_prefix / PLAN_MIN_SPLIT_TOKENS + 1;
  const int sp_cap = (int)(sp_bound < 2 ? 2 : sp_bound > 64 ? 64 : sp_bound);

  AttnPlan plan{};
  auto plan_plain = [&](bool lean) {
    plan = plan_attention(host_node_offsets, host_prefix_offsets, host_prefix_lens, B, Hq, a.Hkv, D, mfma ? 0 : GEN_ROWS, lean);
    while (plan.sp_max > sp_cap) {
      plan.split_len *= 2;
      plan.sp_max = splits_of(plan.max_L, plan.split_len);
    }
    if (paged && plan.split_len > 256 * 64) {  // the matrix-core kernel holds the pages of 256 tiles per split
      plan.split_len = 256 * 64;
      plan.sp_max = splits_of(plan.max_L, plan.split_len);
    }
    a.split_len = plan.split_len; a.sp_max = plan.sp_max; a.n_rb_max = plan.n_rb_max;
  };
  if (!(mfma && plan_worklist_memo(a, host_node_offsets, host_prefix_offsets, host_prefix_lens, B, sp_cap, false))) {
    a.n_tbl = 0;
    a.cmb_row0 = 0;
    a.share = (int64_t)B * a.Hkv > PLAN_SHARE_ITEMS ? 2 : 1;  // (more than 96 sequences, or not for the matrix-core kernel)
    plan_plain(false);
  } else {
    a.split_len = 0; a.n_rb_max = 1;
  }
  const size_t table_bytes = mfma ? align_up(attn_mfma_table_bytes(max_M, NN), 256) : 0;
  size_t need = part_bytes(NN, Hq, D, a.sp_max) + table_bytes;
  // a workspace that is too small for this plan may still hold the one with fewer cuts
  if (!plan_only && a.sp_max > 1 && (workspace == nullptr || workspace_bytes < need)) {
    if (a.n_tbl > 0) plan_worklist_memo(a, host_node_offsets, host_prefix_offsets, host_prefix_lens, B, sp_cap, true);
    else plan_plain(true);
    need = part_bytes(NN, Hq, D, a.sp_max) + table_bytes;
  }
  if (mfma && a.share != 0) {  // (none shares: the launch takes the instantiation without that code)
    bool any = false;
    for (int s = 0; s < B && !any; ++s)
      any = groups_share(row_blocks(a.G, a.half, host_node_offsets[s + 1] - host_node_offsets[s]), a.share);
    if (!any) a.share = 0;
  }
  last_form = mfma ? (1 << a.narrow) + 16 * a.share : 0;
  if (plan_only) {
    const int n_rg_max = mfma ? (a.G * max_M + 255) / 256 : plan.n_rb_max;
    report->totals[0] = mfma ? 1 : 2;
    report->totals[1] = a.n_tbl > 0 ? a.n_items : (int64_t)a.Hkv * n_rg_max * a.sp_max * B;
    report->totals[2] = a.sp_max;
    report->totals[3] = a.split_len;
    report->totals[4] = (int64_t)need;
    report->totals[5] = a.sp_max > 1 ? 1 : 0;
    if (report->per_seq != nullptr) {
      for (int s = 0; s < B; ++s) {
        int32_t* r = report->per_seq + 4 * s;
        const int M = host_node_offsets[s + 1] - host_node_offsets[s];
        const int64_t L = host_prefix_lens != nullptr ? host_prefix_lens[s] : host_prefix_offsets[s + 1] - host_prefix_offsets[s];
        r[0] = M > 0 ? splits_of(L, a.split_len > 0 ? a.split_len : 1 << 30) : 0;
        r[1] = a.split_len / 64;
        r[2] = M > 0 ? (mfma ? (a.G * M + 255) / 256 : (a.G * M + GEN_ROWS - 1) / GEN_ROWS) : 0;
        r[3] = -1;
      }
      for (int k = 0; k < a.n_tbl; ++k) {  // work lists: the table's entries, found back by their first tree row
        const SeqEntry& e = a.tbl[k];
        for (int s = 0; s < B; ++s)
          if (host_node_offsets[s] == e.n0 && host_node_offsets[s + 1] - e.n0 == e.M && report->per_seq[4 * s + 3] < 0) {
            int32_t* r = report->per_seq + 4 * s;
            r[0] = e.n_sp; r[1] = e.tiles_per_split; r[2] = e.n_rg; r[3] = e.first_item;
            break;
          }
      }
    }
    return HS_OK;
  }
  HS_REQUIRE(need == 0 || (workspace && workspace_bytes >= need && reinterpret_cast<uintptr_t>(workspace) % 256 == 0),
             HS_ERR_WORKSPACE, "hs_tree_attention: workspace needs %zu bytes, 256-byte aligned (got %zu)", need,
             workspace_bytes);

  if (mfma) {
    hs_status r = attn_mfma_launch(a, max_M, st, ev_start, ev_stop);
    if (r != HS_OK) return r;
    last_kernel = 1;
  } else {
    dim3 grid((unsigned)(Hkv * plan.n_rb_max * plan.sp_max), (unsigned)B);
    const bool few = generic_short(std::min(plan.max_L, (int64_t)plan.split_len), max_M, D);
#define GEN_LAUNCH(T, D)                                                                                             \
  do {                                                                                                               \
    if (few) hipLaunchKernelGGL((k_attn_generic<T, D, true>), grid, dim3(GEN_THREADS), 0, st, a);                     \
    else hipLaunchKernelGGL((k_attn_generic<T, D, false>), grid, dim3(GEN_THREADS), 0, st, a);                        \
  } while (0)
    if (dt == HS_F32 && D == 64) GEN_LAUNCH(float, 64);
    else if (dt == HS_F32) GEN_LAUNCH(float, 128);
    else if (D == 64) GEN_LAUNCH(bf16_t, 64);
    else GEN_LAUNCH(bf16_t, 128);
#undef GEN_LAUNCH
    hs_status r = launch_status("tree attention");
    if (r != HS_OK) return r;
    last_kernel = 2;
  }
  if (a.sp_max > 1) {
    const int units = std::min(a.Hkv, CMB_UNITS);
    const int rows = (a.Hkv + CMB_UNITS - 1) / CMB_UNITS * a.G;  // of a workgroup
    dim3 grid((unsigned)(NN - a.cmb_row0) * units), block((unsigned)std::min((rows * (D / 4) + 63) / 64 * 64, CMB_THREADS));
    if (dt == HS_F32 && D == 64) hipLaunchKernelGGL((k_attn_combine<float, 64>), grid, block, 0, st, a);
    else if (dt == HS_F32) hipLaunchKernelGGL((k_attn_combine<float, 128>), grid, block, 0, st, a);
    else if (D == 64) hipLaunchKernelGGL((k_attn_combine<bf16_t, 64>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_attn_combine<bf16_t, 128>), grid, block, 0, st, a);
    return launch_status("tree attention combine");
  }
  return HS_OK;
}

extern "C" hs_status hs_tree_attention_lens(const void* q, const void* k_prefix, const void* v_prefix,
                                            const void* k_tree, const void* v_tree, const int32_t* parent,
                                            const int32_t* node_offsets, const int64_t* prefix_offsets,
                                            const int32_t* host_node_offsets, const int64_t* host_prefix_offsets,
                                            const int64_t* prefix_lens, const int64_t* host_prefix_lens, int32_t B,
                                            int32_t Hq, int32_t Hkv, int32_t D, hs_dtype dt, float scale, void* o,
                                            float* lse, void* workspace, size_t workspace_bytes, hs_stream stream) {
  clear_error();
  return attention_impl(q, k_prefix, v_prefix, k_tree, v_tree, parent, node_offsets, prefix_offsets, host_node_offsets,
                        host_prefix_offsets, prefix_lens, host_prefix_lens, nullptr, 0, B, Hq, Hkv, D, dt, scale, o, lse,
                        workspace, workspace_bytes, stream);
}

extern "C" hs_status hs_tree_attention_shared_tree(const void* q, const void* k_prefix, const void* v_prefix,
                                                   const void* k_tree, const void* v_tree, const int32_t* parent,
                                                   const int32_t* node_offsets, const int64_t* prefix_offsets,
                                                   const int32_t* host_node_offsets,
                                                   const int64_t* host_prefix_offsets, int32_t B, int32_t Hq,
                                                   int32_t Hkv, int32_t D, hs_dtype dt, float scale, void* o, float* lse,
                                                   void* workspace, size_t workspace_bytes, hs_stream stream) {
  clear_error();
  if (B > 0 && host_node_offsets != nullptr) {
    const int M = host_node_offsets[1] - host_node_offsets[0];
    for (int s = 1; s < B; ++s)
      HS_REQUIRE(host_node_offsets[s + 1] - host_node_offsets[s] == M, HS_ERR_SHAPE,
                 "hs_tree_attention_shared_tree: entry %d has %d rows, entry 0 has %d", s,
                 host_node_offsets[s + 1] - host_node_offsets[s], M);
  }
  return attention_impl(q, k_prefix, v_prefix, k_tree, v_tree, parent, node_offsets, prefix_offsets, host_node_offsets,
                        host_prefix_offsets, nullptr, nullptr, nullptr, 0, B, Hq, Hkv, D, dt, scale, o, lse, workspace,
                        workspace_bytes, stream, true);
}

extern "C" hs_status hs_tree_attention_paged(const void* q, const void* k_pages, const void* v_pages,
                                             const void* k_tree, const void* v_tree, const int32_t* parent,
                                             const int32_t* node_offsets, const int32_t* host_node_offsets,
                                             const int32_t* block_table, int32_t max_blocks, int32_t page_tokens,
                                             const int64_t* prefix_lens, const int64_t* host_prefix_lens, int32_t B,
                                             int32_t Hq, int32_t Hkv, int32_t D, hs_dtype dt, float scale, void* o,
                                             float* lse, void* workspace, size_t workspace_bytes, hs_stream stream) {
  clear_error();
  HS_REQUIRE(page_tokens == 64, HS_ERR_UNSUPPORTED, "hs_tree_attention_paged: page_tokens=%d (pages of 64 tokens are built)",
             page_tokens);
  HS_REQUIRE(B == 0 || block_table, HS_ERR_NULL, "hs_tree_attention_paged: NULL block_table");
  return attention_impl(q, k_pages, v_pages, k_tree, v_tree, parent, node_offsets, nullptr, host_node_offsets, nullptr,
                        prefix_lens, host_prefix_lens, block_table, max_blocks, B, Hq, Hkv, D, dt, scale, o, lse,
                        workspace, workspace_bytes, stream);
}

extern "C" hs_status hs_tree_attention_plan(const int32_t* host_node_offsets, const int64_t* host_prefix_offsets,
                                            const int64_t* host_prefix_lens, int32_t paged, int32_t max_blocks,
                                            int32_t B, int32_t Hq, int32_t Hkv, int32_t D, hs_dtype dt,
                                            int64_t* totals, int32_t* per_seq) {
  clear_error();
  HS_REQUIRE(totals != nullptr, HS_ERR_NULL, "hs_tree_attention_plan: NULL totals");
  const PlanReport report{totals, per_seq};
  static const int32_t no_table = 0;  // (paged calls are told apart by their block table; none is read on the host)
  return attention_impl(nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, host_node_offsets,
                        paged ? nullptr : host_prefix_offsets, nullptr, host_prefix_lens, paged ? &no_table : nullptr,
                        max_blocks, B, Hq, Hkv, D, dt, 1.0f, nullptr, nullptr, nullptr, 0, nullptr, false, &report);
}
