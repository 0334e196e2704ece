// hs_draft_entropy_topk: one streaming pass over float32 logits rows.
//
// Computes, per row, the softmax statistics (max, sum of exponentials, entropy numerator) and the
// K best (logit, index) pairs (Section 4.1, Eq. 1; Section 2.2 Expansion).  HBM-bound: 4 bytes per
// logit, read once.
//
// One workgroup (four or sixteen waves, see below) scans a row (k_scan_rows), merges its waves'
// results and writes the outputs.  Only when there are too few rows to fill the chip is a row cut
// into slices for several workgroups; a small second kernel then merges the slices
// (k_scan_finalize).
//
// Top-K selection never sorts the data.  Each wave keeps its K best pairs as a sorted list in
// registers, entry l in lane l, a pair being one 64-bit key.  Per tile only the lanes that hold a value
// not worse than the list's K-th entry are looked at: they put their values into LDS, which are taken up 64 at
// a time, one to a lane; those that beat the K-th entry are broadcast and inserted one by one: the lanes
// whose entry it beats take their left neighbour's entry (or the new one), a shift by one lane done
// with a DPP move.  Before a list is full the threshold comes from the first tile: the K-th largest
// of the workgroup's wave maxima (of its 16-lane row maxima when it has fewer waves than K, of a
// wave's 64 lane maxima when even those are too few): K elements reach it, so no
// true Top-K member is ever filtered out, and only about K elements of the whole tile pass it.
// All decisions compare raw float32 logits under the strict order (value descending, index
// ascending), so the indices do not depend on how rows are split or reduced.
#include <limits.h>
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "hs_common.h"

namespace hs {

// The row scan is built for two workgroup sizes.  Sixteen waves: fewest slices to merge, best for a few
// dozen rows.  Four waves, several workgroups per compute unit: the workgroups' set-up, merge and
// write-out phases overlap with other workgroups' streaming, best for many rows (and for very few,
// where a row is cut into many short slices anyway).
constexpr int SCAN_BIG = 1024, SCAN_SMALL = 256;
constexpr int SCAN_VPT = 16;                        // values per thread per tile (4 x float4)
constexpr int scan_tile(int threads) { return threads * SCAN_VPT; }  // logits per workgroup tile
constexpr int FIN_THREADS = 256;
constexpr int FIN_CAP = HS_MAX_TOPK * HS_MAX_TOPK;  // candidates the merge of 64 slices can face
constexpr int SCAN_NBUF = 3;                         // register buffers: tiles that a workgroup has in hand or in flight
constexpr int MAX_SPLITS = 64;                       // slices per row (one list head per lane)
constexpr int SCAN_BIG_WGS = 256;                    // rows are sliced until about so many sixteen-wave workgroups exist ...
constexpr int SCAN_FINE_WGS = 600;                   // ... or four-wave ones (where they are: see plan_scan)
constexpr int SCAN_CUT_WGS = 1024;                   // ... of more than 256 rows
constexpr int64_t SCAN_STREAM = 5 << 21;             // logits of a call (42 MB) from which its loads carry the non-temporal hint
constexpr float LOG2E = 1.4426950408889634f;

struct ScanPlan {
  int threads;       // workgroup size
  int splits;        // workgroups per row
  int tiles_per_wg;  // tiles each of them scans
};

// Cold inputs, K = 10, microseconds a call, best slicing of sixteen / four waves:
//   17 rows of 8193  10.5 / 11.0    97 of 32000 13.6 / 15.5    66 of 128256 21.5 / 21.8   200 of 128256 27.4 / 31.1
//   17 rows of 8000   9.5 /  9.5   256 of 32000 16.2 / 18.9   280 of 128256 48.7 / 40.3   600 of   8193 25.9 / 17.2
// From 257 rows on sixteen-wave workgroups need a second round; rows of one small tile would leave most of sixteen
// waves without a value (17 rows of 1000: 12.1 / 7.9), and so would rows of two, but the first threshold of four waves
// comes from 16 groups only (40 rows of 8000, K = 40: 15.8 / 20.4).
// Slices: 256 workgroups of sixteen waves (97 rows of 100000: 1 slice 21.6, 2 24.1, 3 28.3; 66 of 128256: 24.2, 23.3,
// 21.5); for more than 256 rows none, or two of many tiles (300 of 50257: 1 slice 32.9, 2 34.7; 300 of 151936, merged by the
// scan's launch: 43.9 and 41.1; 400 of 128256 42.4 and 50.3); for up to 16 rows as many as there are tiles, but a
// merge of more than 16 pays for the first few rows only (10 rows of 128256 in 16 slices 12.9, in 32 14.7; 1 row 12.1
// and 11.3), and one slice takes three tiles in the time of a merge (16 rows of 4097: 8.7 and 12.5, of 8000: 9.5
// and 10.9).
// `rows.sparse`: a good part of the rows will be left out (row_active), so that large scans have room for workgroups of
// four waves in more slices (61 rows and their 20 parents of 128256 logits, K = 1, the ratio rule's whole call: 67.8 us,
// 69.7 by the rule for full scans).
// Rows that are not 16-byte aligned were read a value at a time when these rules were made, which only more workgroups made up
// for; read 16 bytes at a time like the others they lose nothing by the finer slices (301 of 132058: 43.9 us, by the rule for aligned
// rows 52.2; 330 of 50257 23.4 both, 7 of 137847 11.8 and 12.2).  Aligned rows keep the coarser slices that they had; the finer ones have not been
// measured for them.  Slices whose
// merge is the caller's (rows.pairs_only) cost no launch.  So the argmax scan takes 257 rows and more in three slices,
// or two, as long as 1024 workgroups allow (277 rows of 50257: 1 slice 31.2, 2 28.7, 3 26.0; 305 of 187620, aligned: 57.1,
// 50.5, 48.9; aligned rows from about 360 on gain nothing, 421 to 520 of 32000 or 50256 would lose 3 %), three-tile
// rows in three slices (2 of 11379: 8.8, 7.0), and the full scan up to 341 long rows in three (301 of 132058: 70.8, 53.2;
// shorter ones break even) and up to 16 rows in up to 256 slices altogether (7 of 137847: 17.1 in 12 slices each, 15.0 in
// 34).
static ScanPlan plan_scan(int R, int V, int K, const ScanRows& rows) {
  ScanPlan p;
  const int small_tiles = (V + scan_tile(SCAN_SMALL) - 1) / scan_tile(SCAN_SMALL);
  const bool fine = rows.sparse && R <= SCAN_BIG_WGS && (int64_t)R * V > (8 << 20);
  p.threads = (R <= 16 || R > SCAN_BIG_WGS || small_tiles == 1 || (small_tiles == 2 && K <= 16) || fine) ? SCAN_SMALL : SCAN_BIG;
  const int tile = scan_tile(p.threads);
  const int n_tiles = (V + tile - 1) / tile;
  int want = 1;
  if (p.threads == SCAN_BIG) {
    want = SCAN_BIG_WGS / R;
  } else if (R <= 16) {
    if (n_tiles > (rows.pairs_only && !rows.aligned ? 1 : 3)) want = R <= 4 ? MAX_SPLITS : rows.pairs_only || rows.aligned ? 16 : SCAN_BIG_WGS / R;
  } else if (fine) {
    want = std::min(16, SCAN_FINE_WGS / R);
  } else if (R > SCAN_BIG_WGS) {
    const int cut = std::min(3, SCAN_CUT_WGS / R);  // (three up to 341 rows, two up to 512)
    if (rows.pairs_only && (cut == 3 || (n_tiles >= 24 && (!rows.aligned || R <= 360)))) want = cut;
    else if (!rows.aligned && !rows.sparse && cut == 3 && n_tiles >= 16) want = cut;
    else if (n_tiles >= 24 && R <= SCAN_FINE_WGS / 2) want = 2;
  }
  if (want > n_tiles) want = n_tiles;
  if (want < 1) want = 1;
  p.tiles_per_wg = (n_tiles + want - 1) / want;
  p.splits = (n_tiles + p.tiles_per_wg - 1) / p.tiles_per_wg;
  return p;
}

// Floats as unsigned numbers in the same order.
__device__ __forceinline__ unsigned ordered_bits(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v + 0.f);
  return u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
}
// Value of an ordered-float number (the upper half of a key); numbers below -inf's stand for -inf.
__device__ __forceinline__ float ordered_value(unsigned u) {
  return __builtin_bit_cast(float, max(u, 0x007fffffu) ^ ((u >> 31) ? 0x80000000u : 0xffffffffu));
}
// Lanes below this one in a mask.
__device__ __forceinline__ int lanes_below(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
}
// A pair as one unsigned number: larger key = better pair (larger value, then lower index); never 0.
// (-0 and +0 are the same value; NaN never gets here: it passes no comparison with a threshold.)
__device__ __forceinline__ unsigned long long pair_key(float v, int i) {
  return ((unsigned long long)ordered_bits(v) << 32) | (0xffffffffu - (unsigned)i);
}
// The pair of a key (0: an unused entry, worse than every pair).
__device__ __forceinline__ void pair_of(unsigned long long k, float& v, int& i) {
  v = ordered_value((unsigned)(k >> 32));
  i = k == 0ull ? INT_MAX : (int)(0xffffffffu - (unsigned)k);
}
// The key of lane l, in scalar registers.
__device__ __forceinline__ unsigned long long lane_key(unsigned long long k, int l) {
  return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(k >> 32), l) << 32) |
         (unsigned)__builtin_amdgcn_readlane((int)k, l);
}

// Rank of this lane's pair among the pairs of lanes 0 .. n-1 (number of them holding a better pair).
__device__ __forceinline__ int wave_rank(float v, int i, int n) {
  int r = 0;
  for (int l = 0; l < n; ++l) {
    float ov = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
    int oi = __builtin_amdgcn_readlane(i, l);
    r += better(ov, oi, v, i) ? 1 : 0;
  }
  return r;
}

// The K-th largest (K <= 16) of 16 values of which every row of 16 lanes holds a copy, in every lane.  The lanes of a row
// rotate (DPP), so there is no chain through scalar registers as in wave_rank.
template <int N>
__device__ __forceinline__ int row_rotated(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x120 + N, 0xf, 0xf, false);  // row_ror:N
}
template <int N = 1>
__device__ __forceinline__ void rank16(float v, int& above, int& not_below) {
  if constexpr (N < 16) {
    const float o = __builtin_bit_cast(float, row_rotated<N>(__builtin_bit_cast(int, v)));
    above += o > v ? 1 : 0;
    not_below += o >= v ? 1 : 0;
    rank16<N + 1>(v, above, not_below);
  }
}
__device__ __forceinline__ float kth_of_16(float v, int K) {
  int above = 0, not_below = 1;
  rank16(v, above, not_below);
  const unsigned long long who = __ballot(above < K && not_below >= K);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), __ffsll((long long)who) - 1));
}
// How many of the 16 keys of a lane's row (a copy in every row) are larger than the lane's.
template <int N = 1>
__device__ __forceinline__ int keys_above16(unsigned long long k) {
  if constexpr (N < 16) {
    const unsigned long long o = ((unsigned long long)(unsigned)row_rotated<N>((int)(k >> 32)) << 32) | (unsigned)row_rotated<N>((int)k);
    return (o > k ? 1 : 0) + keys_above16<N + 1>(k);
  } else {
    return 0;
  }
}

// Inserts the wave-uniform key x into the sorted list held one entry per lane (largest first).
__device__ __forceinline__ void list_insert(unsigned long long x, unsigned long long& list) {
  // the left neighbour's entry (lane 0: one that nothing beats)
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)list, 0x138, 0xf, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)(list >> 32), 0x138, 0xf, 0xf, false);
  const unsigned long long left = ((unsigned long long)hi << 32) | lo;
  list = x > list ? (x > left ? left : x) : list;
}

// Maximum of each row of 16 lanes; lane 15 of a row holds it.
__device__ __forceinline__ float row16_max(float x) {
  const int id = __builtin_bit_cast(int, -HS_INF);
#define HS_DPP_STEP(ctrl, banks) \
  x = fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(id, __builtin_bit_cast(int, x), ctrl, 0xf, banks, false)))
  HS_DPP_STEP(0x111, 0xf);  // row_shr:1
  HS_DPP_STEP(0x112, 0xf);  // row_shr:2
  HS_DPP_STEP(0x114, 0xe);  // row_shr:4
  HS_DPP_STEP(0x118, 0xc);  // row_shr:8
#undef HS_DPP_STEP
  return x;
}

// Statistics of a wave's 64 lanes in one: the common maximum first, then plain sums of the lanes'
// terms rescaled to it.  The lowest lane that holds the maximum keeps its own maximum's unit out of
// s1 (as each lane did for itself); for every other lane that unit is an ordinary term.
__device__ __forceinline__ Stats stats_wave_sum(Stats a, float inv_t) {
  const float m = wave_max(a.m);
  if (m == -HS_INF) return stats_empty();
  const int lane = threadIdx.x & 63;
  const int leader = __ffsll((long long)__ballot(a.m == m)) - 1;
  float cs = 0.f, ct = 0.f;
  if (a.m != -HS_INF) {
    const float d = (a.m - m) * inv_t;  // <= 0
    const float e = exp2_fast(d * 1.4426950408889634f);
    const float w = 1.f + a.s1;
    cs = lane == leader ? a.s1 : e * w;
    ct = e * (a.t + d * w);
  }
  return Stats{m, wave_sum(cs), wave_sum(ct)};
}

// Scratch of the merges (shared memory).
template <int CAP>
struct MergeScratch {
  __attribute__((aligned(16))) unsigned long long key[CAP];  // candidates (pair_key; 0: none)
  unsigned long long best[HS_MAX_TOPK];  // the K best of them, in order (0: fewer than K)
  int cnt;
  Stats total;
};

// A key that at least K entries of S <= 64 sorted lists reach, so that nothing below it is among the K best:
// with r = ceil(K / S), the ceil(K / r)-th largest of the lists' r-th entries (1, which every entry
// reaches, when fewer lists are that long).  `rth`: list s's r-th entry in lane s < S, 0 in the other lanes; up to 16 lists:
// list s's in lane s of every row of 16 lanes (list_lane).
__device__ __forceinline__ int threshold_depth(int S, int K) { return (K + S - 1) / S; }
__device__ __forceinline__ int list_lane(int S, int lane) { return S <= 16 ? lane & 15 : lane; }
__device__ __forceinline__ unsigned long long lists_threshold(unsigned long long rth, int S, int K) {
  const int r = threshold_depth(S, K), m = (K + r - 1) / r;
  int rank = 0;
  if (S <= 16) {
    rank = keys_above16(rth);
  } else {
    for (int l = 0; l < S; ++l) rank += lane_key(rth, l) > rth ? 1 : 0;
  }
  const unsigned long long who = __ballot(rank == m - 1 && rth != 0ull);
  return who != 0ull ? lane_key(rth, __ffsll((long long)who) - 1) : 1ull;
}

// Ranks the candidates sm.key[0, n) by counting (keys differ, zeros aside: ranks are a permutation) and
// leaves those of rank < K, in order, in sm.best (zero on entry).  A wave takes a run of candidates, one to a lane, and
// 64 opponents at a time, one to a lane: a candidate's key goes to a scalar register, one comparison and a count of the
// ballot's bits follow, and no step waits for LDS.  (A loop over LDS, one dependent read to an opponent, and counts
// added up by LDS atomics before: 8 us to 7.4 from a workgroup's start to its slice's result.)  Called by all
// `nthreads` threads; ends with a barrier.
template <int CAP>
__device__ __forceinline__ void rank_candidates(MergeScratch<CAP>& sm, int n, int K, int tid, int nthreads) {
  const int lane = tid & 63;
  const int n_waves = nthreads >> 6, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int per = (n + n_waves - 1) / n_waves;
  const int lo = wave * per, hi = min(n, lo + per);
  for (int c0 = lo; c0 < hi; c0 += 64) {  // one trip unless a wave has more than 64 candidates
    const unsigned long long mine = lane < hi - c0 ? sm.key[c0 + lane] : 0ull;
    const unsigned long long ranked = __ballot(mine != 0ull);
    if (ranked == 0ull) continue;
    int rank = 0;
    for (int o = 0; o < n; o += 64) {
      const unsigned long long opp = o + lane < n ? sm.key[o + lane] : 0ull;
      for (unsigned long long left = ranked; left != 0ull; left &= left - 1ull) {
        const int j = __ffsll((long long)left) - 1;
        const int above = __popcll(__ballot(opp > lane_key(mine, j)));
        rank += lane == j ? above : 0;
      }
    }
    if (mine != 0ull && rank < K) sm.best[rank] = mine;
  }
  __syncthreads();
}

// The same for n <= 64 candidates by one wave alone, a candidate to a lane: the opponents come as broadcast reads of LDS,
// eight requested together.  Leaves the K best in sm.best (zero on entry) for the same wave; no barrier.
template <int CAP>
__device__ __forceinline__ void rank_few(MergeScratch<CAP>& sm, int n, int K, int lane) {
  static_assert(CAP >= 72, "64 candidates and what fills the last eight");
  if (lane < 8) sm.key[n + lane] = 0ull;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  const unsigned long long mine = lane < n ? sm.key[lane] : 0ull;
  int rank = 0;
  for (int o = 0; o < n; o += 8) {
    ulonglong2 k[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) k[q] = reinterpret_cast<const ulonglong2*>(sm.key)[(o >> 1) + q];
#pragma unroll
    for (int q = 0; q < 4; ++q) rank += (k[q].x > mine ? 1 : 0) + (k[q].y > mine ? 1 : 0);
  }
  if (mine != 0ull && rank < K) sm.best[rank] = mine;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// The place of a wave's entry in the order of all lists of a workgroup of four waves, K <= 16 entries each, unused ones (0)
// last: its place in its own list, and what the other lists hold above it.  sm.key: wave w's list from 16 w on,
// filled up with zeros.
template <int PAIRS, int CAP>
__device__ __forceinline__ int place_of_four(const MergeScratch<CAP>& sm, unsigned long long mine, int wave, int lane) {
  int place = lane;
#pragma unroll
  for (int d = 1; d < 4; ++d) {
    const int w = (wave + d) & 3;
    const unsigned long long low = w < wave ? 1ull : 0ull;  // (equal, i.e. unused, entries: the lower wave's first)
    ulonglong2 k[PAIRS];
#pragma unroll
    for (int q = 0; q < PAIRS; ++q) k[q] = reinterpret_cast<const ulonglong2*>(sm.key)[w * 8 + q];
#pragma unroll
    for (int q = 0; q < PAIRS; ++q) place += (k[q].x + low > mine ? 1 : 0) + (k[q].y + low > mine ? 1 : 0);
  }
  return place;
}

// Merges S <= 64 slices of a row: statistics st[s] (m, s1, t) and sorted K-lists pk[s * K + k] of keys.
// COHERENT: the slices were written by other workgroups of the same launch (ld_dev).
// Leaves the row's statistics in sm.total and its K best pairs, in order, in sm.best.
// sm.cnt and sm.best are zero and the workgroup has met a barrier since.  Called by all `nthreads` threads; the results
// are the first wave's (every wave's after a barrier).
// Everything the merge reads from memory is requested at once (one trip, which is most of its
// time when the slices come from other workgroups): the lists by all threads, their heads (fewer lists than K: their
// r-th entries) by every wave once more, the statistics by the last wave.  The heads give a threshold; only a few
// entries pass it, and those are ranked by counting, by the first wave if it can hold them.  (With a threshold for at
// least K lists only, one row of 128256 logits in 32 slices took 957 us for K = 64.  With the heads passed on
// through LDS and all waves ranking, three barriers instead of one, and a slice's own merge likewise: 10 rows of 128256 logits
// in 16 slices 13.0 us a launch, now 11.7; the ratio rule's 61 rows and 20 parents 17.8 and 16.8.)
template <bool COHERENT, int CAP>
__device__ __forceinline__ void merge_slices(const float4* st, const unsigned long long* pk, int S, int K, float inv_t,
                                             MergeScratch<CAP>& sm, int tid, int nthreads) {
  const int lane = tid & 63;
  constexpr int PER = 4;  // entries a thread keeps in registers (a trip covers PER x nthreads of the S x K)
  const int n_all = S * K;
  unsigned long long ek[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int e = tid + q * nthreads;
    ek[q] = 0ull;
    if (e < n_all) ek[q] = COHERENT ? ld_dev(pk + e) : pk[e];
  }
  unsigned long long rth = 0ull;
  if (list_lane(S, lane) < S) {
    const unsigned long long* e = pk + (int64_t)list_lane(S, lane) * K + threshold_depth(S, K) - 1;
    rth = COHERENT ? ld_dev(e) : *e;
  }
  Stats a = stats_empty();
  const bool stats_wave = tid >= nthreads - 64;
  if (stats_wave && lane < S) {
    if (COHERENT) {
      const float* sf = reinterpret_cast<const float*>(st + lane);
      a = Stats{ld_dev(sf), ld_dev(sf + 1), ld_dev(sf + 2)};
    } else {
      const float4 f = st[lane];
      a = Stats{f.x, f.y, f.z};
    }
  }
  const unsigned long long thr = lists_threshold(rth, S, K);
  // (order of arrival does not matter; at most S * K <= CAP entries)
  auto admit = [&](unsigned long long k) {
    const unsigned long long who = __ballot(k >= thr);
    if (who == 0ull) return;
    int base = 0;
    if (lane == 0) base = atomicAdd(&sm.cnt, __popcll(who));
    base = __builtin_amdgcn_readfirstlane(base);
    if (k >= thr) sm.key[base + lanes_below(who)] = k;
  };
#pragma unroll
  for (int q = 0; q < PER; ++q) admit(ek[q]);
  for (int e0 = PER * nthreads; e0 < n_all; e0 += nthreads) {  // (more entries than PER x nthreads: the rest)
    const int e = e0 + tid;
    admit(e < n_all ? (COHERENT ? ld_dev(pk + e) : pk[e]) : 0ull);
  }
  if (stats_wave) {
    a = stats_wave_sum(a, inv_t);
    if (lane == 0) sm.total = a;
  }
  __syncthreads();
  if (sm.cnt <= 64) {
    if (tid < 64) rank_few(sm, sm.cnt, K, lane);
  } else {
    rank_candidates(sm, sm.cnt, K, tid, nthreads);
  }
}

// Writes a row's results from its merged statistics and Top-K list (first wave of the workgroup).
template <int CAP>
__device__ __forceinline__ void write_row(const MergeScratch<CAP>& sm, int64_t row, int K, float inv_t,
                                          int32_t* __restrict__ topk_idx, float* __restrict__ topk_logp,
                                          float* __restrict__ ent_topk, float* __restrict__ ent_full,
                                          float* __restrict__ lse, int tid) {
  if (tid >= 64) return;
  const int lane = tid;
  const float m = sm.total.m, s1 = sm.total.s1, t = sm.total.t;
  const float l1p = log1pf(s1);
  float ov;
  int oi;
  pair_of(lane < K ? sm.best[lane] : 0ull, ov, oi);
  if (lane < K) {
    topk_idx[row * K + lane] = oi;
    topk_logp[row * K + lane] = (ov - m) * inv_t - l1p;
  }
  // Top-K probabilities renormalised over the K: weights relative to the best one (lane = entry);
  // entropy = ln(1 + sum w) - sum(w a) / (1 + sum w), every term of one sign
  const float best = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, ov)));
  float w = 0.f, wa = 0.f;
  if (lane >= 1 && lane < K) {
    const float a = (ov - best) * inv_t;
    if (a > -100.f) {
      w = expf(a);
      wa = w * a;
    }
  }
  w = wave_sum(w);
  wa = wave_sum(wa);
  if (lane == 0) {
    ent_topk[row] = log1pf(w) - wa / (1.f + w);
    if (ent_full) ent_full[row] = l1p - t / (1.f + s1);
    if (lse) lse[row] = m * inv_t + l1p;
  }
}

// grid (S, R): slice `blockIdx.x` of row `blockIdx.y`.  S == 1: the outputs are written here;
// S > 1: the slice's statistics and K-list go to part_* for k_scan_finalize, or, FUSED, for the
// workgroup that finishes a row's last slice: every workgroup draws a ticket from the row's counter
// (`tickets`, zero before the launch), the one that draws S - 1 knows that all slices are written,
// puts the counter back to zero for the next launch, merges the slices and writes the row.
constexpr int FUSED_CAP = 1024;  // slices x K that the merging workgroup's scratch holds
constexpr size_t TICKET_BYTES = 65536 * sizeof(unsigned);  // a counter for each of the at most ROW_SCAN_MAX rows of a call
static_assert(ROW_SCAN_MAX * sizeof(unsigned) <= TICKET_BYTES, "every row has its counter");
// STATS false: only the K best pairs are wanted (the greedy accept walk's argmax scan); the softmax
// statistics, most of the arithmetic of a tile, are left out and part_stats is not written.
// STREAM: the whole tiles' loads carry the non-temporal hint (see row_topk_launch).
// SHORT: a workgroup has at most NBUF tiles, and the loops for more are left out: such launches wait for their instructions, and
// the fewer lie between those they need the better (the loops in all launches: 10 rows of 128256 logits 10.98 us, now 10.74, 61 rows 17.3 and
// 16.8, one of 8000 7.7 and 7.2; the 8B drafting half 91.9 and 90.0.  The second and third tile by one copy of the code, moved to its registers:
// 10.9 and 17.3, as the copy waits for the third tile's loads).
template <int SCAN_THREADS, bool FUSED, int NBUF, bool STATS, bool STREAM, bool SHORT>
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_rows(const float* __restrict__ logits, int64_t row_stride,
                                                            int V, int K, float inv_t, int tiles_per_wg,
                                                            float4* __restrict__ part_stats,
                                                            unsigned long long* __restrict__ part_key,
                                                            int32_t* __restrict__ topk_idx,
                                                            float* __restrict__ topk_logp,
                                                            float* __restrict__ ent_topk,
                                                            float* __restrict__ ent_full, float* __restrict__ lse,
                                                            const uint8_t* __restrict__ row_active,
                                                            const int32_t* __restrict__ row_index,
                                                            const float* __restrict__ logits2, int rows1,
                                                            unsigned* __restrict__ tickets) {
  // (all arguments in one batch: left to itself the compiler fetches each where it is first used, six trips one after the
  // other: 10 rows of 128256 logits 11.2 us a launch and 10.9 so, 61 rows 17.7 and 17.3, one of 32000 8.7 and 8.2, 97 of 32000 13.2 and 12.7)
  asm volatile("" ::"s"(logits), "s"(row_stride), "s"(V), "s"(K), "s"(inv_t), "s"(tiles_per_wg), "s"(part_stats), "s"(part_key),
               "s"(topk_idx), "s"(topk_logp), "s"(ent_topk), "s"(ent_full), "s"(lse), "s"(row_active), "s"(row_index),
               "s"(logits2), "s"(rows1), "s"(tickets));
  if (row_active != nullptr && row_active[blockIdx.y] == 0) return;  // (the whole workgroup: a row nobody will read)
  // (both arms as int64: mixed with the unsigned block index a negative entry would turn positive)
  const int64_t src_row = row_index != nullptr ? (int64_t)__builtin_amdgcn_readfirstlane(row_index[blockIdx.y]) : (int64_t)blockIdx.y;
  if (src_row < 0) return;
  constexpr int SCAN_WAVES = SCAN_THREADS / 64;
  constexpr int SCAN_GROUPS = SCAN_WAVES * 4 < 64 ? SCAN_WAVES * 4 : 64;  // rows of 16 lanes, at most one per lane
  constexpr int SCAN_TILE = scan_tile(SCAN_THREADS);
  // candidates the merge of the waves can face (and, FUSED, the merge of a row's slices)
  constexpr int SCAN_CAP = (FUSED && SCAN_WAVES * HS_MAX_TOPK < FUSED_CAP) ? FUSED_CAP : SCAN_WAVES * HS_MAX_TOPK;
  __shared__ float4 wave_st[SCAN_WAVES];
  __shared__ float group_maxima[SCAN_GROUPS];
  __shared__ __attribute__((aligned(16))) float lane_vals[SCAN_WAVES][64 * SCAN_VPT];  // values of the lanes that reach the threshold
  __shared__ int lane_ids[SCAN_WAVES][64];
  __shared__ MergeScratch<SCAN_CAP> sm;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (uniform for the compiler too)
  const int split = blockIdx.x, S = gridDim.x, row = blockIdx.y;
  // (rows from rows1 on may lie in a second array)
  const float* __restrict__ x = (logits2 != nullptr && src_row >= rows1) ? logits2 + (src_row - rows1) * row_stride
                                                                         : logits + src_row * row_stride;

  // this wave's K best pairs so far, best first, entry l in lane l as a key (0: none yet); `floor_key` is
  // what a pair has to beat to join them, `thr` what its value has to reach
  unsigned long long best = 0ull, floor_key = 0ull;
  float thr = -HS_INF;
  // Statistics in the log2 domain, y = (x - ref) * c with c = log2(e) / T, relative to the maximum of all the
  // values this wave has seen: s1 and t2 are this lane's sums of 2^y and 2^y y over its values, one
  // instance of the maximum held out of them.
  const float c = inv_t * LOG2E;
  float ref = -HS_INF, s1 = 0.f, t2 = 0.f;
  bool masked = false;  // a masked logit has been met: the wave's sums are clamped from there on
  if (tid < HS_MAX_TOPK) sm.best[tid] = 0ull;  // (a slice with fewer than K elements leaves the rest unused)
  if (tid == 0) sm.cnt = 0;

  auto load_tile = [&](int tile, float (&v)[SCAN_VPT]) {
    const int tbase = (split * tiles_per_wg + tile) * SCAN_TILE;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i0 = tbase + (j * SCAN_THREADS + tid) * 4;
      if (i0 + 3 < V) {
        const float4 f = load_float4(x + i0);
        v[j * 4 + 0] = f.x;
        v[j * 4 + 1] = f.y;
        v[j * 4 + 2] = f.z;
        v[j * 4 + 3] = f.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j * 4 + e] = (i0 + e < V) ? x[i0 + e] : -HS_INF;
      }
    }
  };
  // a tile that lies inside the row as a whole: four loads, no conditions, so the
  // compiler can count them when it waits for an older tile
  auto load_full_tile = [&](int tile, float (&v)[SCAN_VPT]) {
    const float* __restrict__ src = x + (int64_t)(split * tiles_per_wg + tile) * SCAN_TILE + tid * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4 f = STREAM ? stream_float4(src + j * SCAN_THREADS * 4) : load_float4(src + j * SCAN_THREADS * 4);
      v[j * 4 + 0] = f.x;
      v[j * 4 + 1] = f.y;
      v[j * 4 + 2] = f.z;
      v[j * 4 + 3] = f.w;
    }
  };
  // tiles this workgroup really has (uniform)
  int n_my = (V - split * tiles_per_wg * SCAN_TILE + SCAN_TILE - 1) / SCAN_TILE;
  n_my = n_my < 0 ? 0 : (n_my > tiles_per_wg ? tiles_per_wg : n_my);
  int n_full = (V - split * tiles_per_wg * SCAN_TILE) / SCAN_TILE;  // leading whole tiles
  n_full = n_full < 0 ? 0 : (n_full > n_my ? n_my : n_full);

  // One tile: statistics of this thread's 16 values, threshold, insertion of the few values that
  // reach it.  The arithmetic of the statistics bounds the scan of many rows, so the tile without a new
  // maximum, nearly every one, does five instructions to a value and no more.  (With the maximum held out
  // per lane every tile searched for it and paid eight: one four-wave workgroup scanned a row of 128256
  // logits in 38.9 us, now 28.6; 896 rows took 98.8 us, now 92.5, which is 5 TB/s.)
  auto process = [&](const float (&v)[SCAN_VPT], int tile, auto is_first) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(is_first)::value;
    const int tbase = (split * tiles_per_wg + tile) * SCAN_TILE;

    float tm = fmaxf(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])), fmaxf(fmaxf(v[4], v[5]), fmaxf(v[6], v[7])));
    tm = fmaxf(tm, fmaxf(fmaxf(fmaxf(v[8], v[9]), fmaxf(v[10], v[11])), fmaxf(fmaxf(v[12], v[13]), fmaxf(v[14], v[15]))));
    if (STATS) {
      float st = 0.f, tt = 0.f;  // the tile's sums
      if (FIRST || __ballot(tm > ref) != 0ull) {
        // a new maximum (FIRST: or no value at all): the sums so far move to it, the old one joins them
        const float wm = wave_max(tm);
        if (wm != -HS_INF) {
          const int leader = __ffsll((long long)__ballot(tm == wm)) - 1;
          if (!FIRST && ref != -HS_INF) {
            const float d2 = (ref - wm) * c;
            const float e = exp2_fast(d2);
            const float w = s1 + (lane == leader ? 1.f : 0.f);
            t2 = e * (t2 + d2 * w);
            s1 = e * w;
          }
          ref = wm;
          int skip = -1;  // the instance that is held out: the leader's first
          if (lane == leader) {
#pragma unroll
            for (int jj = SCAN_VPT - 1; jj >= 0; --jj) skip = (v[jj] == wm) ? jj : skip;
          }
#pragma unroll
          for (int jj = 0; jj < SCAN_VPT; ++jj) {
            // x - ref first: exact near the maximum (an fma with a rounded ref * c would leave the maximum's
            // own y slightly off zero and put that into t2); the clamp keeps 0 * -inf out of t2
            const float y = fmaxf((v[jj] - ref) * c, -1e30f);
            const float e = exp2_fast(y);
            tt = fmaf(e, y, tt);
            st += (jj == skip) ? 0.f : e;
          }
        }
      } else if (ref != -HS_INF) {
        auto sums = [&](auto clamped) {
          st = 0.f;
          tt = 0.f;
#pragma unroll
          for (int jj = 0; jj < SCAN_VPT; ++jj) {
            const float x = (v[jj] - ref) * c;
            const float y = decltype(clamped)::value ? fmaxf(x, -1e30f) : x;
            const float e = exp2_fast(y);
            tt = fmaf(e, y, tt);
            st += e;
          }
        };
        if (!masked) {
          sums(std::false_type{});
          masked = __ballot(!(tt == tt)) != 0ull;  // masked logits among them (0 * -inf)
        }
        if (masked) {
          if (__ballot(tm != -HS_INF) != 0ull) {
            sums(std::true_type{});
          } else {
            st = 0.f;
            tt = 0.f;
          }
        }
      }
      s1 += st;
      t2 += tt;
    }

    // ---- threshold (a value): no element below it can be among the row's K best.  First tile:
    // the K-th largest of the workgroup's group maxima (K elements of the tile reach it), or of
    // this wave's 64 lane maxima; afterwards also the wave's own K-th entry once its list is full.
    if (FIRST) {
      // Groups that hold no value of the row have no maximum: counting them, the K-th largest of the
      // maxima would be -inf and every value of a short row would be inserted one by one (17 rows of
      // 1024 logits: 26.8 us that way; of 1000 without the empty groups 12.1, in workgroups of four waves 7.9).
      const int n_here = min(V - tbase, SCAN_TILE);  // the tile's values; 4 neighbouring ones to a thread
      const int waves_here = min((n_here + 255) >> 8, SCAN_WAVES), groups_here = min((n_here + 63) >> 6, SCAN_GROUPS);
      if (K <= groups_here) {
        // maxima of the waves, or of their rows of 16 lanes when fewer waves than K hold values
        const bool by_wave = K <= waves_here;
        const int n_groups = by_wave ? SCAN_WAVES : SCAN_GROUPS;
        if (by_wave) {
          const float wm = wave_max(tm);
          if (lane == 0) group_maxima[wave] = wm;
        } else {
          const float rm = row16_max(tm);
          if ((lane & 15) == 15) group_maxima[wave * 4 + (lane >> 4)] = rm;
        }
        // an exchange through LDS only: the barrier must not wait for the next tiles' loads
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (n_groups == 16) {
          thr = kth_of_16(group_maxima[lane & 15], K);
        } else {
          const float mine = lane < n_groups ? group_maxima[lane] : -HS_INF;
          const int r = wave_rank(mine, lane, n_groups);
          const unsigned long long who = __ballot(r == K - 1 && lane < n_groups);
          thr = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mine), __ffsll((long long)who) - 1));
        }
      } else {
        const int r = wave_rank(tm, lane, 64);
        const unsigned long long who = __ballot(r == K - 1);
        thr = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, tm), __ffsll((long long)who) - 1));
      }
    }

    // ---- insert the elements that reach the threshold.  A lane whose maximum does puts its 16 values into
    // LDS; 64 of them at a time, one to a lane, are then compared with the list's worst entry, and what
    // beats it is inserted.  That entry is a pair: of equal values only lower indices beat it, or rows of
    // equal logits would send every element through the insertion.  (One copy of the insertion for the whole
    // tile, not one for each register: short scans wait for their instructions more than for anything else, 10
    // rows of 128256 logits in 16 slices 13.9 us to 12.9.)
    const unsigned long long lanes = __ballot(tm >= thr);
    if (lanes != 0ull) {
      float* const vals = lane_vals[wave];
      if (tm >= thr) {
        const int at = lanes_below(lanes);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<float4*>(vals + at * SCAN_VPT + j * 4) = make_float4(v[j * 4], v[j * 4 + 1], v[j * 4 + 2], v[j * 4 + 3]);
        lane_ids[wave][at] = lane;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (other lanes' values; LDS keeps a wave's order)
      const int n = __popcll(lanes) * SCAN_VPT;
      for (int e0 = 0; e0 < n; e0 += 64) {
        unsigned long long key = 0ull;
        if (e0 + lane < n) {
          const float x = vals[e0 + lane];
          const int jj = lane & (SCAN_VPT - 1), from = lane_ids[wave][(e0 + lane) / SCAN_VPT];
          const int idx = tbase + (((jj >> 2) * SCAN_THREADS) + wave * 64 + from) * 4 + (jj & 3);
          // (rows end inside a tile: what lies past the end is no value)
          if (x >= thr && idx < V) key = pair_key(x, idx);
        }
        for (unsigned long long todo = __ballot(key > floor_key); todo != 0ull; todo &= __ballot(key > floor_key)) {
          const int src = __ffsll((long long)todo) - 1;
          todo &= todo - 1ull;
          list_insert(lane_key(key, src), best);
          floor_key = lane_key(best, K - 1);  // (0 while the list is not full)
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (floor_key != 0ull) thr = fmaxf(thr, ordered_value((unsigned)(floor_key >> 32)));
    }
  };
  // NBUF register buffers, NBUF - 1 tiles in flight: the loads of tile t + NBUF - 1 are requested
  // before tile t is processed (what is in flight bounds the bandwidth).  The steady-state loop
  // requests without a condition, so that the wait before a tile's values counts exactly the younger
  // tiles; the last tiles run through the guarded copy below.
  float buf[NBUF][SCAN_VPT];
  const std::true_type YES{};
  const std::false_type NO{};
  int tile = 1;
  if (!SHORT && n_full >= 2 * NBUF) {
    // (requested without a condition as well: a wait counts only loads that are pending on every path to it)
#pragma unroll
    for (int b = 0; b < NBUF; ++b) load_full_tile(b, buf[b]);
    process(buf[0], 0, YES);
    for (; tile + 2 * NBUF - 2 < n_full; tile += NBUF) {
#pragma unroll
      for (int b = 0; b < NBUF; ++b) {
        load_full_tile(tile + b + NBUF - 1, buf[b]);
        process(buf[(b + 1) % NBUF], tile + b, NO);
      }
    }
  } else {
    // (whole tiles by the unconditional loads: the guarded ones wait for each other)
#pragma unroll
    for (int b = 0; b < NBUF; ++b) {
      if (b < n_full) load_full_tile(b, buf[b]);
      else if (b < n_my) load_tile(b, buf[b]);
    }
    if (n_my > 0) process(buf[0], 0, YES);
  }
  if constexpr (SHORT) {
#pragma unroll
    for (int b = 1; b < NBUF; ++b)
      if (b < n_my) process(buf[b], b, NO);
  }
  for (; !SHORT && tile < n_my; tile += NBUF) {
#pragma unroll
    for (int b = 0; b < NBUF; ++b) {
      if (tile + b < n_my) {
        if (tile + b + NBUF - 1 < n_my) load_tile(tile + b + NBUF - 1, buf[b]);
        process(buf[(b + 1) % NBUF], tile + b, NO);
      }
    }
  }

  // ---- the waves' statistics and the real entries of their lists meet in LDS
  if (STATS) {
    // (the maximum is the whole wave's: plain sums; t back in natural-log units)
    const float ws = wave_sum(s1), wt = wave_sum(t2);
    if (lane == 0) wave_st[wave] = make_float4(ref, ws, wt * 0.6931471805599453f, 0.f);
  }
  static_assert(STATS || !FUSED, "rows are finished by the caller of a scan without statistics");
  // What becomes of the slice's k-th best pair: kept for write_row when the row is one slice, else handed on.
  const int64_t slot = (int64_t)row * S + split;
  auto put = [&](int k, unsigned long long key) {
    if (S == 1) {
      if (STATS) sm.best[k] = key;
      else if (key != 0ull) topk_idx[row * K + k] = (int)(0xffffffffu - (unsigned)key);
      else topk_idx[row * K + k] = INT_MAX;
    } else if (FUSED) {
      st_dev(part_key + slot * K + k, key);  // (a store that the other XCDs see)
    } else {
      part_key[slot * K + k] = key;
    }
  };
  // The workgroup's statistics, by its first wave (after the barrier that publishes wave_st).
  auto put_stats = [&]() {
    Stats a = stats_empty();
    if (lane < SCAN_WAVES) {
      const float4 f = wave_st[lane];
      a = Stats{f.x, f.y, f.z};
    }
    a = stats_wave_sum(a, inv_t);
    if (S == 1) {
      if (lane == 0) sm.total = a;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    } else if (FUSED) {
      if (lane < 3) st_dev(reinterpret_cast<float*>(part_stats + slot) + lane, lane == 0 ? a.m : lane == 1 ? a.s1 : a.t);
    } else {
      if (lane == 0) part_stats[slot] = make_float4(a.m, a.s1, a.t, 0.f);
    }
  };
  // Lists that fit one wave of opponents: every wave finds the places of its own entries and hands them on itself (see
  // merge_slices).  Of longer ones only the entries that reach a
  // threshold join, a wave's in one piece (ranked whole, or with the threshold but from the lists' places, K = 40: 40 rows of
  // 16384 logits 49 and 21 us, 15 now; 200 rows 51 and 23, 17 now).
  __shared__ unsigned long long rth[SCAN_WAVES];
  const bool whole = SCAN_WAVES * K <= 64;
  if (SCAN_WAVES == 4 && whole) {
    if (lane < 16) sm.key[wave * 16 + lane] = lane < K ? best : 0ull;
    __syncthreads();
    const int place = K <= 4 ? place_of_four<2>(sm, best, wave, lane) : K <= 10 ? place_of_four<5>(sm, best, wave, lane) : place_of_four<8>(sm, best, wave, lane);
    if (lane < K && place < K) put(place, best);
    if (STATS && wave == 0) put_stats();
    if (S == 1) {
      if (!STATS) return;
      __syncthreads();
      write_row(sm, row, K, inv_t, topk_idx, topk_logp, ent_topk, ent_full, lse, tid);
      return;
    }
  } else {
    if (whole) {
      if (lane < K) sm.key[wave * K + lane] = best;
    } else if (lane == threshold_depth(SCAN_WAVES, K) - 1) {
      rth[wave] = best;
    }
    __syncthreads();
    if (!whole) {
      const int l = list_lane(SCAN_WAVES, lane);
      const unsigned long long list_thr = lists_threshold(l < SCAN_WAVES ? rth[l] : 0ull, SCAN_WAVES, K);
      const bool joins = lane < K && best >= list_thr;  // (a list's first entries)
      const int n_joins = __popcll(__ballot(joins));
      int base = 0;
      if (lane == 0) base = atomicAdd(&sm.cnt, n_joins);
      base = __builtin_amdgcn_readfirstlane(base);
      if (joins) sm.key[base + lane] = best;
      __syncthreads();
    }
    const int n = whole ? SCAN_WAVES * K : sm.cnt;
    if (n <= 64) {  // (by the first wave alone: the others only wait to be told whether to merge)
      if (tid < 64) rank_few(sm, n, K, lane);
    } else {
      rank_candidates(sm, n, K, tid, SCAN_THREADS);
    }
    if (tid < 64) {
      if (STATS) put_stats();
      if (!(S == 1 && STATS) && lane < K) put(lane, sm.best[lane]);
      if (S == 1) {
        if (STATS) write_row(sm, row, K, inv_t, topk_idx, topk_logp, ent_topk, ent_full, lse, tid);
      } else if (FUSED) {  // (for the merge of the slices)
        sm.best[lane] = 0ull;
        if (lane == 0) sm.cnt = 0;
      }
    }
    if (S == 1) return;
  }
  if (FUSED) {
    __shared__ int is_last;
    // Once the slice's results are acknowledged (each wave waits for its own stores) the ticket is drawn.  The workgroup
    // that draws the last one finds every slice of the row written.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      const unsigned drawn = __hip_atomic_fetch_add(&tickets[row], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      is_last = drawn == (unsigned)(S - 1) ? 1 : 0;
      // (nobody else touches this row's counter any more: back to zero for the next launch)
      if (is_last) __hip_atomic_store(&tickets[row], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (is_last) {
      merge_slices<true>(part_stats + (int64_t)row * S, part_key + (int64_t)row * S * K, S, K, inv_t, sm, tid, SCAN_THREADS);
      write_row(sm, row, K, inv_t, topk_idx, topk_logp, ent_topk, ent_full, lse, tid);
    }
  }
}

// Clears a workspace (hs_workspace_prepare): a fill kernel, not a memset, so that it may be captured.
__global__ __launch_bounds__(256) void k_fill_zero(uint4* __restrict__ p, size_t n16) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(FIN_THREADS) void k_scan_finalize(const float4* __restrict__ part_stats,
                                                               const unsigned long long* __restrict__ part_key, int S, int K,
                                                               float inv_t, int32_t* __restrict__ topk_idx,
                                                               float* __restrict__ topk_logp,
                                                               float* __restrict__ ent_topk,
                                                               float* __restrict__ ent_full,
                                                               float* __restrict__ lse,
                                                               const uint8_t* __restrict__ row_active,
                                                               const int32_t* __restrict__ row_index) {
  __shared__ MergeScratch<FIN_CAP> sm;
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  if (row_active != nullptr && row_active[row] == 0) return;
  if (row_index != nullptr && row_index[row] < 0) return;
  if (tid < HS_MAX_TOPK) sm.best[tid] = 0ull;
  if (tid == 0) sm.cnt = 0;
  __syncthreads();
  merge_slices<false>(part_stats + row * S, part_key + row * S * K, S, K, inv_t, sm, tid, FIN_THREADS);
  write_row(sm, row, K, inv_t, topk_idx, topk_logp, ent_topk, ent_full, lse, tid);
}

// Bytes for the slices' results of a call.
static size_t slots_bytes(size_t n, int K) {
  return TICKET_BYTES + align_up(n * sizeof(float4), 256) + align_up(n * K * sizeof(unsigned long long), 256);
}

// What the scan of R rows needs ...
size_t row_topk_need(int R, int V, int K, const ScanRows& rows) {
  return R <= 0 ? 0 : slots_bytes((size_t)R * plan_scan(R, V, K, rows).splits, K);
}

// ... and what any scan of up to R rows can need: fewer rows are cut into more slices each (see plan_scan).
size_t row_topk_workspace(int R, int V, int K, bool sparse) {
  if (R <= 0) return 0;
  const int64_t small = (V + scan_tile(SCAN_SMALL) - 1) / scan_tile(SCAN_SMALL);
  const int64_t big = (V + scan_tile(SCAN_BIG) - 1) / scan_tile(SCAN_BIG);
  int64_t n = std::max({(int64_t)R, std::min(R, 4) * std::min<int64_t>(small, MAX_SPLITS), std::min<int64_t>(std::min(R, 16) * small, SCAN_BIG_WGS),
                        std::min<int64_t>(R * big, SCAN_BIG_WGS)});
  if (sparse) n = std::max(n, std::min<int64_t>(R * std::min<int64_t>(small, 16), SCAN_FINE_WGS));
  if (R > SCAN_BIG_WGS) n = std::max(n, std::min<int64_t>(R * std::min<int64_t>(small, 3), SCAN_CUT_WGS));
  return slots_bytes((size_t)n, K);
}

hs_status row_topk_launch(const float* logits, int64_t row_stride, int R, int V, int K, float temperature,
                          int32_t* topk_idx, float* topk_logp, float* ent_topk, float* ent_full, float* lse,
                          void* workspace, hipStream_t stream, ScanSlices* slices, const uint8_t* row_active,
                          const int32_t* row_index, const float* logits2, int rows1, bool prepared) {
  // (rows are the grid's second dimension)
  HS_REQUIRE(R <= ROW_SCAN_MAX, HS_ERR_UNSUPPORTED, "row scan: %d rows in one call (at most %d)", R, ROW_SCAN_MAX);
  const ScanRows rows{scan_aligned(logits, logits2, row_stride), row_active != nullptr, slices != nullptr && slices->pairs_only};
  ScanPlan p = plan_scan(R, V, K, rows);
  Carver c(workspace);
  size_t n = (size_t)R * p.splits;
  // one counter per row, zero in a prepared workspace and left at zero; always the same leading part
  // of the workspace, whatever the shape, so that calls of different shapes can share a prepared one
  unsigned* tickets = c.take<unsigned>(TICKET_BYTES / sizeof(unsigned));
  float4* part_stats = c.take<float4>(n);
  unsigned long long* part_key = c.take<unsigned long long>(n * K);
  const float inv_t = 1.0f / temperature;
  dim3 grid(p.splits, R);
  // one launch: the rows' last slices merge (needs the zeroed counters of a prepared workspace)
  const bool fused = prepared && slices == nullptr && p.splits > 1 && p.splits * K <= FUSED_CAP;
  // (the ratio rule reads its rows again, and not all of those that are counted here)
  // Argmax scans gain either way: 97 rows of 128256 17.7, 16.3 and (held) 14.1, 13.1; 896 84.8, 74.5; 2000 of 32000 51.8, 45.0 and 44.0, 43.6.  Full scans
  // of logits that the kernel before has just written, both together: 97 of 128256 37.8, 38.2, 400 of 32000 35.4, 35.9, 200 of 128256 55.0, 54.9, 2000 of 32000 144.8,
  // 132.1, 896 of 128256 256.8, 238.0.
  // The hint leaves the caches to what is read again.  Cold inputs and ones that the last-level cache holds, K = 10: 896 rows of 128256
  // logits 93.4 us without it, 84.5 with it; 2000 of 32000 56.1, 51.5 and (held) 50.4, 51.5; 200 of 128256 28.1, 26.0 and 26.0, 25.9;
  // 97 of 128256 24.0, 22.6 and 22.5, 21.3; 600 of 32000 25.5, 24.0 and 24.0, 23.1; but 1000 of 8192, which the L2 caches hold, 15.7, 15.5 and 12.9, 14.3.
  const bool stream_in = !rows.sparse && (int64_t)R * V >= SCAN_STREAM;
  const bool few_tiles = p.tiles_per_wg <= SCAN_NBUF && !stream_in;
#define HS_SCAN_LAUNCH_AS(T, F, ST, NT, SH)                                                                                   \
  hipLaunchKernelGGL((k_scan_rows<T, F, SCAN_NBUF, ST, NT, SH>), grid, dim3(T), 0, stream, logits, row_stride, V, K, inv_t, p.tiles_per_wg, \
                     part_stats, part_key, topk_idx, topk_logp, ent_topk, ent_full, lse, row_active, row_index, logits2, rows1, tickets)
#define HS_SCAN_LAUNCH(F, ST)                                                                        \
  do {                                                                                               \
    if (p.threads == SCAN_BIG && stream_in) HS_SCAN_LAUNCH_AS(SCAN_BIG, F, ST, true, false);           \
    else if (p.threads == SCAN_BIG && few_tiles) HS_SCAN_LAUNCH_AS(SCAN_BIG, F, ST, false, true);      \
    else if (p.threads == SCAN_BIG) HS_SCAN_LAUNCH_AS(SCAN_BIG, F, ST, false, false);                  \
    else if (stream_in) HS_SCAN_LAUNCH_AS(SCAN_SMALL, F, ST, true, false);                             \
    else if (few_tiles) HS_SCAN_LAUNCH_AS(SCAN_SMALL, F, ST, false, true);                             \
    else HS_SCAN_LAUNCH_AS(SCAN_SMALL, F, ST, false, false);                                           \
  } while (0)
  if (slices != nullptr && slices->pairs_only) HS_SCAN_LAUNCH(false, false);
  else if (fused) HS_SCAN_LAUNCH(true, true);
  else HS_SCAN_LAUNCH(false, true);
#undef HS_SCAN_LAUNCH
#undef HS_SCAN_LAUNCH_AS
  hs_status st = launch_status("row scan");
  if (slices != nullptr) {
    slices->key = part_key;
    slices->count = p.splits;
  }
  if (st != HS_OK || p.splits == 1 || slices != nullptr || fused) return st;
  hipLaunchKernelGGL(k_scan_finalize, dim3(R), dim3(FIN_THREADS), 0, stream, part_stats, part_key, p.splits, K, inv_t, topk_idx, topk_logp, ent_topk, ent_full, lse, row_active, row_index);
  return launch_status("row scan merge");
}

}  // namespace hs

extern "C" size_t hs_draft_entropy_topk_workspace(int32_t R, int32_t V, int32_t K) {
  if (R <= 0 || V <= 0 || K <= 0 || K > HS_MAX_TOPK) return 0;
  return hs::row_topk_workspace(R, V, K, false);
}

static hs_status entropy_topk_impl(const float* logits, int64_t row_stride, const int32_t* row_index, int32_t R,
                                   int32_t V, int32_t K, float temperature, int32_t* topk_idx, float* topk_logp,
                                   float* ent_topk, float* ent_full, float* lse, void* workspace,
                                   size_t workspace_bytes, hs_stream stream, bool prepared = false) {
  hs::clear_error();
  HS_REQUIRE(R >= 0 && V >= 1, HS_ERR_SHAPE, "hs_draft_entropy_topk: R=%d V=%d", R, V);
  HS_REQUIRE(K >= 1 && K <= V, HS_ERR_SHAPE, "hs_draft_entropy_topk: K=%d must be in 1..V=%d", K, V);
  HS_REQUIRE(K <= HS_MAX_TOPK, HS_ERR_UNSUPPORTED, "hs_draft_entropy_topk: K=%d exceeds HS_MAX_TOPK=%d", K,
             HS_MAX_TOPK);
  HS_REQUIRE(row_stride >= V, HS_ERR_SHAPE, "hs_draft_entropy_topk: row_stride=%lld < V=%d", (long long)row_stride, V);
  HS_REQUIRE(temperature > 0.f, HS_ERR_SHAPE, "hs_draft_entropy_topk: temperature must be positive");
  if (R == 0) return HS_OK;
  HS_REQUIRE(logits && topk_idx && topk_logp && ent_topk, HS_ERR_NULL, "hs_draft_entropy_topk: NULL argument");
  const size_t need = hs::row_topk_need(R, V, K, hs::ScanRows{hs::scan_aligned(logits, nullptr, row_stride), false, false});
  HS_REQUIRE(workspace && workspace_bytes >= need && reinterpret_cast<uintptr_t>(workspace) % 256 == 0,
             HS_ERR_WORKSPACE, "hs_draft_entropy_topk: workspace needs %zu bytes, 256-byte aligned (got %zu)", need,
             workspace_bytes);
  return hs::row_topk_launch(logits, row_stride, R, V, K, temperature, topk_idx, topk_logp, ent_topk, ent_full, lse,
                             workspace, static_cast<hipStream_t>(stream), nullptr, nullptr, row_index, nullptr, 0, prepared);
}

extern "C" hs_status hs_draft_entropy_topk(const float* logits, int64_t row_stride, int32_t R, int32_t V, int32_t K,
                                           float temperature, int32_t* topk_idx, float* topk_logp, float* ent_topk,
                                           float* ent_full, float* lse, void* workspace, size_t workspace_bytes,
                                           hs_stream stream) {
  return entropy_topk_impl(logits, row_stride, nullptr, R, V, K, temperature, topk_idx, topk_logp, ent_topk, ent_full,
                           lse, workspace, workspace_bytes, stream);
}

extern "C" hs_status hs_draft_entropy_topk_rows(const float* logits, int64_t row_stride, const int32_t* row_index,
                                                int32_t R, int32_t V, int32_t K, float temperature,
                                                int32_t* topk_idx, float* topk_logp, float* ent_topk, float* ent_full,
                                                float* lse, void* workspace, size_t workspace_bytes,
                                                hs_stream stream) {
  HS_REQUIRE(R <= 0 || row_index != nullptr, HS_ERR_NULL, "hs_draft_entropy_topk_rows: row_index is NULL");
  return entropy_topk_impl(logits, row_stride, row_index, R, V, K, temperature, topk_idx, topk_logp, ent_topk,
                           ent_full, lse, workspace, workspace_bytes, stream);
}

extern "C" hs_status hs_draft_entropy_topk_fused(const float* logits, int64_t row_stride, const int32_t* row_index,
                                                 int32_t R, int32_t V, int32_t K, float temperature,
                                                 int32_t* topk_idx, float* topk_logp, float* ent_topk, float* ent_full,
                                                 float* lse, void* workspace, size_t workspace_bytes,
                                                 hs_stream stream) {
  return entropy_topk_impl(logits, row_stride, row_index, R, V, K, temperature, topk_idx, topk_logp, ent_topk,
                           ent_full, lse, workspace, workspace_bytes, stream, true);
}

extern "C" hs_status hs_workspace_prepare(void* workspace, size_t workspace_bytes, hs_stream stream) {
  hs::clear_error();
  if (workspace_bytes == 0) return HS_OK;
  HS_REQUIRE(workspace != nullptr, HS_ERR_NULL, "hs_workspace_prepare: NULL workspace");
  HS_REQUIRE(reinterpret_cast<uintptr_t>(workspace) % 256 == 0 && workspace_bytes % 16 == 0, HS_ERR_WORKSPACE,
             "hs_workspace_prepare: the workspace must be 256-byte aligned and a multiple of 16 bytes long (got %zu)",
             workspace_bytes);
  const size_t n16 = workspace_bytes / 16;
  HS_REQUIRE((n16 + 255) / 256 <= 0x7fffffffull, HS_ERR_UNSUPPORTED, "hs_workspace_prepare: %zu bytes", workspace_bytes);
  hipLaunchKernelGGL(hs::k_fill_zero, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<uint4*>(workspace), n16);
  return hs::launch_status("workspace prepare");
}
