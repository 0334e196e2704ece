// Shared pieces of the tree-attention kernels (internal).
//
// Work decomposition, plain launches (float32 / any-shape kernel; matrix-core kernel when a batch
// has more sequences than the table below holds): grid.y = sequence, grid.x enumerates (key split, row block,
// KV head) of that sequence; workgroups whose indices fall outside their sequence's extent exit at
// once.  The prefix of sequence s is cut into n_sp = max(1, ceil(L_s / split_len)) splits; the last
// split also handles the tree rows themselves (the masked part).  Rows of one KV head g are
// r = i * G + gi for tree row i and group member gi (query head h = g * G + gi).
//
// Partial results (only when some sequence has more than one split): one record of D + 4 floats per
// (node, head, split): unnormalised output o[D], reference maximum m (in units of the scaled score),
// denominator l (relative to m) and two pad floats (records stay 16-byte aligned);
// slot = (node_global * Hq + h) * sp_max + split.
#pragma once
#include <cstddef>

#include "hs_common.h"

namespace hs {

typedef unsigned short bf16_t;  // raw bfloat16 bits

constexpr int ATTN_REC_PAD = 4;  // floats after o[D] in a partial record: m, l, pad, pad

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __builtin_bit_cast(float, (unsigned)b << 16); }
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {  // round to nearest, ties to even
  unsigned u = __builtin_bit_cast(unsigned, f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
// Four neighbouring elements as float32, at any element's address (the type's alignment is an element's).
typedef unsigned short bf16x4_any __attribute__((ext_vector_type(4), aligned(2)));
template <typename T>
__device__ __forceinline__ float4 load4(const T* p);
template <>
__device__ __forceinline__ float4 load4<float>(const float* p) {
  const float4_any f = *reinterpret_cast<const float4_any*>(p);
  return make_float4(f[0], f[1], f[2], f[3]);
}
template <>
__device__ __forceinline__ float4 load4<bf16_t>(const bf16_t* p) {
  const bf16x4_any f = *reinterpret_cast<const bf16x4_any*>(p);
  return make_float4(bf16_to_f32(f[0]), bf16_to_f32(f[1]), bf16_to_f32(f[2]), bf16_to_f32(f[3]));
}
template <typename T>
__device__ __forceinline__ void store4(T* p, float4 v);
template <>
__device__ __forceinline__ void store4<float>(float* p, float4 v) {
  *reinterpret_cast<float4_any*>(p) = float4_any{v.x, v.y, v.z, v.w};
}
template <>
__device__ __forceinline__ void store4<bf16_t>(bf16_t* p, float4 v) {
  *reinterpret_cast<bf16x4_any*>(p) = bf16x4_any{f32_to_bf16(v.x), f32_to_bf16(v.y), f32_to_bf16(v.z), f32_to_bf16(v.w)};
}

template <typename T>
__device__ __forceinline__ void store_elem(T* p, float v);
template <>
__device__ __forceinline__ void store_elem<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void store_elem<bf16_t>(bf16_t* p, float v) { *p = f32_to_bf16(v); }

// One sequence of the launch as the host planned it (work-list launches).  Its work items are
// numbered first_item + (split * n_rg + row_group) * Hkv + kv_head; entries are listed by falling
// cost of an item, so that the hardware's in-order dispatch starts the long items first.  The
// prefix is cut into n_sp splits of tiles_per_split 64-key tiles (the last one takes the rest and
// the tree rows).
struct SeqEntry {
  int first_item;
  int n0;               // first tree row of the sequence (global row number)
  int M;                // tree rows
  int L;                // prefix tokens
  long long p0;         // first prefix token (global); paged caches: first entry of the sequence's block-table row
  int tiles_per_split;
  short n_sp, n_rg;
};
static_assert(sizeof(SeqEntry) == 32, "eight dwords, fetched as two 16-byte loads per lane");
constexpr int ATTN_TBL = 96;  // entries that fit the kernel-argument segment next to the rest

struct AttnArgs {
  const void* q;
  const void* k_prefix;
  const void* v_prefix;
  const void* k_tree;
  const void* v_tree;
  const int32_t* parent;
  int tree_shared;  // 1: `parent` holds one tree that every batch entry uses (all entries have its row count)
  const int32_t* node_offsets;
  const int64_t* prefix_offsets;
  const int64_t* prefix_lens;  // used tokens of each sequence's prefix region; NULL: the whole region
  const int32_t* block_table;  // paged caches: page of each 64-token block, row s at s * max_blocks; else NULL
  int max_blocks;
  int B, Hq, Hkv, G;
  int half;        // 1 (matrix-core kernel, D = 64): Hkv counts pairs of KV heads and G the 2 Hq / Hkv query heads of a pair
  float scale;
  int split_len;   // prefix tokens per split (multiple of 64)
  int sp_max;      // largest split count of any sequence; 1 = results are written directly
  int n_rb_max;    // largest row-block count of any sequence (generic kernel)
  void* o;
  float* lse;
  float* part;
  int n_tbl;       // > 0: work-list launch (1-D grid over the items of tbl[0 .. n_tbl)); 0: grid.y = sequence
  int n_items;
  int narrow;      // work-list launches: 1 = two workgroups to an item, one for each 128 of its up to 256 rows; 2 = four
  int share;       // matrix-core kernel: equal row groups of five or six blocks share what is behind the fourth, 1 = of
                   // sequences with several groups, 2 = of all; 0 also where no group of the launch would
  int cmb_row0;    // first tree row that the merge of the splits looks at
  alignas(16) SeqEntry tbl[ATTN_TBL];  // (lanes fetch their entry with 16-byte loads)
};
static_assert(offsetof(AttnArgs, tbl) % 16 == 0, "16-byte loads of the table entries");

// Row groups of the matrix-core kernel: a KV head's rows, in blocks of 32, are spread over as many workgroups of up to
// eight blocks (a block to a wave) as they need.  Where that leaves room for groups of at most six blocks each, they get
// equal shares; otherwise full groups and a rest.  Groups of equal size pass over their keys at one pace and find
// them in L2, and five or six blocks need not take as long as eight (`share` in AttnArgs).  (40 layers of the 8B layout in
// one call, 73 rows on 2048 tokens, ten blocks as 5 + 5: whole step 197 -> 180 us, as 8 + 2 before; of the 70B layout, 71
// rows, 18 blocks as 6 + 6 + 6: 852 -> 778.  No gain from unequal ones: 13 blocks as 8 + 5 with the five shared 2 %
// slower, 25 as 8 + 6 + 6 + 5 1 %.)
__host__ __device__ __forceinline__ int row_groups(int n_blk) { return (n_blk + 7) >> 3; }
__host__ __device__ __forceinline__ bool equal_row_groups(int n_blk) { return n_blk <= 6 * row_groups(n_blk); }
// 32-row blocks of M tree rows; head dimension 64: counted head by head of the pair.
__host__ __device__ __forceinline__ int row_blocks(int G, int half, int M) {
  return half ? 2 * ((G / 2 * M + 31) >> 5) : (G * M + 31) >> 5;
}
// Whether groups of such a sequence share blocks under AttnArgs::share (equal groups beyond four blocks hold five or six each,
// or, of nine, five and four).
__host__ __device__ __forceinline__ bool groups_share(int n_blk, int share) {
  return share > (n_blk <= 6 ? 1 : 0) && n_blk > 4 && equal_row_groups(n_blk);
}
// First block and number of blocks of group rg (<= 0 when there is no such group).
__host__ __device__ __forceinline__ void row_group(int n_blk, int rg, int* first, int* count) {
  const int n_rg = row_groups(n_blk);
  if (n_rg > 3 || !equal_row_groups(n_blk)) {  // (four groups hold more than 24 blocks)
    *first = 8 * rg;
    *count = n_blk - 8 * rg < 8 ? n_blk - 8 * rg : 8;
    return;
  }
  const int each = n_rg == 1 ? n_blk : n_rg == 2 ? n_blk >> 1 : 5, more = n_blk - each * n_rg;  // (three: 17 or 18 blocks)
  *first = rg * each + (rg < more ? rg : more);
  *count = rg >= n_rg ? 0 : each + (rg < more ? 1 : 0);
}

// Prefix length of sequence s (plain launches read it on the device).
__device__ __forceinline__ int64_t prefix_len_of(const AttnArgs& a, int s) {
  return a.prefix_lens != nullptr ? a.prefix_lens[s] : a.prefix_offsets[s + 1] - a.prefix_offsets[s];
}

__host__ __device__ __forceinline__ int splits_of(int64_t L, int split_len) {
  int n = (int)((L + split_len - 1) / split_len);
  return n < 1 ? 1 : n;
}

}  // namespace hs
