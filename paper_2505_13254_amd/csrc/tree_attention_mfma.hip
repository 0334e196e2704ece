// bfloat16 tree attention on the matrix cores (head dimension 128; head dimension 64 by taking
// the KV heads in pairs, see HALF below).
//
// One workgroup = up to 256 query rows of one (sequence, KV head, key split); each of its eight
// waves owns 32 rows and keeps their output accumulators in registers for the whole pass, so K and
// V are read from HBM once per workgroup and shared through LDS by all G x M rows of the KV head
// (Section 2.2: every tree row attends to the same prefix).
//
// Both products are computed transposed with v_mfma_f32_32x32x16_bf16:
//     S^T[key, row] = K[key, :] . Q[row, :]      A = K fragment (LDS), B = Q fragment (registers)
//     O^T[d,  row] += V^T[d, key] P^T[key, row]  A = V fragment (LDS), B = P (registers)
// In the S^T accumulator a lane holds 16 keys of ONE row, so the softmax maximum and sum are
// in-lane reductions plus one exchange between the two half-waves, and P^T is already laid out as
// the B operand of the second product: no transposition of P through LDS.  The contraction order of
// the keys inside a 16-key MFMA step is permuted to match that layout, and the V^T fragments are
// fetched from the row-major V tile with the transposing LDS read (ds_read_b64_tr_b16), which hands
// each lane four keys of one output column.
//
// Softmax runs in the log2 domain.  Q is pre-multiplied by scale * log2(e), and the first MFMA of a
// score block starts from an accumulator holding minus the row's reference maximum, so the matrix
// core delivers x - m directly and the only per-score vector work is exp2, the row sum and the
// conversion to bf16.
//
// The reference maximum of a row is the exact maximum of its first 32-key block and then stays
// fixed: nothing is rescaled inside the loop.  P and the accumulators are floating point, so a later
// score above the reference only makes them larger, with the same relative precision; the result
// is exact after the final division by the equally referenced denominator.  Only an overflow (a
// score more than ~2^6 octaves above the reference) would break this; it shows in the denominator at
// the end of the pass, and the workgroup then repeats its pass with the classic block-by-block
// update of the maximum (rare, slow, same result).
//
// Schedule.  Each 32-key block passes through two windows of eight matrix instructions (head dimension
// 64: four): its scores, then its second product.  A window also takes half of a block's exponentials (the second half of
// the block whose product comes next, or the first half of the block whose scores were just
// finished) and requests the LDS fragments of the next step of two matrix instructions, so matrix, vector and LDS pipes of a wave all have independent work at any time.
//
// The tree part (ancestor mask) is a bit table built in LDS from the parent pointers: of all rows of a tree (up to
// 256), or, in launches with larger trees (BIG, up to 1024 rows), of the tree rows that the workgroup's own blocks
// hold, block by block.
//
// K/V tiles go from HBM straight into LDS (global_load_lds_dwordx4, 16 bytes per lane, no staging
// registers) through a ring of four tile buffers: one tile is being multiplied, the next one has
// landed, two more are on their way (64 KB per compute unit in flight).  The XOR swizzle that keeps
// LDS reads conflict-free is applied on the global side: the lane that fills LDS slot c of a row
// fetches chunk c ^ swz_key(row).  Waits are explicit (s_waitcnt vmcnt(n) counts this wave's younger
// tile loads) and the workgroup barrier carries no memory fence, so outstanding loads survive it.
#include <type_traits>

#include <hip/hip_ext.h>

#include "attn_common.h"

namespace hs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;
typedef __attribute__((address_space(3))) shortx4* lds_s4_ptr;

constexpr int MF_ROWS = 256;       // query rows per workgroup
constexpr int MF_THREADS = 512;    // eight waves of 32 rows, two per SIMD
constexpr int MF_TILE = 64;        // keys per LDS tile (two 32-key blocks)
constexpr int MF_NBUF = 4;         // LDS ring: one tile in use, one landed, two on their way from HBM
constexpr int MF_MAX_M = 256;      // tree rows per sequence whose ancestor bit table (M x 8 words) is built in LDS
constexpr int MF_ANC_STRIDE = 9;   // words from one row of that table to the next (eight, and one so that the rows of a wave lie in different banks)
constexpr int MF_BIG_M = 1024;     // tree rows per sequence at most
constexpr int MF_BIG_WORDS = 7424; // words of a workgroup's table in launches with more than MF_MAX_M rows (AncBlocks)
constexpr int MF_ROW_BYTES = 256;  // one K or V row of a head: 128 bf16
constexpr int MF_TILE_BYTES = MF_TILE * MF_ROW_BYTES;
constexpr int MF_BLOCK_BYTES = 32 * MF_ROW_BYTES;
constexpr int MF_LOADS = MF_TILE * 16 / MF_THREADS;  // 16-byte chunks of K (and of V) per thread per tile
constexpr int MF_AHEAD = 1;        // LDS fragments are requested this many steps (of two matrix instructions) ahead
constexpr float MF_LOG2E = 1.4426950408889634f;
constexpr float MF_LN2 = 0.6931471805599453f;
constexpr float MF_SUM_LIMIT = 0x1p64f;  // a denominator beyond it (or NaN) sends the pass to the exact path

// (D = 64: the caller also makes sure that the number of KV heads is even)
bool attn_mfma_supported(int D, hs_dtype dt, int max_tree_rows, float scale) {
  return (D == 128 || D == 64) && dt == HS_BF16 && max_tree_rows <= MF_BIG_M && scale > 0.f;
}

// Bytes that launches with more than MF_MAX_M rows in a tree ask for besides the partial records.  Nothing is kept in
// them (an ancestor table was, before workgroups built their own).  They are asked for all the same: a call whose workspace has no room
// for them is refused, or its keys are cut coarser, and so the calls that are refused and the bits of the others stay the same.
size_t attn_mfma_table_bytes(int max_tree_rows, int64_t NN) {
  return max_tree_rows > MF_MAX_M ? (size_t)NN * (MF_BIG_M / MF_TILE) * 8 : 0;
}

// The part of tree row i's root path inside its own word of 32 tree rows, as bits, and the first row of the path outside of
// it (negative: none).  par: the tree's parent pointers in LDS, up: that of row i.
__device__ __forceinline__ int2 anc_hop(const int* par, int i, int up) {
  unsigned bits = 1u << (i & 31);
  for (int j = i;; up = par[j]) {
    j = up < j ? up : -1;  // (a malformed tree cannot keep the walk from ending)
    if (j < (i & ~31)) return make_int2((int)bits, j);
    bits |= 1u << (j & 31);
  }
}

// Where a workgroup of a launch with large trees keeps the ancestor bits of its rows: an area for each of its blocks
// (b: 0 .. 7, by their order in the row group), in it a row of words for each tree row of the block, word q for the tree
// rows 32 q ..  .  With one query head to a KV head a block is 32 tree rows and eight blocks reach 1024 rows of up to 32
// words: there each block has the words of its own last row only, which is one word more from block to block.  Otherwise all
// have the words of the tree's visible rows, an odd number, so that the rows lie in different banks.
struct AncBlocks {
  int stride, base;  // words from row to row; first word of block b
  __host__ __device__ AncBlocks(int Gh, int tree_keys, int first_blk, int b) {
    const int rows = Gh == 1 ? 32 : 31 / Gh + 2;
    stride = ((tree_keys + 31) >> 5) | 1;
    base = b * rows * stride;
    if (8 * rows * stride > MF_BIG_WORDS) {  // (Gh == 1, beyond 928 rows)
      stride = first_blk + b + 1;
      base = 32 * (b * (first_blk + 1) + ((b * (b - 1)) >> 1));
    }
  }
};

// 16-byte chunk c (0..15) of row r lives at chunk position c ^ swz_key(r).  The key takes 16
// different values over 16 consecutive rows (one K row per lane: conflict-free 16-byte reads) and
// its upper two bits are the row's low two bits: the four rows that a transposing V read touches
// within a half-wave land in four different 64-byte bank ranges.
__device__ __forceinline__ int swz_key(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }
__device__ __forceinline__ int swz(int row, int chunk) { return row * MF_ROW_BYTES + ((chunk ^ swz_key(row)) << 4); }

// One tile from global memory straight into LDS: four loads of 16 bytes per lane (K and V, two row
// groups each).  A load lands at its wave-uniform LDS byte address (taken from M0, which is saved
// and restored) + 16 * lane; its source is a scalar base plus a 32-bit lane offset.
// ONCE: no other workgroup reads these keys, every head's rows fit one row group (a property of the
// launch, so that the hot loop has no branch for it).  The loads then carry the non-temporal hint, so that the stream does not push the data of
// the step's other kernels out of the caches (measured on the 32-layer launch: this kernel 1.5 us
// faster, the step's other kernels 3 us; 8 % on the 64-sequence batch).  With several row groups the
// later ones find the keys in L2, and the hint would cost that (3 % on the 1023-row workload).
#define MF_DMA_TILE(HINT)                                                                                  \
  asm volatile("s_mov_b32 %0, m0\n\t"                                                                      \
               "s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %5, %7" HINT "\n\t"                             \
               "s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %5, %8" HINT "\n\t"                             \
               "s_mov_b32 m0, %3\n\tglobal_load_lds_dwordx4 %6, %7" HINT "\n\t"                             \
               "s_mov_b32 m0, %4\n\tglobal_load_lds_dwordx4 %6, %8" HINT "\n\t"                             \
               "s_mov_b32 m0, %0"                                                                          \
               : "=&s"(saved)                                                                              \
               : "s"(lds_k0), "s"(lds_v0), "s"(lds_k1), "s"(lds_v1), "v"(off0), "v"(off1), "s"(kbase), "s"(vbase) \
               : "memory")
template <bool ONCE>
__device__ __forceinline__ void lds_dma_tile(const char* kbase, const char* vbase, unsigned off0, unsigned off1,
                                             unsigned lds_k0, unsigned lds_v0, unsigned lds_k1, unsigned lds_v1) {
  unsigned saved;
  if constexpr (ONCE) MF_DMA_TILE(" nt");
  else MF_DMA_TILE("");
}
#undef MF_DMA_TILE

// s_waitcnt on the LDS counter alone (vmcnt and expcnt fields at their maxima)
#define MF_WAIT_LDS_CONST(n) __builtin_amdgcn_s_waitcnt(0xC07F | ((n) << 8))
__device__ __forceinline__ void wait_lds(int n) {  // n is a constant once the windows are unrolled
  switch (n) {
    case 0: MF_WAIT_LDS_CONST(0); break;
    case 2: MF_WAIT_LDS_CONST(2); break;
    case 4: MF_WAIT_LDS_CONST(4); break;
    case 6: MF_WAIT_LDS_CONST(6); break;
    case 8: MF_WAIT_LDS_CONST(8); break;
    case 10: MF_WAIT_LDS_CONST(10); break;
    case 12: MF_WAIT_LDS_CONST(12); break;
    default: break;  // no hint: the compiler's own waits stand
  }
}

#define MF_PIN() __builtin_amdgcn_sched_barrier(0)

// PAGED: the prefix K/V live in pages of MF_TILE tokens ([page, token, Hkv, D]); a tile is a page.
// BIG: trees of more than MF_MAX_M rows may occur; a workgroup's ancestor table is of its own rows (AncBlocks).  (Until it was,
// a launch ahead of this one laid a table out in the workspace and its slices travelled with the tree tiles: 300 rows on 300 tokens,
// 32 heads on 8, 20.8 us a call and now 18.2; on 2048 tokens 32.3, 30.0; 1000 rows on 1000, 16 heads of one row each, 41.6, 37.7;
// 12 ragged sequences of up to 300 rows, paged, 4 layers 634, 626.)
// HALF: head dimension 64.  Two neighbouring KV heads of a token are 256 contiguous bytes, i.e. one
// row of this kernel, and a.Hkv / a.G count such pairs and the 2 G query heads that read them.  A
// wave's rows all belong to one head of the pair, whose half of the 256-byte rows it multiplies; K and
// V are read once, in whole rows.  (Query rows widened to 128 elements with zeros took twice the matrix
// instructions: 32 query heads, trees of 21 to 97 rows on 700 to 6001 tokens, 26.2 us -> 20.3 us.)
// SHARE: waves share row blocks behind the fourth, or four of them a block (a.share, a.narrow == 2).  The code for it is kept
// out of the other launches: with it in all of them, 8 KB of 47, launches of short items lost up to 1 us (one row, 40 heads on 1056
// tokens, 9 / 20 layers 42.4 / 85.7 us before there was sharing, 43.3 / 86.2 with its code in every launch, 42.1 / 85.0 now).
template <bool PAGED, bool ONCE, bool BIG, bool HALF, bool SHARE>
__global__ __launch_bounds__(MF_THREADS) void k_attn_mfma(AttnArgs a, int n_rg_max) {
  constexpr int Q_ROW_BYTES = HALF ? MF_ROW_BYTES / 2 : MF_ROW_BYTES;  // a row of Q and of O
  constexpr int NK = HALF ? 4 : 8;  // matrix instructions (and K fragments) of a 32-key score block
  constexpr int NT = HALF ? 2 : 4;  // 32-column blocks of a head's output row
  constexpr int STEPS = NK / 2;     // steps of two matrix instructions in a window
  constexpr int EPS = 4 / STEPS;    // pairs of exponentials a step takes along
  static_assert(!(BIG && ONCE), "more than 256 tree rows are several row groups");
  __shared__ __attribute__((aligned(16))) char lds_k[MF_NBUF][MF_TILE_BYTES];
  __shared__ __attribute__((aligned(16))) char lds_v[MF_NBUF][MF_TILE_BYTES];
  __shared__ unsigned anc[BIG ? MF_BIG_WORDS : MF_MAX_M * MF_ANC_STRIDE];
  __shared__ int par_small[BIG ? 1 : MF_MAX_M];
  // (large trees: in the ring's last slot, which is requested after the barrier that follows the paths' walk)
  int* const par_lds = BIG ? reinterpret_cast<int*>(lds_v[MF_NBUF - 1]) : par_small;
  __shared__ int exact_flag;
  __shared__ int page_lds[PAGED ? 256 : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (uniform for the compiler too: scalar branches)
  const int col = lane & 31, half = lane >> 5;
  // The first 64 entries of the work-list table are requested before anything else (the table is
  // part of the kernel arguments, so entry `lane` exists whatever the launch), and every scalar
  // argument the kernel needs is fetched in one batch right behind: left to itself the compiler
  // fetches each argument where it is first used, one scalar-cache round trip after another.
  // (h_half is not looked at: it comes with its neighbours, and its register, free otherwise, would be given to a later load of the
  // batch, which then waits for this one.  D = 64, calls in a graph, six runs of either: 4 sequences of 61 rows on 2000 tokens 18.84 us, now 18.57, on
  // 1990 18.73 and 18.47, 3 of 97 on 2500 24.31 and 24.17; launches with another instantiation as before)
  uintx4 t0_lo = *reinterpret_cast<const uintx4*>(&a.tbl[lane]);
  uintx4 t0_hi = *(reinterpret_cast<const uintx4*>(&a.tbl[lane]) + 1);
  const void* const h_q = a.q;
  const void* const h_k_prefix = a.k_prefix;
  const void* const h_v_prefix = a.v_prefix;
  const void* const h_k_tree = a.k_tree;
  const void* const h_v_tree = a.v_tree;
  const int32_t* const h_parent = a.parent;
  void* const h_o = a.o;
  float* const h_lse = a.lse;
  float* const h_part = a.part;
  const float h_scale = a.scale;
  const int h_sp_max = a.sp_max, h_n_tbl = a.n_tbl, h_tree_shared = a.tree_shared, h_narrow = a.narrow, h_share = a.share;
  const int G = a.G, Hkv = a.Hkv, Hq = a.Hq, h_half = a.half;
  asm volatile("" : "+v"(t0_lo), "+v"(t0_hi));  // (keeps the request here instead of inside the branch that uses it)
  asm volatile("" ::"s"(h_q), "s"(h_k_prefix), "s"(h_v_prefix), "s"(h_k_tree), "s"(h_v_tree), "s"(h_parent), "s"(h_o),
               "s"(h_lse), "s"(h_part), "s"(h_scale), "s"(h_sp_max), "s"(h_n_tbl), "s"(G), "s"(Hkv), "s"(Hq),
               "s"(n_rg_max), "s"(h_tree_shared), "s"(h_narrow), "s"(h_share), "s"(h_half));
  int n0, M, g, rg, sp, n_sp, tiles_per_split;
  int64_t p0, L;
  if (h_n_tbl > 0) {
    // Work-list launch: the table of sequences sits in the kernel arguments; lane l fetches entry
    // l (and l + 64), a ballot finds the entry whose item range holds this workgroup, and its
    // fields are read from that lane: one memory round trip, no dependent offset loads.
    const int x = blockIdx.x, item = x >> h_narrow;  // (narrow launches: two or four workgroups to an item of the table)
    unsigned f[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int base = 0; base < h_n_tbl; base += 64) {
      const int idx = base + lane;
      uintx4 lo = {0x7fffffffu, 0, 0, 0}, hi = {0, 0, 0, 0};
      if (base == 0) {
        if (idx < h_n_tbl) {
          lo = t0_lo;
          hi = t0_hi;
        }
      } else if (idx < h_n_tbl) {
        lo = *reinterpret_cast<const uintx4*>(&a.tbl[idx]);
        hi = *(reinterpret_cast<const uintx4*>(&a.tbl[idx]) + 1);
      }
      const unsigned long long below = __ballot((int)lo[0] <= item);  // entries are in rising first_item order
      if (below == 0ull) break;
      const int e = __builtin_popcountll(below) - 1;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        f[k] = __builtin_amdgcn_readlane(lo[k], e);
        f[4 + k] = __builtin_amdgcn_readlane(hi[k], e);
      }
      if (below != ~0ull) break;
    }
    n0 = (int)f[1];
    M = (int)f[2];
    L = (int)f[3];
    p0 = (int64_t)(((unsigned long long)f[5] << 32) | f[4]);
    tiles_per_split = (int)f[6];
    n_sp = (int)(short)(f[7] & 0xffffu);
    const int n_rg = (int)(short)(f[7] >> 16) << h_narrow;
    int local = x - ((int)f[0] << h_narrow);
    g = local % Hkv;
    local /= Hkv;
    rg = local % n_rg;
    sp = local / n_rg;
  } else {
    const int s = blockIdx.y;
    n0 = a.node_offsets[s];
    M = a.node_offsets[s + 1] - n0;
    p0 = PAGED ? (int64_t)s * a.max_blocks : a.prefix_offsets[s];
    L = prefix_len_of(a, s);
    if (M <= 0) return;
    n_sp = splits_of(L, a.split_len);
    tiles_per_split = a.split_len / MF_TILE;
    int x = blockIdx.x;
    g = x % Hkv;
    x /= Hkv;
    rg = x % n_rg_max;
    sp = x / n_rg_max;
    if (rg >= (G * M + MF_ROWS - 1) / MF_ROWS || sp >= n_sp) return;
  }
  // Rows.  The rows of a (pair of) KV head(s) are numbered head by head in blocks of 32, tree row by tree
  // row inside a head: block b belongs to head b / nbh of the pair and holds its rows 32 (b % nbh) ...
  // (HALF: a wave's rows all read the same head of the pair, so it multiplies that head's half of the
  // 256-byte K and V rows only).  A row group is up to eight blocks, in narrow launches up to four or two.
  const int Gh = HALF ? G >> 1 : G;      // query heads per KV head
  const int Rh = Gh * M;                  // rows of a KV head
  const int nbh = (Rh + 31) >> 5;
  const int n_blk = HALF ? 2 * nbh : nbh;  // (row_blocks)
  int blk0, blk_n;  // first block of this group, and how many
  if (h_narrow != 0) {
    const int most = 8 >> h_narrow;
    blk0 = rg * most;
    blk_n = n_blk - blk0 < most ? n_blk - blk0 : most;
  } else {
    row_group(n_blk, rg, &blk0, &blk_n);
  }
  if (blk_n <= 0) return;  // (narrow: an item of few rows needs some of its two or four workgroups)
  // Narrow launches have compute units to spare and are bound by each workgroup's own pace: the
  // four blocks' waves alone, one to a SIMD, would have nothing to hide their chains of dependent
  // steps behind.  There two waves share a row block, one takes the even 32-key blocks of the
  // tiles, the other the odd ones, and their results meet in LDS at the end: `kpar` is the wave's key
  // parity, `pair_shift` tells how far apart the two waves are.  (Groups of at most four blocks in
  // launches that fill the chip are bound by HBM at 1.25 us a tile either way, and sharing made them
  // run ahead of the other row groups of their keys, out of reach of the L2 copies: 0.8 % slower.)
  const bool ksplit = h_narrow != 0;
  const int pair_shift = !ksplit ? 3 : blk_n <= 1 ? 0 : blk_n == 2 ? 1 : 2;
  // With four workgroups to an item there are at most two blocks for the eight waves: four waves share one, each with
  // every fourth 32 keys (`quarter`).  (61 rows on 2048 tokens, 8 KV heads, 32 layers one by one: 589 -> 535 us.)
  const bool quarter = SHARE && h_narrow == 2;
  // Groups of five or six blocks, all groups being so: the first four waves, one to a SIMD, take a block each, and
  // of the other four two share each block that is left, as above.  `ways` is the number of waves that share this wave's block,
  // kpar its share.  (With a wave to a block one or two SIMDs have two waves' work and the others one's: 129 rows on 4096 tokens, 40
  // layers and heads, 703 -> 675 us the whole step; ten blocks in two groups (row_group) 185 -> 180.  A fifth block shared by all four
  // of the others, each with every fourth 32 keys, kept two of the SIMDs busy for as long in every tile, the other two in the next, and in one go
  // without overlap: 1.51 us a tile, where six blocks took 1.31 and five do now.  When: see a.share.)
  const bool shared_tail = SHARE && (blk_n == 5 || blk_n == 6) && groups_share(n_blk, h_share);
  const int ways = quarter ? 4 : ksplit || (shared_tail && wave >= 4) ? 2 : 1;
  const int my_blk = blk0 + (shared_tail && wave >= 4 ? 4 + (blk_n == 6 ? wave & 1 : 0) : wave & ((1 << pair_shift) - 1));
  const int kpar = shared_tail ? (wave < 4 ? 0 : blk_n == 6 ? (wave - 4) >> 1 : wave - 4) : wave >> pair_shift;  // (without sharing: 0)
  const bool wave_active = my_blk < blk0 + blk_n && kpar < ways;
  const int hb = HALF && my_blk >= nbh ? 1 : 0;          // head of the pair
  const int row_base = (my_blk - hb * nbh) * 32;          // of the head's rows

  const char* kp = static_cast<const char*>(h_k_prefix) + ((PAGED ? 0 : p0) * Hkv + g) * MF_ROW_BYTES;
  const char* vp = static_cast<const char*>(h_v_prefix) + ((PAGED ? 0 : p0) * Hkv + g) * MF_ROW_BYTES;
  const char* kt = static_cast<const char*>(h_k_tree) + ((int64_t)n0 * Hkv + g) * MF_ROW_BYTES;
  const char* vt = static_cast<const char*>(h_v_tree) + ((int64_t)n0 * Hkv + g) * MF_ROW_BYTES;
  const int64_t tok_stride = (int64_t)Hkv * MF_ROW_BYTES;

  const bool last_split = sp == n_sp - 1;
  const int64_t k_lo = (int64_t)sp * tiles_per_split * MF_TILE;
  const int64_t k_hi = last_split ? L : k_lo + (int64_t)tiles_per_split * MF_TILE;
  const int n_ptiles = (int)((k_hi - k_lo + MF_TILE - 1) / MF_TILE);
  // (large trees: tree rows behind the last row of this row group are on nobody's root path, their tiles are left out)
  int tree_keys = M;
  if constexpr (BIG) {
    const int last = blk0 + blk_n - 1;
    if (!HALF || blk0 >= nbh || last < nbh) {  // (all of one head)
      const int past = (last - (HALF && blk0 >= nbh ? nbh : 0)) * 32 + 32;  // first row behind the group
      if (past < Rh) tree_keys = (past - 1) / Gh + 1;
    }
  }
  const int n_ttiles = last_split ? (tree_keys + MF_TILE - 1) / MF_TILE : 0;
  const int n_tiles = n_ptiles + n_ttiles;  // >= 1: a split holds prefix keys, or it is the last one
  const int n_full = (int)((k_hi - k_lo) / MF_TILE);  // leading tiles made of 64 prefix keys
  const int n_plain = (int)((k_hi - k_lo) >> 5);      // leading blocks that need no mask

  // ---- tile loads.  Issued as inline assembly: the compiler then neither tracks them in its own
  // wait counters nor orders LDS reads of other ring slots behind them.  The lane that fills the
  // 16-byte LDS slot c of a tile (row c / 16, position c % 16) fetches chunk (c % 16) ^ swz_key(row).
  static_assert(MF_LOADS == 2, "lds_dma_tile moves two row groups of K and of V");
  const unsigned lds_k_addr = (unsigned)(uintptr_t)(lds_ptr)&lds_k[0][0];
  const unsigned lds_v_addr = (unsigned)(uintptr_t)(lds_ptr)&lds_v[0][0];
  const unsigned wave_lds = __builtin_amdgcn_readfirstlane((unsigned)(wave * 64 * 16));  // this wave's 1 KB of a row group
  const int dma_row = tid >> 4;                                                        // + 32 for the second row group
  const unsigned dma_chunk = (unsigned)(((tid & 15) ^ swz_key(dma_row)) << 4);         // swz_key(row + 32) == swz_key(row)
  const unsigned lane_off0 = (unsigned)(dma_row * (int)tok_stride) + dma_chunk;        // inside a full tile: fixed
  const unsigned lane_off1 = lane_off0 + (unsigned)(32 * (int)tok_stride);
  // Large trees: where the bits of this wave's block lie, and its first tree row.
  const int blk_in_head = blk0 - (HALF && blk0 >= nbh ? nbh : 0);
  const AncBlocks anc_at(Gh, tree_keys, blk_in_head, my_blk - blk0);
  // Paged caches: the pages of this split's tiles (at most 256) are staged in LDS; the requests
  // go out here, before the Q rows are asked for, so that waiting for them waits for nothing else.
  // A tile's page is then one LDS read.  (That read is older than every fragment read requested
  // after it, so the windows' counted LDS waits at most wait for one fragment more than they need.)
  if (PAGED) {
    const int32_t* bt = a.block_table + p0 + k_lo / MF_TILE;
    if (tid < n_ptiles) page_lds[tid] = bt[tid];
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  // byte offset, from kp / vp, of prefix tile t of this split
  auto prefix_tile = [&](int t) -> int64_t {
    if (!PAGED) return (k_lo + (int64_t)t * MF_TILE) * tok_stride;
    return (int64_t)__builtin_amdgcn_readfirstlane(page_lds[t]) * MF_TILE * tok_stride;
  };
  // a full tile of prefix keys into ring slot `slot`
  auto issue_full = [&](int t, int slot) {
    const int64_t tile_off = prefix_tile(t);
    const unsigned ring = (unsigned)slot * MF_TILE_BYTES + wave_lds;
    lds_dma_tile<ONCE>(kp + tile_off, vp + tile_off, lane_off0, lane_off1, lds_k_addr + ring, lds_v_addr + ring,
                 lds_k_addr + ring + MF_BLOCK_BYTES, lds_v_addr + ring + MF_BLOCK_BYTES);
  };
  // any tile: the last prefix tile may be partial, tree tiles come from the tree buffers; rows past
  // the end repeat the last row (their scores are masked)
  auto issue = [&](int t) {
    if (t < n_full) {
      issue_full(t, t % MF_NBUF);
      return;
    }
    const bool tree = t >= n_ptiles;
    const char* ks = tree ? kt : kp;
    const char* vs = tree ? vt : vp;
    const int64_t base = tree ? (int64_t)(t - n_ptiles) * MF_TILE : k_lo + (int64_t)t * MF_TILE;
    const int rows = (int)((tree ? (int64_t)M : k_hi) - base);  // >= 1 rows of this tile exist
    const int r0 = dma_row < rows ? dma_row : rows - 1;
    const int r1 = dma_row + 32 < rows ? dma_row + 32 : rows - 1;
    const unsigned ring = (unsigned)(t % MF_NBUF) * MF_TILE_BYTES + wave_lds;
    const int64_t off = tree ? base * tok_stride : prefix_tile(t);
    lds_dma_tile<ONCE>(ks + off, vs + off, (unsigned)(r0 * (int)tok_stride) + dma_chunk,
                 (unsigned)(r1 * (int)tok_stride) + dma_chunk, lds_k_addr + ring, lds_v_addr + ring,
                 lds_k_addr + ring + MF_BLOCK_BYTES, lds_v_addr + ring + MF_BLOCK_BYTES);
  };
  // waits until at most n (a multiple of four, at most 16) of this wave's loads are pending
  auto wait_vm = [&](int n) {
    switch (n) {
      case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
      case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
      case 8: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
      case 12: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
      default: asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
    }
  };
  // Start of a pass: tiles 0 and 1 are on their way; wait for this wave's part of tile 0, meet the
  // other waves, request tile 2.
  auto first_arrival = [&]() {
    if (n_tiles > 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * MF_LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (2 < n_tiles) issue(2);
  };
  // Middle of trip t (tile t is being multiplied): wait for this wave's part of tile t + 1 (tile
  // t + 2 may still be pending), meet the other waves, request tile t + 3.  Every wave has finished
  // tile t - 1 by then: its slot is the one that tile t + 3 goes to.
  auto next_arrival = [&](int t) {
    if (t + 2 < n_tiles) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * MF_LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (t + 3 < n_tiles) issue(t + 3);
  };

  // ---- set-up.  Its global reads (parent pointers, Q rows) are requested first and the first two
  // K/V tiles right behind them, so that HBM is busy while the ancestor table is built and Q is
  // converted.  (Loads return in order: waiting for the Q rows never waits for a tile.)
  // r / Gh for a row number r < 2^16 without the integer-division sequence: (r + 0.5) / Gh is at least
  // 1 / (2 Gh) away from an integer, far more than the rounding of the float product
  const float inv_G = 1.0f / (float)Gh;
  auto div_G = [&](int r) { return (int)(((float)r + 0.5f) * inv_G); };
  // These loads are inline assembly like the tile loads: the compiler does not see the tile loads, so
  // a load of its own would be waited for with vmcnt(0), i.e. together with every tile requested
  // behind it.  Here the waits count the younger loads (wait_vm), and an empty asm statement that
  // "writes" the registers keeps their uses behind the wait.  Lanes without a row of their own load
  // a valid row (the last one; tree row 0) and zero it afterwards.
  // (first tree row of the block, and how many it has: the same for all lanes)
  const int blk_node = __builtin_amdgcn_readfirstlane(div_G(row_base < Rh ? row_base : Rh - 1));
  const int nodes = !wave_active ? 0 : __builtin_amdgcn_readfirstlane(div_G(row_base + 31 < Rh ? row_base + 31 : Rh - 1)) - blk_node + 1;
  int my_parent = 0, far_parent = 0;  // (far: of tree row 512 + tid)
  {
    const int32_t* src = h_parent + (h_tree_shared ? 0 : n0) + (tid < M ? tid : 0);  // (one tree for all entries, or each its own)
    asm volatile("global_load_dword %0, %1, off" : "=v"(my_parent) : "v"(src) : "memory");
    if constexpr (BIG) {
      const int32_t* far = h_parent + (h_tree_shared ? 0 : n0) + (tid + MF_THREADS < M ? tid + MF_THREADS : 0);
      asm volatile("global_load_dword %0, %1, off" : "=v"(far_parent) : "v"(far) : "memory");
    }
  }
  uintx4 qraw[NK];
  bool row_real;
  const int head0 = g * G + hb * Gh;  // first query head of this wave's KV head
  {
    const int r = row_base + col;
    const int rc = r < Rh ? r : Rh - 1;
    const int i = div_G(rc), gi = rc - i * Gh;
    row_real = r < Rh;
    const char* qrow = static_cast<const char*>(h_q) + ((int64_t)(n0 + i) * Hq + head0 + gi) * Q_ROW_BYTES + half * 16;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk)
      asm volatile("global_load_dwordx4 %0, %1, off offset:%2" : "=v"(qraw[kk]) : "v"(qrow), "n"(32 * kk) : "memory");
  }
  issue(0);
  if (n_tiles > 1) issue(1);
  const int first_tile_loads = 2 * MF_LOADS * (n_tiles < 2 ? n_tiles : 2);
  // ---- ancestor bit table: bit j of row i's words is set iff tree row j is on the root path of i.
  // The parent pointers are staged in LDS and the paths are walked there, a bit at a time straight into the row: a
  // step is one dependent read and an OR that nobody waits for.  Trees of up to 64 rows are the first wave's
  // alone, which need not wait until every other wave has got its requests out.  (The row in eight registers and a
  // barrier for every tree: workgroups with the tree part of a 61-row tree were ready for their first tile 2.5 us after the others, now 1.1.)
  if (!BIG && last_split && tid < M) {
#pragma unroll
    for (int q = 0; q < 8; ++q) anc[tid * MF_ANC_STRIDE + q] = 0u;
  }
  wait_vm(NK + first_tile_loads);  // the parent pointers are there (the Q loads and the tiles are younger)
  asm volatile("" : "+v"(my_parent), "+v"(far_parent));
  if (BIG && last_split) {
    // A lane walks one tree row's path, a word of 32 tree rows at a time: first every tree row of the entry finds the part of its
    // path inside its own word.  No walk is longer than 32 steps, twice.  (Row by row up to the root: 8 chains of 1024 rows on 500 tokens, 32
    // heads on 8, 341 us, now 192; 96 chains of 300 rows on 100 tokens 445, now 295.  With the words read by every workgroup from a table that
    // a launch ahead makes with the same steps: 187 and 281, but 300 rows on 300 tokens 20.6 us, so 18.1, and 96 trees of 12 levels no less.)
    // (Two waves that share a block write the same bits: they are cleared before the barrier and only set behind it.)
    unsigned* const area = &anc[anc_at.base];
    for (int i = lane; i < nodes * anc_at.stride; i += 64) area[i] = 0u;
    par_lds[tid] = my_parent;
    if (M > MF_THREADS) par_lds[tid + MF_THREADS] = far_parent;
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    int2* const hops = reinterpret_cast<int2*>(par_lds + MF_BIG_M);
    hops[tid] = anc_hop(par_lds, tid, my_parent);
    if (M > MF_THREADS) hops[tid + MF_THREADS] = anc_hop(par_lds, tid + MF_THREADS, far_parent);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (lane < nodes) {
      unsigned* const row = area + lane * anc_at.stride;
      for (int j = blk_node + lane; j >= 0;) {
        const int2 hop = hops[j];
        row[j >> 5] = (unsigned)hop.x;
        j = hop.y;
      }
    }
  }
  if (!BIG && last_split) {
    if (tid < M) par_lds[tid] = my_parent;
    if (M > 64) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (tid < M) {
      unsigned* const row = &anc[tid * MF_ANC_STRIDE];
      atomicOr(row + (tid >> 5), 1u << (tid & 31));
      for (int j = tid, up = my_parent; up >= 0 && up < j;) {  // (a malformed tree cannot keep the walk from ending)
        j = up;
        up = par_lds[j];
        atomicOr(row + (j >> 5), 1u << (j & 31));
      }
    }
  }
  if (tid == 0) exact_flag = 0;

  // ---- Q fragments (B operand of the first product), pre-multiplied by scale * log2(e) so that
  // the scores come out of the MFMA in the log2 domain
  const float c2 = row_real ? h_scale * MF_LOG2E : 0.f;
  wait_vm(first_tile_loads);  // the Q rows are there (the tiles are younger)
  if constexpr (HALF) {
    asm volatile("" : "+v"(qraw[0]), "+v"(qraw[1]), "+v"(qraw[2]), "+v"(qraw[3]));
  } else {
    asm volatile("" : "+v"(qraw[0]), "+v"(qraw[1]), "+v"(qraw[2]), "+v"(qraw[3]), "+v"(qraw[4]), "+v"(qraw[5]),
                 "+v"(qraw[6]), "+v"(qraw[7]));
  }
  bf16x8 qf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const bf16x8 raw = __builtin_bit_cast(bf16x8, qraw[kk]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      floatx2 f = {(float)raw[2 * e] * c2, (float)raw[2 * e + 1] * c2};
      bf16x2 hb = __builtin_convertvector(f, bf16x2);
      qf[kk][2 * e] = hb[0];
      qf[kk][2 * e + 1] = hb[1];
    }
  }

  floatx16 acc[NT];  // O^T: [d block of 32][16 values]: d = 32 tt + 8 (v / 4) + 4 half + v % 4
  floatx16 negm;     // minus the reference maximum in all 16 slots: start value of a score block
  float m_ref = 0.f, l_sum = 0.f;
#pragma unroll
  for (int v = 0; v < 16; ++v) negm[v] = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

  // ---- LDS fragments.  Per-lane addresses for block 0 of ring slot 0; a block of slot s, parity b
  // lies s * MF_TILE_BYTES + b * MF_BLOCK_BYTES further (an immediate offset when s is static).
  // K: lane (col, half) reads chunk 2 kk + half of key row col.  V: the transposing read returns, to
  // lane l of a 16-lane group, element l % 4 of the 8-byte pieces addressed by lanes l / 4 + {0, 4,
  // 8, 12} of the group: lane (a = l % 4, j = l / 4) therefore addresses key j of the wanted four at
  // columns 4a .. 4a+3; fragment f = NT k2 + tt holds the 16 keys of contraction step k2 for the 32
  // output columns of d block tt.  (HALF: the second head's half of a row begins at chunk 8.)
  const int tr_a = lane & 3, tr_j = (lane >> 2) & 3, tr_dh = (lane >> 4) & 1;
  const char* kl[NK];
  const char* vl[NK][2];
  const int chunk0 = 8 * hb;
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) kl[kk] = &lds_k[0][0] + swz(col, chunk0 + 2 * kk + half);
#pragma unroll
  for (int f = 0; f < NK; ++f)
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int key = 16 * (f / NT) + 8 * r + 4 * half + tr_j;
      vl[f][r] = &lds_v[0][0] + swz(key, chunk0 + 4 * (f % NT) + 2 * tr_dh + (tr_a >> 1)) + (tr_a & 1) * 8;
    }
  auto ldk = [&](int off, int kk) { return *reinterpret_cast<const bf16x8*>(kl[kk] + off); };
  auto ldv = [&](int off, int f) {
    bf16x8 vf;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const shortx4 got = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr)(vl[f][r] + off));
      const bf16x4 gb = __builtin_bit_cast(bf16x4, got);
      vf[4 * r + 0] = gb[0];
      vf[4 * r + 1] = gb[1];
      vf[4 * r + 2] = gb[2];
      vf[4 * r + 3] = gb[3];
    }
    return vf;
  };
  // byte offset of block (slot, parity) inside a ring
  auto blk_off = [](int slot, int parity) { return slot * MF_TILE_BYTES + parity * MF_BLOCK_BYTES; };

  // ---- masks of a block's scores: tree keys off the row's root path, keys past the end of the
  // split.  Only the blocks from n_plain on need it (the partial prefix tail and the tree part).
  // (the lane's tree row is found again where a tree tile is masked, which the empty statements keep the compiler
  // from doing ahead of the loops: registers for it would be spilled, and read back behind a wait for the tiles)
  // (large trees: where the words of tree row 0 would be; in a scalar register, as a vector one would be spilled likewise: 200 trees of 260 rows without a
  // prefix, 8 heads, 212 us, now 180)
  const int anc_row0 = BIG ? __builtin_amdgcn_readfirstlane(anc_at.base - blk_node * anc_at.stride) : 0;
  const float inv_G_scalar = BIG ? __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, inv_G))) : 0.f;
  auto tree_row = [&]() {
    unsigned l = ~0u;
    int g = Gh;
    asm volatile("" : "+s"(l), "+s"(g));
    const int r = row_base + (int)(__builtin_amdgcn_mbcnt_hi(l, __builtin_amdgcn_mbcnt_lo(l, 0)) & 31);
    return (int)(((float)(r < Rh ? r : Rh - 1) + 0.5f) * (BIG ? inv_G_scalar : __builtin_amdgcn_rcpf((float)g)));  // (as div_G)
  };
  auto mask_block = [&](int blk, floatx16& S) {
    const int t = blk >> 1;
    if (t >= n_ptiles) {
      const int bbase = (t - n_ptiles) * MF_TILE + (blk & 1) * 32;
      unsigned word;
      if constexpr (BIG) word = (bbase >> 5) < anc_at.stride ? anc[anc_row0 + (int)__umul24((unsigned)tree_row(), (unsigned)anc_at.stride) + (bbase >> 5)] : 0u;
      else word = bbase < M ? anc[tree_row() * MF_ANC_STRIDE + (bbase >> 5)] : 0u;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int bit = 8 * (v >> 2) + 4 * half + (v & 3);
        S[v] = ((word >> bit) & 1u) ? S[v] : -HS_INF;
      }
    } else {
      const int64_t bbase = k_lo + (int64_t)t * MF_TILE + (blk & 1) * 32;
      if (bbase + 32 > k_hi) {
        const int valid = (int)(k_hi - bbase);  // may be <= 0: the whole block is past the end
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = 8 * (v >> 2) + 4 * half + (v & 3);
          S[v] = key < valid ? S[v] : -HS_INF;
        }
      }
    }
  };
  // exact maximum of a row's 32 scores of a block (both half-waves)
  auto row_max = [&](const floatx16& S) {
    float m4[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) m4[c] = fmaxf(fmaxf(S[c], S[4 + c]), fmaxf(S[8 + c], S[12 + c]));
    const float mx = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
    return fmaxf(mx, __shfl_xor(mx, 32));
  };
  // moves the reference maximum up by delta (>= 0 except at the very first block)
  auto move_reference = [&](float delta) {
    const float alpha = exp2_fast(-delta);
    m_ref += delta;
    l_sum *= alpha;
#pragma unroll
    for (int v = 0; v < 16; ++v) negm[v] = -m_ref;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tt][v] *= alpha;
  };
  // the first reference of a pass (denominator and accumulators are still zero: nothing to rescale,
  // and no 0 x 2^(-m) = 0 x inf for a first block whose scores are all hugely negative)
  auto set_reference = [&](float mx) {
    m_ref = mx;
#pragma unroll
    for (int v = 0; v < 16; ++v) negm[v] = -mx;
  };
  // the pieces of a window: two exponentials (keys 2j, 2j + 1 of half h of a block), and, one step
  // later, their bf16 pair; the two values also go into two running denominators
  float l0 = 0.f, l1 = 0.f;
  auto exp_pair = [&](const floatx16& S, int h, int j) {
    floatx2 pp = {exp2_fast(S[8 * h + 2 * j]), exp2_fast(S[8 * h + 2 * j + 1])};
    return pp;
  };
  auto pack_pair = [&](const floatx2& pp, uintx4& P, int j) {
    l0 += pp[0];
    l1 += pp[1];
    P[j] = __builtin_bit_cast(unsigned, __builtin_convertvector(pp, bf16x2));
  };
  // half h of a block outside the windows
  auto exp_half = [&](const floatx16& S, int h, uintx4& P) {
#pragma unroll
    for (int j = 0; j < 4; ++j) pack_pair(exp_pair(S, h, j), P, j);
  };

  bf16x8 kf[NK], vf[NK];  // fragment registers: four of each are alive at any time
  // Score window: S_out = K(block at oq) Q^T, started from -m_ref, in STEPS steps of two matrix
  // instructions.  A step first requests the fragments of the next step (the window's last step:
  // the first two V fragments of the block at ov, whose product window follows), waits for its own,
  // and pairs its matrix instructions with EPS pairs of exponentials of half h of S_in.
  // Wave priority: the two waves of a SIMD compete for its issue slots.  A wave raises its priority
  // for a window (product windows above score windows) and drops it afterwards, so that whichever wave
  // is inside a window, and of two the one in its product window, issues first: 3 % on every shape
  // (paired A/B: -2.4 us of 78 on the 32-layer launch, -3.7 % on the 70B shape).  Toggling around each
  // matrix instruction instead was slower than no priorities at all.
  auto win_qk = [&](int oq, int ov, floatx16& S_out, const floatx16& S_in, int h, uintx4& P) {
    floatx2 pp[4];
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
      const int sN = j + MF_AHEAD;  // the step whose fragments are requested now (STEPS: the product window's first)
      if (sN < STEPS) {
        kf[2 * sN] = ldk(oq, 2 * sN);
        kf[2 * sN + 1] = ldk(oq, 2 * sN + 1);
      } else {
        vf[2 * (sN - STEPS)] = ldv(ov, 2 * (sN - STEPS));
        vf[2 * (sN - STEPS) + 1] = ldv(ov, 2 * (sN - STEPS) + 1);
      }
      int pending = 0;  // LDS reads requested after those of step j: K steps count 2, V steps 4
#pragma unroll
      for (int d = 1; d <= MF_AHEAD; ++d) pending += (j + d < STEPS) ? 2 : 4;
      wait_lds(pending);
      S_out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[2 * j], qf[2 * j], j == 0 ? negm : S_out, 0, 0, 0);
#pragma unroll
      for (int e = EPS * j; e < EPS * (j + 1); ++e) pp[e] = exp_pair(S_in, h, e);
      S_out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[2 * j + 1], qf[2 * j + 1], S_out, 0, 0, 0);
      if (j > 0) {
#pragma unroll
        for (int e = EPS * (j - 1); e < EPS * j; ++e) pack_pair(pp[e], P, e);
      }
      MF_PIN();
    }
#pragma unroll
    for (int e = EPS * (STEPS - 1); e < 4; ++e) pack_pair(pp[e], P, e);
    __builtin_amdgcn_s_setprio(0);
  };
  // Product window: O^T += V^T(block at ov) P^T with P = (P0, P1), same step structure; its last
  // steps request the first K fragments of the block at oq, whose score window follows
  // (with_kf: there is such a block).  with_exp: exponentials of half h of S_in are taken.
  auto win_pv = [&](int ov, int oq, const uintx4& P0, const uintx4& P1, const floatx16& S_in, int h, uintx4& P,
                    auto with_exp, auto with_kf) {
    constexpr bool EXP = decltype(with_exp)::value, KF = decltype(with_kf)::value;
    __builtin_amdgcn_s_setprio(2);
    const bf16x8 b0 = __builtin_bit_cast(bf16x8, P0), b1 = __builtin_bit_cast(bf16x8, P1);
    floatx2 pp[4];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
      const int sN = j + MF_AHEAD;
      if (sN < STEPS) {
        vf[2 * sN] = ldv(ov, 2 * sN);
        vf[2 * sN + 1] = ldv(ov, 2 * sN + 1);
      } else if (KF) {
        kf[2 * (sN - STEPS)] = ldk(oq, 2 * (sN - STEPS));
        kf[2 * (sN - STEPS) + 1] = ldk(oq, 2 * (sN - STEPS) + 1);
      }
      if (KF) {
        int pending = 0;
#pragma unroll
        for (int d = 1; d <= MF_AHEAD; ++d) pending += (j + d < STEPS) ? 4 : 2;
        wait_lds(pending);
      }
      acc[(2 * j) % NT] =
          __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[2 * j], 2 * j < NT ? b0 : b1, acc[(2 * j) % NT], 0, 0, 0);
      if (EXP) {
#pragma unroll
        for (int e = EPS * j; e < EPS * (j + 1); ++e) pp[e] = exp_pair(S_in, h, e);
      }
      acc[(2 * j + 1) % NT] =
          __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[2 * j + 1], 2 * j < NT ? b0 : b1, acc[(2 * j + 1) % NT], 0, 0, 0);
      if (EXP && j > 0) {
#pragma unroll
        for (int e = EPS * (j - 1); e < EPS * j; ++e) pack_pair(pp[e], P, e);
      }
      MF_PIN();
    }
    if (EXP) {
#pragma unroll
      for (int e = EPS * (STEPS - 1); e < 4; ++e) pack_pair(pp[e], P, e);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  const std::true_type YES{};
  const std::false_type NO{};

  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the ancestor table is complete
  first_arrival();
  const int n_blocks = 2 * n_tiles;

  if (wave_active) {
    floatx16 sA, sB;    // scores of the even / odd block of the tile in hand
    uintx4 pa, pb, pc;  // halves of P (bf16 pairs): first half of the even block, a second half, first half of the odd block
    // ---- first block: it always has a visible key (a prefix token, or the root), and its exact
    // maximum is the reference of the whole pass
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) kf[kk] = ldk(0, kk);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], kk == 0 ? negm : sA, 0, 0, 0);
    if (n_plain < 1) mask_block(0, sA);
    {
      const float mx = row_max(sA);
#pragma unroll
      for (int v = 0; v < 16; ++v) sA[v] -= mx;
      set_reference(mx);
    }
    if (ways == 4) {
      // ---- four waves to a row block: this one takes 32-key block kpar of every two tiles, in one go: it
      // is busy for a quarter of what its SIMD's other wave has to do, so nothing is gained by overlapping its
      // steps.  All four start from the first block's maximum.
      const int par = kpar & 1, odd_tile = kpar >> 1;
      for (int t = 0; t < n_tiles; ++t) {
        if (t + 1 < n_tiles) next_arrival(t);
        if ((t & 1) != odd_tile) continue;
        const int off = blk_off(t % MF_NBUF, par);
        if (t > 0 || par != 0) {
#pragma unroll
          for (int kk = 0; kk < NK; ++kk)
            sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ldk(off, kk), qf[kk], kk == 0 ? negm : sA, 0, 0, 0);
          if (2 * t + par >= n_plain) mask_block(2 * t + par, sA);
        }
        exp_half(sA, 0, pa);
        exp_half(sA, 1, pb);
        const bf16x8 b0 = __builtin_bit_cast(bf16x8, pa), b1 = __builtin_bit_cast(bf16x8, pb);
#pragma unroll
        for (int f = 0; f < NK; ++f)
          acc[f % NT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ldv(off, f), f < NT ? b0 : b1, acc[f % NT], 0, 0, 0);
      }
    } else if (ways == 2) {
      // ---- two waves to a row block: this one takes 32-key block `kpar` of every tile.  Both start from
      // the first block's maximum, so their sums need no rescaling when they meet.
      //   window 1: scores of tile t+1  | second half of tile t
      //   window 2: product of tile t   | first half of tile t+1
      // The barrier that lets tile t + 1 in stands at the start of the trip; every wave has finished tile
      // t - 1 by then.
      const int kofs = kpar * MF_BLOCK_BYTES;
      if (kpar != 0) {
#pragma unroll
        for (int kk = 0; kk < NK; ++kk)
          sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ldk(kofs, kk), qf[kk], kk == 0 ? negm : sA, 0, 0, 0);
        if (n_plain < 2) mask_block(1, sA);
      }
      exp_half(sA, 0, pa);
      auto trip = [&](int t, int s, floatx16& S_cur, floatx16& S_next, uintx4& P_cur, uintx4& P_next, auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        const int s1 = (s + 1) % MF_NBUF;
        if (MASKED) {
          next_arrival(t);
        } else {
          asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * MF_LOADS) : "memory");
          issue_full(t + 3, (s + 3) % MF_NBUF);
        }
#pragma unroll
        for (int kk = 0; kk < 2 * MF_AHEAD; ++kk) kf[kk] = ldk(blk_off(s1, 0) + kofs, kk);
        win_qk(blk_off(s1, 0) + kofs, blk_off(s, 0) + kofs, S_next, S_cur, 1, pb);
        if (MASKED && 2 * (t + 1) + kpar >= n_plain) mask_block(2 * (t + 1) + kpar, S_next);
        win_pv(blk_off(s, 0) + kofs, 0, P_cur, pb, S_next, 0, P_next, YES, NO);
      };
      int t = 0;
      for (; t + 6 < n_full; t += 4) {
        trip(t, 0, sA, sB, pa, pc, NO);
        trip(t + 1, 1, sB, sA, pc, pa, NO);
        trip(t + 2, 2, sA, sB, pa, pc, NO);
        trip(t + 3, 3, sB, sA, pc, pa, NO);
      }
      for (; t + 1 < n_tiles; ++t) {
        trip(t, t % MF_NBUF, sA, sB, pa, pc, YES);
        sA = sB;
        pa = pc;
      }
      const int off = blk_off(t % MF_NBUF, 0) + kofs;
      exp_half(sA, 1, pb);
#pragma unroll
      for (int f = 0; f < 2 * MF_AHEAD; ++f) vf[f] = ldv(off, f);
      win_pv(off, 0, pa, pb, sA, 0, pc, NO, NO);
    } else {
      exp_half(sA, 0, pa);
#pragma unroll
      for (int kk = 0; kk < 2 * MF_AHEAD; ++kk) kf[kk] = ldk(blk_off(0, 1), kk);
      // ---- one trip per tile t (blocks 2t and 2t + 1, ring slot s = t % 4); the barrier in its
      // middle lets tile t + 1 in
      //   window 1: scores of 2t+1      | second half of 2t
      //   window 2: product of 2t       | first half of 2t+1
      //   window 3: scores of 2t+2      | second half of 2t+1
      //   window 4: product of 2t+1     | first half of 2t+2
      // MASKED: blocks from n_plain on are masked and the tile that is requested may be any tile.
      auto trip = [&](int t, int s, auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        const int s1 = (s + 1) % MF_NBUF;
        win_qk(blk_off(s, 1), blk_off(s, 0), sB, sA, 1, pb);
        if (MASKED && 2 * t + 1 >= n_plain) mask_block(2 * t + 1, sB);
        if (MASKED) {
          next_arrival(t);
        } else {
          asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * MF_LOADS) : "memory");
          issue_full(t + 3, (s + 3) % MF_NBUF);
        }
        win_pv(blk_off(s, 0), blk_off(s1, 0), pa, pb, sB, 0, pc, YES, YES);
        win_qk(blk_off(s1, 0), blk_off(s, 1), sA, sB, 1, pb);
        if (MASKED && 2 * t + 2 >= n_plain) mask_block(2 * t + 2, sA);
        win_pv(blk_off(s, 1), blk_off(s1, 1), pc, pb, sA, 0, pa, YES, YES);
      };
      // Four tiles per round with the ring slots spelled out, while they and the tiles they request
      // (up to t + 6) are full prefix tiles: every LDS address is then a register plus an immediate.
      int t = 0;
      for (; t + 6 < n_full; t += 4) {
        trip(t, 0, NO);
        trip(t + 1, 1, NO);
        trip(t + 2, 2, NO);
        trip(t + 3, 3, NO);
      }
      for (; t + 1 < n_tiles; ++t) trip(t, t % MF_NBUF, YES);
      {  // last tile: nothing follows its odd block
        const int s = t % MF_NBUF;
        win_qk(blk_off(s, 1), blk_off(s, 0), sB, sA, 1, pb);
        if (2 * t + 1 >= n_plain) mask_block(2 * t + 1, sB);
        win_pv(blk_off(s, 0), 0, pa, pb, sB, 0, pc, YES, NO);
        exp_half(sB, 1, pb);
#pragma unroll
        for (int f = 0; f < 2 * MF_AHEAD; ++f) vf[f] = ldv(blk_off(s, 1), f);
        win_pv(blk_off(s, 1), 0, pc, pb, sB, 0, pa, NO, NO);
      }
    }
    l_sum = l0 + l1;
  } else {
    // no rows: this wave only moves tiles and meets the barriers
    for (int t = 0; t + 1 < n_tiles; ++t) next_arrival(t);
  }

  // ---- did the fixed reference hold?  (denominator of both half-waves; NaN counts as no)
  float l_tot = l_sum + __shfl_xor(l_sum, 32);
  if (wave_active && __ballot(!(l_tot < MF_SUM_LIMIT)) != 0ull && lane == 0) exact_flag = 1;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // also: every LDS read of the pass is done
  if (exact_flag != 0) {
    // ---- exact path (rare): the pass again, one block at a time, the reference following the
    // running maximum: classic online softmax, no overlap between the steps
    m_ref = 0.f;
    l_sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) negm[v] = 0.f;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tt][v] = 0.f;
    issue(0);
    if (n_tiles > 1) issue(1);
    first_arrival();
    for (int blk = 0; blk < n_blocks; ++blk) {
      // the barrier of next_arrival also keeps any wave from reading tile t + 1 before all of it is there
      if ((blk & 1) && blk + 1 < n_blocks) next_arrival(blk >> 1);
      if (!wave_active || kpar != 0) continue;  // (of two waves that share a row block the first does it all)
      const int off = blk_off((blk >> 1) % MF_NBUF, blk & 1);
      floatx16 S;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk)
        S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ldk(off, kk), qf[kk], kk == 0 ? negm : S, 0, 0, 0);
      if (blk >= n_plain) mask_block(blk, S);
      const float mx = row_max(S);
      if (blk == 0 || __ballot(mx > 0.f) != 0ull) {
        const float delta = (blk == 0 || mx > 0.f) ? mx : 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) S[v] -= delta;
        if (blk == 0) set_reference(delta);
        else move_reference(delta);
      }
      uintx4 P0, P1;
      l0 = 0.f;
      l1 = 0.f;
      exp_half(S, 0, P0);
      exp_half(S, 1, P1);
      l_sum += l0 + l1;
      const bf16x8 b0 = __builtin_bit_cast(bf16x8, P0), b1 = __builtin_bit_cast(bf16x8, P1);
#pragma unroll
      for (int f = 0; f < NK; ++f)
        acc[f % NT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ldv(off, f), f < NT ? b0 : b1, acc[f % NT], 0, 0, 0);
    }
    l_tot = l_sum + __shfl_xor(l_sum, 32);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  if (ksplit && !quarter) {
    // ---- the two waves of a row block swap halves of their columns through the (now free) tile ring:
    // each ends up with the sums of NT / 2 column blocks, kept in acc[0 .. NT / 2), and the denominator.
    // A wave's 8 NT KB of floats lie 16 bytes to a lane, so both sides move whole 1 KB pieces.
    float* const ex = reinterpret_cast<float*>(wave < 4 ? &lds_k[0][0] : &lds_v[0][0]);  // (each 64 KB: four waves)
    if (wave_active) {
      if (kpar != 0) {
#pragma unroll
        for (int tt = 0; tt < NT / 2; ++tt) {
          const floatx16 x = acc[tt];
          acc[tt] = acc[tt + NT / 2];
          acc[tt + NT / 2] = x;
        }
      }
#pragma unroll
      for (int tt = 0; tt < NT / 2; ++tt)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          float4 f = {acc[tt + NT / 2][4 * b], acc[tt + NT / 2][4 * b + 1], acc[tt + NT / 2][4 * b + 2], acc[tt + NT / 2][4 * b + 3]};
          *reinterpret_cast<float4*>(ex + (wave & 3) * 4096 + (tt * 4 + b) * 256 + lane * 4) = f;
        }
      ex[(wave & 3) * 4096 + 2048 + lane] = l_tot;
      if (kpar == 0) ex[(wave & 3) * 4096 + 2112 + lane] = m_ref;  // (the exact path moves the first wave's reference only)
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const int other = wave ^ (1 << pair_shift);  // (a wave without rows reads some wave's piece and drops it)
    const float* const from = reinterpret_cast<const float*>(other < 4 ? &lds_k[0][0] : &lds_v[0][0]) + (other & 3) * 4096;
#pragma unroll
    for (int tt = 0; tt < NT / 2; ++tt)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const float4 f = *reinterpret_cast<const float4*>(from + (tt * 4 + b) * 256 + lane * 4);
        acc[tt][4 * b] += f.x;
        acc[tt][4 * b + 1] += f.y;
        acc[tt][4 * b + 2] += f.z;
        acc[tt][4 * b + 3] += f.w;
      }
    l_tot += from[2048 + lane];
    if (kpar != 0) m_ref = from[2112 + lane];
    // (every wave has its sums before the staging below reuses the ring)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  if (shared_tail || quarter) {
    // ---- the waves that share a row block leave their sums in the (now free) V ring (quarter: the first four in
    // the K ring), 16 bytes to a lane, and each adds up its part of the columns, wave by wave in rising order.
    float* const den = reinterpret_cast<float*>(&anc[0]);  // [wave][denominators, reference maxima]
    const bool sharing = quarter ? wave_active : wave >= 4 && wave_active;
    auto left_by = [&](int w) { return reinterpret_cast<float*>(w < 4 ? lds_k[w] : lds_v[w - 4]); };
    if (sharing) {
      float* const ex = left_by(wave);
#pragma unroll
      for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          float4 f = {acc[tt][4 * b], acc[tt][4 * b + 1], acc[tt][4 * b + 2], acc[tt][4 * b + 3]};
          *reinterpret_cast<float4*>(ex + (tt * 4 + b) * 256 + lane * 4) = f;
        }
      den[wave * 128 + lane] = l_tot;
      den[wave * 128 + 64 + lane] = m_ref;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (sharing) {
      // the first of the sharing waves, and how far it is to the next one
      const int step = quarter ? 1 << pair_shift : blk_n - 4;
      const int first = quarter ? wave & (step - 1) : my_blk - blk0;
      const int keep = ways == 4 ? 1 : NT / 2;          // column blocks of this wave
      const int tt0 = kpar * keep;
      if (tt0 >= NT) {  // (head dimension 64: two column blocks for four waves)
        if (quarter) asm volatile("s_barrier" ::: "memory");
        return;
      }
      m_ref = den[first * 128 + 64 + lane];  // (the exact path moves the first wave's only)
      l_tot = 0.f;
      for (int w = 0; w < ways; ++w) l_tot += den[(first + w * step) * 128 + lane];
#pragma unroll
      for (int tt = 0; tt < NT / 2; ++tt) {
        if (tt >= keep) break;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[tt][v] = 0.f;
        for (int w = 0; w < ways; ++w) {
          const float* from = left_by(first + w * step) + (tt0 + tt) * 1024;
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const float4 f = *reinterpret_cast<const float4*>(from + b * 256 + lane * 4);
            acc[tt][4 * b] += f.x;
            acc[tt][4 * b + 1] += f.y;
            acc[tt][4 * b + 2] += f.z;
            acc[tt][4 * b + 3] += f.w;
          }
        }
      }
    }
    // (quarter: every wave has its sums before the staging below reuses the rings)
    if (quarter) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  if (!wave_active) return;

  // `NB` column blocks (acc[0 .. NB)) of this wave's 32 rows, from column col0 of the head's row on
  auto write_out = [&](auto nb, int col0) {
    constexpr int NB = decltype(nb)::value;
    constexpr int CPR = 4 * NB;  // 16-byte chunks of a row
    if (n_sp == 1) {
      // ---- results, sequence with a single split: normalised rows go out as bf16.  Each wave turns its
      // block around in LDS (the tile ring is free: every wave has passed the last barrier),
      // so that a lane stores 16 contiguous bytes and a store instruction covers whole rows.
      constexpr int ST_ROW = 64 * NB + 16;  // padded row: the 8-byte writes of 16 rows spread over all banks
      // (waves that share a block still read each other's sums in the V ring: they turn theirs around behind
      // the first four waves' rows)
      char* stage = shared_tail && wave >= 4 ? lds_k[wave - 4] + 32 * (64 * NT + 16) : wave < 4 ? lds_k[wave] : lds_v[wave - 4];
      static_assert(32 * (64 * 4 + 16) + 32 * (64 * 2 + 16) <= MF_TILE_BYTES, "two waves' rows in a tile buffer");
      const float inv = 1.f / l_tot;
#pragma unroll
      for (int tt = 0; tt < NB; ++tt)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int d0 = 32 * tt + 8 * b + 4 * half;
          floatx2 f01 = {acc[tt][4 * b] * inv, acc[tt][4 * b + 1] * inv};
          floatx2 f23 = {acc[tt][4 * b + 2] * inv, acc[tt][4 * b + 3] * inv};
          uint2 pk;
          pk.x = __builtin_bit_cast(unsigned, __builtin_convertvector(f01, bf16x2));
          pk.y = __builtin_bit_cast(unsigned, __builtin_convertvector(f23, bf16x2));
          *reinterpret_cast<uint2*>(stage + col * ST_ROW + d0 * 2) = pk;
        }
      const int r = row_base + col;
      if (h_lse && half == 0 && r < Rh && col0 == 0) {
        const int i = div_G(r), gi = r - i * Gh;
        h_lse[(int64_t)(n0 + i) * Hq + head0 + gi] = (m_ref + __log2f(l_tot)) * MF_LN2;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave's staging writes are in LDS
#pragma unroll
      for (int j = 0; j < CPR / 2; ++j) {
        const int row_l = (64 / CPR) * j + lane / CPR, chunk = lane % CPR;
        const int ro = row_base + row_l;
        const int i = div_G(ro < Rh ? ro : 0), gi = ro - i * Gh;
        if (ro < Rh) {
          const uint4 val = *reinterpret_cast<const uint4*>(stage + row_l * ST_ROW + chunk * 16);
          char* dst = static_cast<char*>(h_o) + ((int64_t)(n0 + i) * Hq + head0 + gi) * Q_ROW_BYTES + col0 * 2 + chunk * 16;
          // non-temporal: the rows start their way to memory now instead of waiting in L2 for the
          // write-back at the end of the kernel, when every workgroup's rows would go at once
          __builtin_nontemporal_store(__builtin_bit_cast(uintx4, val), reinterpret_cast<uintx4*>(dst));
        }
      }
    } else {
      // ---- this split's partial record: unnormalised accumulators, reference maximum, denominator
      const int r = row_base + col;
      if (r < Rh) {
        const int i = div_G(r), gi = r - i * Gh;
        const int64_t row = (int64_t)(n0 + i) * Hq + head0 + gi;
        constexpr int REC_D = 32 * NT;  // a record: o[REC_D], m, l, two pad floats
        float* rec = h_part + (row * h_sp_max + sp) * (REC_D + ATTN_REC_PAD);
#pragma unroll
        for (int tt = 0; tt < NB; ++tt)
#pragma unroll
          for (int b = 0; b < 4; ++b) {
            const int d0 = col0 + 32 * tt + 8 * b + 4 * half;
            float4 f = {acc[tt][4 * b], acc[tt][4 * b + 1], acc[tt][4 * b + 2], acc[tt][4 * b + 3]};
            *reinterpret_cast<float4*>(rec + d0) = f;
          }
        if (half == 0 && col0 == 0) {
          rec[REC_D] = m_ref * MF_LN2;
          rec[REC_D + 1] = l_tot;
        }
      }
    }
  };
  if (ways == 1) write_out(std::integral_constant<int, NT>{}, 0);
  else if (ways == 2 || NT == 2) write_out(std::integral_constant<int, NT / 2>{}, kpar * (16 * NT));
  else write_out(std::integral_constant<int, 1>{}, kpar * 32);
}

// `ev_start` / `ev_stop` (may be NULL): HIP events attached to this dispatch; the runtime stamps them
// when the kernel begins and ends, so their elapsed time is the kernel's own duration.
hs_status attn_mfma_launch(const AttnArgs& a, int max_tree_rows, hipStream_t stream, hipEvent_t ev_start,
                           hipEvent_t ev_stop) {
  const int n_rg_max = (a.G * max_tree_rows + MF_ROWS - 1) / MF_ROWS;
  dim3 grid((unsigned)(a.Hkv * n_rg_max * a.sp_max), (unsigned)a.B);
  if (a.n_tbl > 0) grid = dim3((unsigned)a.n_items << a.narrow, 1u);
  const bool once = n_rg_max == 1 && a.narrow == 0;  // every (sequence, head) is one row group: its keys have one reader
  const bool big = max_tree_rows > MF_MAX_M;
  const dim3 block(MF_THREADS);
  const bool share = a.share != 0 || a.narrow == 2;
#define MF_LAUNCH_AS(PAGED, ONCE, BIG, HALF, SHARE) \
  hipExtLaunchKernelGGL((k_attn_mfma<PAGED, ONCE, BIG, HALF, SHARE>), grid, block, 0, stream, ev_start, ev_stop, 0, a, n_rg_max)
#define MF_LAUNCH(PAGED, ONCE, BIG)                                 \
  do {                                                              \
    if (a.half && share) MF_LAUNCH_AS(PAGED, ONCE, BIG, true, true);   \
    else if (a.half) MF_LAUNCH_AS(PAGED, ONCE, BIG, true, false);      \
    else if (share) MF_LAUNCH_AS(PAGED, ONCE, BIG, false, true);       \
    else MF_LAUNCH_AS(PAGED, ONCE, BIG, false, false);                 \
  } while (0)
  if (a.block_table != nullptr) {
    if (big) MF_LAUNCH(true, false, true);
    else if (once) MF_LAUNCH(true, true, false);
    else MF_LAUNCH(true, false, false);
  } else {
    if (big) MF_LAUNCH(false, false, true);
    else if (once) MF_LAUNCH(false, true, false);
    else MF_LAUNCH(false, false, false);
  }
#undef MF_LAUNCH
#undef MF_LAUNCH_AS
  return launch_status("tree attention (mfma)");
}

}  // namespace hs
