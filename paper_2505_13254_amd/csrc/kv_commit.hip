// hs_kv_commit: the accepted path joins the KV cache (Section 2.1: what an accepted path means for
// the context of the next step; rows of rejected nodes go nowhere).
//
// Per sequence the K/V rows of the tree's root and of the accepted rows, in path order, are copied
// behind the used part of the sequence's cache region and the used length grows by their number.
// A copy of a few kilobytes per sequence: one workgroup per sequence, 16 bytes per lane and step.  It is a chain of trips to
// memory: the arguments; the lengths, offsets and the path's rows; the pages; the rows themselves, of a few accepted tokens all
// in one step.  (256 threads, the arguments and lengths one after the other, 64-bit divisions for rows and pages: 12 sequences, a
// few rows of 2 KB each, paged, 5.4 us a launch, now 5.1; 4 of 1 KB, dense, 3.5 and 2.4.  With 4 attention layers and commits 624.6 us, 617.9 now.)
#include "hs_common.h"

namespace hs {

// Workgroups of 1024 threads for up to one sequence to a compute unit, of 256 beyond that, where most of the threads of those of 1024 have no
// piece and only take their time to start.  1024 and 256 threads, us a call: 64 sequences, 4 rows of 2 KB 3.9 and 4.1, 6 of 10 KB 6.6 and 8.8; 256, 4 of
// 2 KB 4.4 and 4.7, 1 of 2 KB 4.1 and 3.8; 512, 2 of 1 KB 4.7 and 4.0; 1024, 2 of 1 KB 6.1 and 4.4; 4096, 1 of 2 KB 14.1 and 7.7, 6 of 256 bytes 13.8 and
// 7.2; but 512, 9 of 10 KB 33.1 and 37.4.  (A thread's later pieces found by 64-bit divisions, the page requested behind the row: 256 threads, paged, 600
// sequences, 61 rows of 2 KB 89 us, now 68.)
constexpr int KC_THREADS = 1024, KC_THREADS_MANY = 256;
constexpr int KC_MANY = 256;  // sequences

// block_table == NULL: sequence s owns tokens cache_offsets[s] .. cache_offsets[s+1] of the caches.
// Otherwise the caches are pools of pages of `page_tokens` tokens and token t of sequence s lives in
// page block_table[s * max_blocks + t / page_tokens].
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_kv_commit(const char* __restrict__ k_tree,
                                                          const char* __restrict__ v_tree,
                                                          const int32_t* __restrict__ node_offsets,
                                                          const int32_t* __restrict__ accept_path,
                                                          const int32_t* __restrict__ accept_len, int max_depth,
                                                          char* __restrict__ k_cache, char* __restrict__ v_cache,
                                                          const int64_t* __restrict__ cache_offsets,
                                                          const int32_t* __restrict__ block_table, int max_blocks,
                                                          int page_tokens, int64_t* __restrict__ cache_lens,
                                                          int row_bytes) {
  const int s = blockIdx.x, tid = threadIdx.x;
  const bool paged = block_table != nullptr;
  const int n0 = node_offsets[s], n1 = node_offsets[s + 1];
  const int64_t used = cache_lens[s];
  int n_acc = accept_len[s];
  const int64_t* const bounds = paged ? cache_lens : cache_offsets;  // (paged: read for nothing, but without a branch)
  const int64_t c_lo = bounds[s], c_hi = bounds[paged ? s : s + 1];
  asm volatile("" ::"s"(k_tree), "s"(v_tree), "s"(accept_path), "s"(max_depth), "s"(k_cache), "s"(v_cache), "s"(cache_offsets),
               "s"(max_blocks), "s"(page_tokens), "s"(row_bytes));
  const unsigned chunks = (unsigned)row_bytes / 16;  // 16-byte pieces of a token's K (or V) row
  const int32_t* const path = accept_path + (int64_t)s * max_depth;
  // the row of this thread's first piece comes with the lengths
  const unsigned t0 = (unsigned)tid / chunks;
  const int r0 = t0 >= 1 && t0 <= (unsigned)max_depth ? path[t0 - 1] : 0;
  asm volatile("" ::"s"(n0), "s"(n1), "s"(used), "s"(n_acc), "s"(c_lo), "s"(c_hi));  // (requested by here, all of them)
  const int64_t c0 = paged ? 0 : c_lo;
  const int64_t c1 = paged ? (int64_t)max_blocks * page_tokens : c_hi;
  const int M = n1 - n0;
  if (M <= 0) return;
  const int64_t room = c1 - c0 - used;
  n_acc = n_acc < 0 ? 0 : (n_acc > max_depth ? max_depth : n_acc);
  int64_t rows = 1 + n_acc;  // the root, then the accepted rows
  rows = rows > room ? (room > 0 ? room : 0) : rows;
  const bool small = (used + rows) >> 32 == 0;  // (a 64-bit division is a long sequence of instructions)
  const int32_t* const table = block_table + (int64_t)s * max_blocks;
  auto copy = [&](unsigned t, unsigned c, int r) {
    int64_t pos = c0 + used + t;  // token position in the caches
    if (paged) {
      const int64_t tok = used + t;
      const int64_t blk = small ? (int64_t)((unsigned)tok / (unsigned)page_tokens) : tok / page_tokens;
      pos = (int64_t)table[blk] * page_tokens + (tok - blk * page_tokens);
    }
    r = t == 0 || r < 0 ? 0 : (r >= M ? M - 1 : r);  // (a path entry outside the tree would be a caller's error)
    const int64_t src = ((int64_t)(n0 + r)) * row_bytes + c * 16, dst = pos * row_bytes + c * 16;
    const uint4 k = *reinterpret_cast<const uint4*>(k_tree + src), v = *reinterpret_cast<const uint4*>(v_tree + src);
    *reinterpret_cast<uint4*>(k_cache + dst) = k;
    *reinterpret_cast<uint4*>(v_cache + dst) = v;
  };
  unsigned t = t0, c = tid - t0 * chunks;
  if (t < rows) copy(t, c, r0);
  if (rows * chunks > THREADS) {
    // a thread's next pieces, THREADS apart each; the row and the page of a piece are requested together
    const unsigned dt = THREADS / chunks, dc = THREADS % chunks;
    for (;;) {
      t += dt;
      c += dc;
      if (c >= chunks) {
        c -= chunks;
        ++t;
      }
      if (t >= rows) break;
      copy(t, c, path[t > 0 ? t - 1 : 0]);
    }
  }
  __syncthreads();  // every thread has read the old length
  if (tid == 0) cache_lens[s] = used + rows;
}

}  // namespace hs

using namespace hs;

static hs_status kv_commit_impl(const void* k_tree, const void* v_tree, const int32_t* node_offsets,
                                const int32_t* accept_path, const int32_t* accept_len, int32_t max_depth, void* k_cache,
                                void* v_cache, const int64_t* cache_offsets, const int32_t* block_table,
                                int32_t max_blocks, int32_t page_tokens, int64_t* cache_lens, int32_t B, int32_t Hkv,
                                int32_t D, hs_dtype dt, hs_stream stream) {
  HS_REQUIRE(B >= 0 && Hkv >= 1 && D >= 1 && max_depth >= 1, HS_ERR_SHAPE, "hs_kv_commit: B=%d Hkv=%d D=%d max_depth=%d",
             B, Hkv, D, max_depth);
  HS_REQUIRE(dt == HS_F32 || dt == HS_BF16, HS_ERR_SHAPE, "hs_kv_commit: unknown dtype %d", (int)dt);
  const int64_t row_bytes = (int64_t)Hkv * D * (dt == HS_F32 ? 4 : 2);
  HS_REQUIRE(row_bytes % 16 == 0 && row_bytes < ((int64_t)1 << 30), HS_ERR_UNSUPPORTED,
             "hs_kv_commit: a token's K row (%lld bytes) must be a multiple of 16 bytes", (long long)row_bytes);
  if (B == 0) return HS_OK;
  HS_REQUIRE(k_tree && v_tree && node_offsets && accept_path && accept_len && k_cache && v_cache &&
                 (cache_offsets || block_table) && cache_lens,
             HS_ERR_NULL, "hs_kv_commit: NULL argument");
  auto aligned16 = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  HS_REQUIRE(aligned16(k_tree) && aligned16(v_tree) && aligned16(k_cache) && aligned16(v_cache), HS_ERR_UNSUPPORTED,
             "hs_kv_commit: tensors must be 16-byte aligned");
#define KC_LAUNCH(T)                                                                                              \
  hipLaunchKernelGGL(k_kv_commit<T>, dim3((unsigned)B), dim3(T), 0, static_cast<hipStream_t>(stream),               \
                     static_cast<const char*>(k_tree), static_cast<const char*>(v_tree), node_offsets, accept_path, \
                     accept_len, max_depth, static_cast<char*>(k_cache), static_cast<char*>(v_cache), cache_offsets, \
                     block_table, max_blocks, page_tokens, cache_lens, (int)row_bytes)
  if (B <= KC_MANY) KC_LAUNCH(KC_THREADS);
  else KC_LAUNCH(KC_THREADS_MANY);
#undef KC_LAUNCH
  return launch_status("kv commit");
}

extern "C" hs_status hs_kv_commit(const void* k_tree, const void* v_tree, const int32_t* node_offsets,
                                  const int32_t* accept_path, const int32_t* accept_len, int32_t max_depth,
                                  void* k_cache, void* v_cache, const int64_t* cache_offsets, int64_t* cache_lens,
                                  int32_t B, int32_t Hkv, int32_t D, hs_dtype dt, hs_stream stream) {
  clear_error();
  HS_REQUIRE(B == 0 || cache_offsets, HS_ERR_NULL, "hs_kv_commit: NULL cache_offsets");
  return kv_commit_impl(k_tree, v_tree, node_offsets, accept_path, accept_len, max_depth, k_cache, v_cache,
                        cache_offsets, nullptr, 0, 1, cache_lens, B, Hkv, D, dt, stream);
}

extern "C" hs_status hs_kv_commit_paged(const void* k_tree, const void* v_tree, const int32_t* node_offsets,
                                        const int32_t* accept_path, const int32_t* accept_len, int32_t max_depth,
                                        void* k_pages, void* v_pages, const int32_t* block_table, int32_t max_blocks,
                                        int32_t page_tokens, int64_t* cache_lens, int32_t B, int32_t Hkv, int32_t D,
                                        hs_dtype dt, hs_stream stream) {
  clear_error();
  HS_REQUIRE(page_tokens >= 1 && max_blocks >= 0, HS_ERR_SHAPE, "hs_kv_commit_paged: page_tokens=%d max_blocks=%d",
             page_tokens, max_blocks);
  HS_REQUIRE(B == 0 || block_table, HS_ERR_NULL, "hs_kv_commit_paged: NULL block_table");
  return kv_commit_impl(k_tree, v_tree, node_offsets, accept_path, accept_len, max_depth, k_pages, v_pages, nullptr,
                        block_table, max_blocks, page_tokens, cache_lens, B, Hkv, D, dt, stream);
}
