// Internal helpers shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>

#include "heterospec.h"

namespace hs {

// Records the message for hs_last_error() and returns `st`.
hs_status fail(hs_status st, const char* fmt, ...);
void clear_error();

inline hs_status launch_status(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HS_ERR_RUNTIME, "%s: %s", what, hipGetErrorString(e));
  return HS_OK;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Carves 256-byte aligned pieces out of the caller's workspace.
struct Carver {
  char* base;
  size_t used = 0;
  explicit Carver(void* p) : base(static_cast<char*>(p)) {}
  template <typename T>
  T* take(size_t n) {
    T* r = reinterpret_cast<T*>(base + used);
    used += align_up(n * sizeof(T), 256);
    return r;
  }
};

// Row scan shared by hs_draft_entropy_topk and hs_verify_accept (defined in entropy_topk.hip).
// What of a call, besides R, V and K, decides how its rows are cut.
struct ScanRows {
  bool aligned;     // scan_aligned
  bool sparse;      // with `row_active`
  bool pairs_only;  // with `slices`, pairs_only
};
// Every row begins at a multiple of 16 bytes.  (logits2 may be NULL)
inline bool scan_aligned(const float* logits, const float* logits2, int64_t row_stride) {
  return reinterpret_cast<uintptr_t>(logits) % 16 == 0 && reinterpret_cast<uintptr_t>(logits2) % 16 == 0 && row_stride % 4 == 0;
}
// row_topk_workspace never falls as R grows (a workspace for R rows holds fewer); a call asks for row_topk_need.
size_t row_topk_workspace(int R, int V, int K, bool sparse);
size_t row_topk_need(int R, int V, int K, const ScanRows& rows);
// `slices` (may be NULL): when the rows had to be cut into slices, the merge launch is left to the
// caller, who receives the per-slice results instead: entry (row * count + slice) * K + k of `key` is
// the slice's k-th best pair as one number: of two keys the larger is the better pair, the lower half
// is 2^32 - 1 - index, 0 is an unused entry.  count == 1 means the outputs were written in full.
// `row_active` (device, may be NULL): one byte per row; a row whose byte is 0 is neither read nor
// written.  `row_index` (device, may be NULL): result row r is computed from logits row
// row_index[r]; a negative entry leaves row r's results as they are.  `logits2` (may be NULL):
// rows rows1, rows1 + 1, ... are rows 0, 1, ... of this second array (same row stride).
// `prepared`: the workspace was cleared by hs_workspace_prepare and has since been used by completed
// calls of this kind only; rows cut into slices are then merged by the scan's own launch.
struct ScanSlices {
  const unsigned long long* key;
  int count;
  bool pairs_only = false;  // in: the caller wants the slices' best pairs only, no softmax statistics
};
constexpr int ROW_SCAN_MAX = 65535;  // rows of a scan (they are a grid's second dimension)
hs_status row_topk_launch(const float* logits, int64_t row_stride, int R, int V, int K, float temperature,
                          int32_t* topk_idx, float* topk_logp, float* ent_topk, float* ent_full, float* lse,
                          void* workspace, hipStream_t stream, ScanSlices* slices = nullptr,
                          const uint8_t* row_active = nullptr, const int32_t* row_index = nullptr,
                          const float* logits2 = nullptr, int rows1 = 0, bool prepared = false);

#define HS_REQUIRE(cond, st, ...) \
  do {                            \
    if (!(cond)) return ::hs::fail(st, __VA_ARGS__); \
  } while (0)

// ------------------------------------------------------------------ device helpers
#define HS_INF __builtin_huge_valf()

// Strict total order on (value, index): larger value first, then lower index.
__device__ __forceinline__ bool better(float av, int ai, float bv, int bi) {
  return av > bv || (av == bv && ai < bi);
}

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Four neighbouring floats at any float's address: the type's alignment is an element's, and global memory takes wide
// accesses at any address.  (Rows that do not begin at multiples of 16 bytes read a value at a time: scan of 600 rows of 50257 logits
// 45.3 us, 33.1 now, of 50256 33.1; their ratio rule went without the sorted residual: 61 rows of 50257, whole step 215 us,
// 132 now.)
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load_float4(const float* p) {
  const float4_any f = *reinterpret_cast<const float4_any*>(p);
  return make_float4(f[0], f[1], f[2], f[3]);
}

// The same for data that nobody reads again.
__device__ __forceinline__ float4 stream_float4(const float* p) {
  const float4_any f = __builtin_nontemporal_load(reinterpret_cast<const float4_any*>(p));
  return make_float4(f[0], f[1], f[2], f[3]);
}

// Running softmax statistics of a set of raw logits x, with y = x * inv_t:
//   m  = max x (raw units, so comparisons stay exact);
//   s1 = sum exp(y - y_max) over all elements but ONE instance of the max;
//   t  = sum exp(y - y_max) (y - y_max)   (every term <= 0).
// Keeping the max's own unit out of s1 keeps entropy and lse accurate for nearly one-hot rows:
//   lse = m * inv_t + log1p(s1),  entropy = log1p(s1) - t / (1 + s1).
struct Stats {
  float m, s1, t;
};

__device__ __forceinline__ Stats stats_empty() { return Stats{-HS_INF, 0.f, 0.f}; }

// Reductions over the 64 lanes of a wave with DPP moves (no LDS traffic): partial results travel
// right inside each row of 16 lanes, then from row to row; lane 63 ends up with the total, which
// is broadcast.  `idle` is what a lane without a source takes (the identity of the operation).
template <typename Op>
__device__ __forceinline__ float wave_reduce_dpp(float x, float idle, Op op) {
  const int id = __builtin_bit_cast(int, idle);
#define HS_DPP_STEP(ctrl, rows, banks)                                                                        \
  x = op(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(id, __builtin_bit_cast(int, x), ctrl, rows, \
                                                                  banks, false)))
  HS_DPP_STEP(0x111, 0xf, 0xf);  // row_shr:1
  HS_DPP_STEP(0x112, 0xf, 0xf);  // row_shr:2
  HS_DPP_STEP(0x114, 0xf, 0xe);  // row_shr:4
  HS_DPP_STEP(0x118, 0xf, 0xc);  // row_shr:8
  HS_DPP_STEP(0x142, 0xa, 0xf);  // row_bcast:15
  HS_DPP_STEP(0x143, 0xc, 0xf);  // row_bcast:31
#undef HS_DPP_STEP
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
// Inclusive prefix sums over the lanes of a wave, same DPP steps: lane l receives x_0 + ... + x_l.
__device__ __forceinline__ int wave_prefix_sum(int x) {
#define HS_DPP_STEP(ctrl, rows, banks) x += __builtin_amdgcn_update_dpp(0, x, ctrl, rows, banks, false)
  HS_DPP_STEP(0x111, 0xf, 0xf);  // row_shr:1
  HS_DPP_STEP(0x112, 0xf, 0xf);  // row_shr:2
  HS_DPP_STEP(0x114, 0xf, 0xe);  // row_shr:4
  HS_DPP_STEP(0x118, 0xf, 0xc);  // row_shr:8
  HS_DPP_STEP(0x142, 0xa, 0xf);  // row_bcast:15
  HS_DPP_STEP(0x143, 0xc, 0xf);  // row_bcast:31
#undef HS_DPP_STEP
  return x;
}
__device__ __forceinline__ float wave_max(float x) {
  return wave_reduce_dpp(x, -HS_INF, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ float wave_sum(float x) {
  return wave_reduce_dpp(x, 0.f, [](float a, float b) { return a + b; });
}

// Loads and stores that are coherent across the chip's XCDs (each has an L2 of its own): relaxed
// atomics of device scope, which go past a stale or private cache line.  What workgroups of one
// launch use to hand their slices' results to each other: a fence that reaches the other XCDs
// would write back and invalidate a whole L2, and cost the scan several times its own duration.
__device__ __forceinline__ float ld_dev(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ unsigned long long ld_dev(const unsigned long long* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_dev(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_dev(unsigned long long* p, unsigned long long v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

}  // namespace hs
