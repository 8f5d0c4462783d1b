// Internal helpers shared by the translation units of libbbm (no kernels live here).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "bbm.h"

namespace bbm {

// Records a thread-local message and returns `code` so call sites can `return fail(...)`.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Checks the launch status of the kernel just enqueued.
inline int launch_status(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(BBM_EHIP, "%s: %s", what, hipGetErrorString(e));
  return BBM_OK;
}

// Layout of the split schedule that bbm_build_sparse_index writes and bbm_attn_fwd (LIST mode) reads; int32 units.
//   [kSchedNParts]           number of parts (0 if no block row was cut)
//   [kSchedSplitT]           split threshold T: block rows with more than T list entries are cut into parts
//   [kSchedNCutRows]         number of block rows that were cut
//   [kSchedPartBase + 8*q]   part q (ordered by row, then part): row (= plane*nbr + block row), first entry in the
//                            plane's list, entries, part index, parts of the row, q of the row's first part, index
//                            of the row among the cut rows, list entry at the part's first position
//   [order_base + 4*(m*nbr + k)]  record of the k-th block row of plane m in launch order: block row, position of
//                            its first entry in the plane's list, entries, first list entry (-1 if none);
//                            order_base = kSchedPartBase + 8*Mb*nbr.  Launch order: groups of kSchedGroupRows
//                            consecutive rows if T is at its floor, else single rows; the group holding the longest row
//                            first (ties: higher rows first), inside a group the longest row first (ties: higher row first); planes with more
//                            than kSchedMaxSortRows block rows are simply listed from the last row to the first
constexpr int kSchedNParts = 0, kSchedSplitT = 1, kSchedNCutRows = 2;
constexpr int kSchedPartBase = 8;
constexpr int kSchedPartInts = 8;
constexpr int kSchedMinSplit = 32;
constexpr int kSchedMaxSortRows = 4096;
constexpr int kSchedRowInts = 4;
constexpr int kSchedGroupRows = 4;
// Column schedule of the backward pass (bbm_build_col_index writes it, bbm_attn_bwd reads it): the same header and
// 8-int part records with block columns in place of block rows, launch-order records of single columns (longest
// first; ties: higher column first) after the Mb*nbc part slots, and a lower floor of the
// split threshold (a column entry stands for Br/64 sub-tiles of twice the work of a forward tile).
constexpr int kColSchedMinSplit = 16;
__host__ __device__ inline int64_t sched_order_base(int64_t Mb, int64_t nbr) { return kSchedPartBase + kSchedPartInts * Mb * nbr; }
__host__ __device__ inline int64_t sched_ints(int64_t Mb, int64_t nbr) { return sched_order_base(Mb, nbr) + kSchedRowInts * Mb * nbr; }

// Launch order of the attention kernels: how many (batch, head) planes have their block rows (columns) interleaved
// inside one XCD's contiguous share of the launch.  Interleaving lets the long rows of several planes start first
// (packed short sequences: 20-35 % faster with 8 planes than with 1), but the work-groups of one XCD then stream the
// tensors of all those planes through its 4 MiB L2: with heads of 4 MiB (N = 8192, d = 128, dense) 8 planes made
// 41 % of the dK/dV kernel's L2 requests miss against 4 % with one plane, and cost 4-5 % of the run time.  So large
// heads are not interleaved.  `streamed_bytes` is what one plane's work-groups read over and over (K and V, or Q
// and dO, of one head).
constexpr int64_t kInterleaveMaxHeadBytes = 2 << 20;
inline int32_t interleaved_planes(int64_t planes, int64_t streamed_bytes) {
  if (streamed_bytes >= kInterleaveMaxHeadBytes) return 1;
  const int64_t g = planes / 8;
  return (int32_t)(g < 1 ? 1 : g > 8 ? 8 : g);
}

// Partial results pass from one work-group to another through memory that both reach past their XCD's own cache: they are written
// through and read around it (the cache policy of an access of agent scope).  A device-wide release fence instead makes the cache
// write back everything it holds, once per work-group and one after the other: with 512 work-groups parking 64 KiB each they stood
// there for 16-22 us.  hand_over() completes a work-group's stores before any of its threads goes on.
// A record: [register / 4][lane][register % 4], 16 bytes a lane and access; `at` is this lane's place, LANES the number of them.
// Plain loads with a cache policy, not atomic ones: those the compiler issues one at a time where it can reuse the address
// register, each with a wait behind it, some 120 round trips past the cache for a row of seven parts at d = 64.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kAgentScope = 16;  // sc1

__device__ __forceinline__ __amdgpu_buffer_rsrc_t record_rsrc(const float* record, int floats) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(record), 0, floats * 4, 0x00027000);
}
template <int DB, int LANES>
__device__ __forceinline__ void store_record(__amdgpu_buffer_rsrc_t r, int at, const f32x16 (&acc)[DB]) {
#pragma unroll
  for (int n = 0; n < 4 * DB; ++n) {
    u32x4 x;
    for (int e = 0; e < 4; ++e) x[e] = __float_as_uint(acc[n / 4][n % 4 * 4 + e]);
    __builtin_amdgcn_raw_buffer_store_b128(x, r, at * 16, n * LANES * 16, kAgentScope);
  }
}
template <int DB, int LANES>
__device__ __forceinline__ void load_record(__amdgpu_buffer_rsrc_t r, int at, f32x16 (&x)[DB]) {
#pragma unroll
  for (int n = 0; n < 4 * DB; ++n) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, at * 16, n * LANES * 16, kAgentScope);
    for (int e = 0; e < 4; ++e) x[n / 4][n % 4 * 4 + e] = __uint_as_float(v[e]);
  }
}
// The pair of floats that follows the accumulators in a record that has one.
template <int DB, int LANES>
__device__ __forceinline__ void store_pair(__amdgpu_buffer_rsrc_t r, int at, float a, float b) {
  __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(a), __float_as_uint(b)}, r, at * 8, 16 * DB * LANES * 4, kAgentScope);
}
template <int DB, int LANES>
__device__ __forceinline__ float2 load_pair(__amdgpu_buffer_rsrc_t r, int at) {
  const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, at * 8, 16 * DB * LANES * 4, kAgentScope);
  return make_float2(__uint_as_float(x[0]), __uint_as_float(x[1]));
}
// add(record k, its pair) for each of the `count` records `stride` floats apart, in this order; BATCH records' loads in flight
// together.  (Without the scheduling barrier the compiler moves the loads down to where they are used.)
template <int DB, int LANES, bool PAIR, int BATCH, typename Add>
__device__ __forceinline__ void for_records(const float* first, int64_t stride, int count, int at, Add add) {
  static_assert(BATCH == 1 || BATCH == 2, "one record, or two");
  constexpr int FLOATS = (16 * DB + (PAIR ? 2 : 0)) * LANES;
  f32x16 x[DB], y[DB];
  float2 px = make_float2(0.0f, 0.0f), py = px;
  auto load = [&](int k, f32x16 (&rec)[DB], float2& pair) {
    const __amdgpu_buffer_rsrc_t r = record_rsrc(first + k * stride, FLOATS);
    if constexpr (PAIR) pair = load_pair<DB, LANES>(r, at);
    load_record<DB, LANES>(r, at, rec);
  };
  int k = 0;
#pragma unroll 1
  for (; k < (BATCH == 2 ? count & 1 : count); ++k) {
    load(k, x, px);
    __builtin_amdgcn_sched_barrier(0);
    add(x, px);
  }
#pragma unroll 1
  for (; BATCH == 2 && k < count; k += 2) {
    load(k, x, px);
    load(k + 1, y, py);
    __builtin_amdgcn_sched_barrier(0);
    add(x, px);
    add(y, py);
  }
}
__device__ __forceinline__ void hand_over() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

}  // namespace bbm
