// What the attention kernels of both directions share: operand types, the chain of matrix instructions, partial results in memory.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>

namespace bbm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int V>
struct IntC {
  static constexpr int value = V;
};

// A kernel's arguments where they lie in memory (its only parameter, at the start of the argument segment).  Taken by value they are
// read into scalar registers when the kernel starts, more than there are, and kept in lanes of vector registers for the next item:
// 110-160 lane accesses before the backward kernels' first matrix instruction, 20-90 this way, where they are read again where they
// are wanted.
template <typename Params>
using InPlace = const Params __attribute__((address_space(4)))*;
template <typename Params>
__device__ __forceinline__ InPlace<Params> kernel_args() { return (InPlace<Params>)__builtin_amdgcn_kernarg_segment_ptr(); }
// A pointer of the arguments points to global memory (the compiler cannot see that, and would take it for one into LDS as well).
template <typename T>
__device__ __forceinline__ T* global(T* p) {
  return (T*)(T __attribute__((address_space(1)))*)p;
}

__device__ __forceinline__ uint32_t scalar(uint32_t uniform) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)uniform); }

__device__ __forceinline__ float partner_sum(float x) {
  // lanes l and l^32 exchange: swap(x, x) gives {x[l%32], x[l%32 + 32]} in some order on every lane
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// A chain of COUNT matrix instructions (or groups of them) whose LDS operands are read R instructions ahead: load(n) reads the
// operand of instruction n, mul(n, operand) issues it, between(n) is whatever is to be issued behind it.  Left alone the
// compiler reads one operand, waits, multiplies and only then reads the next, so that every matrix instruction stands behind
// a whole LDS latency; the scheduling barriers keep it from going back to that order where registers are short.
// (n comes as a type, IntC<n>: the chain has to be unrolled whole, longer than the compiler unrolls a loop.)
template <typename F, int... N>
__device__ __forceinline__ void for_each_n(F f, std::integer_sequence<int, N...>) {
  (f(IntC<N>{}), ...);
}
template <int COUNT, int R, typename Load, typename Mul, typename Between>
__device__ __forceinline__ void mfma_ring(Load load, Mul mul, Between between) {
  bf16x8 f[R];
  for_each_n([&](auto n) { f[decltype(n)::value] = load(n); }, std::make_integer_sequence<int, R>{});
  __builtin_amdgcn_sched_barrier(0);
  for_each_n(
      [&](auto i) {
        constexpr int n = decltype(i)::value;
        mul(i, f[n % R]);
        if constexpr (n + R < COUNT) f[n % R] = load(IntC<n + R>{});
        between(i);
        __builtin_amdgcn_sched_barrier(0);
      },
      std::make_integer_sequence<int, COUNT>{});
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
// The first `rows` (0 .. 32) rows of a 32 x D bf16 slab from LDS, where 16-byte chunk c of row r sits at chunk position c ^ (r % (D / 8)),
// to memory as whole rows; row0, chunk: this lane's place in a piece of 1 KiB.  Rows past those lie outside the buffer: a branch
// and a 64-bit address a piece instead took a third of the epilogue's instructions (this alone, forward in us: 1 x 2 x 256
// 6.91 -> 6.76 at D = 64, 8.98 -> 8.76 at D = 128, packed sequences of 3001 13.44 -> 13.20, 23.7 -> 23.2).
template <int D>
__device__ __forceinline__ void store_rows(const __bf16* stage, __bf16* dst, int rows, int row0, int chunk) {
  constexpr int RC = D / 8, RPB = 64 / RC;
  const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(dst, 0, (int)scalar((uint32_t)(rows * D * 2)), 0x00027000);
  const int at = (row0 * D + chunk * 8) * 2;
#pragma unroll
  for (int n = 0; n < 32 / RPB; ++n) {
    const int r = n * RPB + row0;
    const u32x4 x = *reinterpret_cast<const u32x4*>(stage + r * D + (chunk ^ (r % RC)) * 8);
    __builtin_amdgcn_raw_buffer_store_b128(x, out, at + n * RPB * D * 2, 0, 0);
  }
}
__device__ __forceinline__ void hand_over() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

}  // namespace bbm
