// Backward pass of the fused masked attention (paper Sec. 3 "Flash Attention": the attention matrix is recomputed in
// the backward pass; Sec. 4: only non-zero blocks are visited and the element mask is applied only on partial ones).
//
// With P = softmax over the allowed keys (recomputed from the stored log-sum-exp), dP = dO V^T, D_i = <dO_i, O_i>,
// dS = P o (dP - D):   dV = P^T dO,   dK = scale * dS^T Q,   dQ = scale * dS K.
//
// Two kernels, both deterministic (no atomics):
//   dq kernel   one work-group per block row of Br = 32*NW queries, one lane per query (the layout of the forward
//               kernel): walks the row's list of key tiles, S^T = K Q^T and dP^T = V dO^T with the tile rows as the
//               A operand, dQ^T += K^T dS^T with K read through transposing LDS reads.  It also computes D_i and
//               leaves -D_i and -lse_i*log2(e) in the workspace for the second kernel.
//   dkv kernel  one work-group (4 waves) per block column of 64 keys, one lane per key and query half: walks the column's
//               list of query blocks in sub-tiles of 64 queries, S = Q K^T and dP = dO V^T with the tile rows as A operand,
//               dV^T += dO^T P and dK^T += Q^T dS with transposing LDS reads of the same two tiles.
// Both start the score accumulators at -lse (in exponent units) and the dP accumulators at -D, so that exp2 and one
// multiplication per element give P and dS.
#include "bbm_internal.h"
#include "bbm_mfma.h"

#include <algorithm>

namespace {

using bbm::bf16x2, bbm::bf16x4, bbm::bf16x8, bbm::f32x16, bbm::global, bbm::IntC, bbm::mfma_ring, bbm::partner_sum, bbm::s16x4, bbm::scalar;

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kWin = 128;                   // list entries per LDS window
constexpr uint32_t kNoTile = 0xffffffffu;

struct BwdParams {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  const __bf16* o;
  const __bf16* d_o;
  const float* lse;
  __bf16* dq;
  __bf16* dk;
  __bf16* dv;
  float* nl2;      // workspace [B*H*N]: -lse*log2(e), -inf for fully masked rows
  float* ndelta;   // workspace [B*H*N]: -<dO_i, O_i>
  const uint64_t* packed;  // [Mb][W][N]
  const int32_t* row_ptr;
  const uint32_t* col_idx;
  const int32_t* sched;    // may be NULL: block rows are then started from the last to the first
  const int32_t* col_ptr;
  const uint32_t* row_idx;
  int64_t N;
  int32_t H, Mb, nbr, nbc, W;
  int32_t total_wgs;
  int32_t G, Gc;    // (batch, head) planes whose block rows / block columns are interleaved in launch order
  int32_t br;       // query rows per block row
  float scale;
  float qscale;  // factor folded into the bf16 Q (dQ step) resp. K (dK/dV step) operand, see the forward kernel
  float rmul;    // EXACT instances: the rest of softmax_scale*log2(e), applied in fp32 inside the exponential; else 1
  // Cut block rows (dQ) and cut block columns (dK, dV): the split schedules (read-only), and in the caller's workspace
  // the work-queue state and the fp32 partial results of the parts.  Counters: [0] part items handed out, [1] leading
  // work-groups done, [8 + rho*hbp + hb] finished parts of cut row/column rho; all zero between calls.
  const int32_t* csched;   // column schedule; may be NULL (no column is cut then)
  int32_t* row_queue;
  int32_t* col_queue;
  float* row_partials;     // [(cut part)*hbp + hb][Br*D]
  float* col_partials;     // [(cut part)*hbp + hb][2][64*D]
  int32_t hbp;             // (batch, head) pairs per mask plane
  int32_t n_extra;         // leading work-groups that serve the queue of parts before their own row/column
};

// Sum over each group of RC = 8 or 16 consecutive lanes, in all of them.
template <int RC>
__device__ __forceinline__ float row_sum(float x) {
  auto other = [](float v, auto ctrl) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  x += other(x, IntC<0xB1>{});              // lane ^ 1
  x += other(x, IntC<0x4E>{});              // lane ^ 2
  x += other(x, IntC<0x141>{});             // mirrored within 8 lanes
  if constexpr (RC == 16) x += other(x, IntC<0x140>{});  // mirrored within 16 lanes
  return x;
}

typedef bbm::InPlace<BwdParams> Args;

// LDS layout of a 64-row x D tile, shared by every tile of both kernels.  One asynchronous copy instruction of a wave
// fills one 1 KiB block with RPB rows that lie NBLK rows apart: row r sits in block r % NBLK at slot r / NBLK; blocks
// are 1 KiB + 64 B apart, and the 16-byte chunk c of row r sits at chunk position c ^ ((r >> 2) & 3).  With that both
// access patterns are free of bank conflicts: 16 lanes reading the same chunk of 16 consecutive rows (A operand from
// tile rows), and 32 lanes reading 64 contiguous bytes of 4 consecutive rows (transposing read).
template <int D>
struct TL {
  static constexpr int RC = D / 8;          // 16-byte chunks per row
  static constexpr int RPB = 64 / RC;       // rows per 1 KiB block
  static constexpr int NBLK = 64 / RPB;     // blocks per tile
  static constexpr int TBLK = 512 + 32;     // block stride in elements
  static constexpr int ELEMS = NBLK * TBLK;
};

// Two floats rounded to bf16, the first in the low half; eight of them as a matrix operand.
__device__ __forceinline__ uint32_t pack(float a, float b) {
  const bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ bf16x8 operand(const uint32_t (&w)[4]) {
  const uint4 v = make_uint4(w[0], w[1], w[2], w[3]);
  return __builtin_bit_cast(bf16x8, v);
}

// The lane's number, found anew at each use: for what is needed once a step and not worth a register throughout the loop.
__device__ __forceinline__ int lane_now() {
  int x;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(x));
  return x;
}

// An asynchronous copy of SIZE bytes per lane into LDS, from byte `off` (per lane) of the `bytes` bytes at the wave-uniform p;
// lanes whose bytes lie past those write zeros (the bounds check of the buffer resource).  The buffer form also matters to the
// compiler: it counts the global form as possibly touching LDS through the flat path, and with one in flight it waits for ALL
// outstanding LDS reads at every use of one, which undoes the reads that run ahead (mfma_ring).
template <int SIZE>
__device__ __forceinline__ void copy_async(const void* p, int bytes, uint32_t off, void* dst) {
  static_assert(SIZE == 16 || SIZE == 4, "the builtin wants literal sizes");
  auto* const lds = (void __attribute__((address_space(3)))*)dst;
  const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)scalar(bytes), 0x00027000);
  if constexpr (SIZE == 16)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, lds, 16, off, 0, 0, 0);
  else
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, lds, 4, off, 0, 0, 0);
}

// Asynchronous global -> LDS copy of the first `rows` (0 .. 64) of the 64 rows of a [..][D] matrix at `tile`; zeros for the rest.
// This is copy instruction n of the NBLK / NW of a wave.  Lane l of a copy instruction lands at block base + 16*l, i.e. slot
// l / RC, chunk position l % RC.  One address register per lane (`base`, from tile_copy_base) serves all instructions: the XOR
// of the chunk position splits into a part of the lane and one of the block.
template <int D, int NW>
__device__ __forceinline__ uint32_t tile_copy_base(int wave, int lane) {
  using L = TL<D>;
  static_assert(L::NBLK % 16 == 0 || L::NBLK == 8, "(row >> 2) & 3 must be the XOR of the lane's part and the block's part");
  const int slot = lane / L::RC, pos = lane % L::RC;
  return (uint32_t)((wave + L::NBLK * slot) * D + (pos ^ ((L::NBLK * slot >> 2) & 3)) * 8) * 2u;
}
template <int D, int NW>
__device__ __forceinline__ void tile_copy_piece(const __bf16* __restrict__ tile, int rows, uint32_t base, __bf16* dst, int n, int wave) {
  using L = TL<D>;
  static_assert(L::NBLK % NW == 0, "tile must split evenly over the waves");
  const int blk = n * NW + wave;
  asm volatile("" : "+v"(base));  // one register throughout the tile loop, not one per block
  copy_async<16>(tile, rows * D * 2, (base ^ (uint32_t)(((blk >> 2) & 3) << 4)) + n * NW * D * 2, dst + blk * L::TBLK);
}
// How many of the 64 rows from row0 on lie below N.  (A scalar by force: the compiler clamps in a vector register, and a buffer
// resource in one costs a loop around every copy.)
__device__ __forceinline__ int rows_of_tile(int row0, int N) { return (int)scalar(max(0, min(64, N - row0))); }

// Per-lane base addresses (in elements) of the two read patterns.
template <int D>
struct TileAddr {
  int ra[2];  // A operand from tile rows: row 32*blk + lane%32, chunk 2t + lane/32; ra[t & 1] + (t >> 1)*32 + blk*(32/NBLK)*D
  int ta[2];  // transposing read of 16-row step u, half a, column block db: ta[a] + u*(D == 64 ? 2*D : D) + db*32
  __device__ __forceinline__ void init(int lane) {
    using L = TL<D>;
    const int lq = lane & 31, hh = lane >> 5;
    const int hq = (lq >> 2) & 3;
    const int rowbase = (lq % L::NBLK) * L::TBLK + (lq / L::NBLK) * D;
    const int x = hh ^ (hq & 1), y = hq >> 1;
    ra[0] = rowbase + (2 * y + x) * 8;
    ra[1] = rowbase + (2 * (1 ^ y) + x) * 8;
    const int vy = (lane & 15) >> 2, vg = (lane >> 4) & 1, vx = (lane & 3) >> 1;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int blockrow = D == 64 ? (4 * hh + vy) * L::TBLK + a * D : (8 * a + 4 * hh + vy) * L::TBLK;
      ta[a] = blockrow + (2 * (vg ^ a) + (vx ^ hh)) * 8 + 4 * (lane & 1);
    }
  }
  __device__ __forceinline__ bf16x8 row_frag(const __bf16* tile, int blk, int t) const {
    using L = TL<D>;
    return *reinterpret_cast<const bf16x8*>(tile + ra[t & 1] + (t >> 1) * 32 + blk * (32 / L::NBLK) * D);
  }
  // rows 16u + 8a + 4*(lane/32) + 0..3 (a = 0, 1) of column 32*db + lane%32: the order in which a lane's accumulator
  // registers 8*(u%2) .. 8*(u%2)+7 of row block u/2 list the rows of a 32x32 product
  __device__ __forceinline__ bf16x8 tr_frag(const __bf16* tile, int u, int db) const {
    s16x4 part[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
      part[a] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (s16x4 __attribute__((address_space(3)))*)(tile + ta[a] + u * (D == 64 ? 2 * D : D) + db * 32));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// acc * mult, rounded to bf16, to rows row0 .. of a [N][D] matrix: lane l holds row l%32 of the wave's 32-row slab,
// columns 32*db + 8*(e/4) + 4*(l/32) + e%4.  The slab is staged in LDS (`stage`, 32*D elements, this wave's own) so
// that the global stores are whole rows: 16-byte chunk ch of row r sits at chunk position ch ^ (r % RC).  (With the forward's
// store_rows, by buffer, more registers of these kernels lie in scratch memory: 1 to 2 % slower at D = 64.)
template <int D>
__device__ __forceinline__ void store_slab(const f32x16 (&acc)[D / 32], float mult, __bf16* stage, __bf16* __restrict__ dst,
                                           int row0, int N, int lane) {
  using L = TL<D>;
  // behind an optimisation barrier: otherwise the staging addresses are hoisted out of the loop over items and stay in
  // registers (or in scratch memory) throughout the tile loop
  asm volatile("" : "+v"(lane));
  const int lq = lane & 31, hh = lane >> 5, gro = lane / L::RC, gco = lane % L::RC;
#pragma unroll
  for (int db = 0; db < D / 32; ++db) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bf16x4 ov;
      for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(acc[db][4 * g + e] * mult);
      *reinterpret_cast<bf16x4*>(stage + lq * D + (((4 * db + g) ^ (lq % L::RC)) * 8) + 4 * hh) = ov;
    }
  }
  __bf16* og = dst + (int64_t)row0 * D;
#pragma unroll
  for (int n = 0; n < 32 / L::RPB; ++n) {
    const int r = n * L::RPB + gro;
    const bf16x8 ov = *reinterpret_cast<const bf16x8*>(stage + r * D + ((gco ^ (r % L::RC)) * 8));
    if (row0 + r < N) *reinterpret_cast<bf16x8*>(og + r * D + gco * 8) = ov;
  }
}

// (On the bits: the kernels are compiled with a flag that lets the compiler take any number for not a NaN.)
__device__ __forceinline__ bool is_nan(float x) {
  uint32_t bits = __float_as_uint(x);
  asm volatile("" : "+v"(bits));
  return (bits & 0x7fffffffu) > 0x7f800000u;
}

// The `bytes` bytes at the wave-uniform p: loads past them give zeros, stores are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)scalar(bytes), 0x00027000);
}

// XCD-aware logical work-group id: work-groups are handed to the 8 XCDs round-robin; give each XCD a contiguous range
// of logical ids so that the work-groups of one head (which share its tensors) meet in one XCD's L2.
__device__ __forceinline__ int logical_wg(int wg, int total) {
  const int xcd = wg & 7, slot = wg >> 3;
  const int per = total >> 3, rem = total & 7;
  return xcd * per + (xcd < rem ? xcd : rem) + slot;
}

// ------------------------------------------------------------------------------------------------------------------
// dQ (and D, and the negated statistics for the dK/dV kernel)
// ------------------------------------------------------------------------------------------------------------------
// One work-group per (block row, batch, head).  The first P.n_extra work-groups, before turning to their own block
// row, take the parts of the block rows which the split schedule cut from a queue; the work-group that completes a
// row's last part adds the parts up in part order and writes the row, and the row's own work-group only writes the
// statistics.
// EXACT (softmax scales sharper than 1/sqrt(d)): only the power-of-two part of softmax_scale*log2(e) is folded into
// the bf16 operand, the rest multiplies the recomputed score inside the exponential, as in the forward kernel.
// Kernel time with the copies spread, the phases in one chain, one loop for parts and own row and the rows of Q, dO and O fetched
// whole, against each of these not so: packed sequences of 4096, D = 64, 65.1 -> 55.8 us, of 3001, D = 128, 40.7 -> 35.9; 2 x 32
// heads of 8192 causal tokens, D = 128, 1470 -> 1400; 4 x 16 of 4096, D = 64, 226 -> 220 (exponentials beside the matrix pipe).
template <int D, int NW, bool EXACT>
__global__ __launch_bounds__(NW * 64, (D == 128 && NW >= 4) ? 2 : (D == 64 && NW == 4) ? 3 : 1) void attn_bwd_dq_kernel(const BwdParams) {
  Args P = bbm::kernel_args<BwdParams>();
  using L = TL<D>;
  constexpr int NT = NW * 64;
  constexpr int BR = NW * 32;
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int kRing = 3;
  constexpr int REGS = DB * 16;
  static_assert(2 * 32 * D <= L::ELEMS && NW <= 8, "two 32 x D output slabs must fit in each tile buffer");

  __shared__ __attribute__((aligned(16))) __bf16 k_s0[L::ELEMS];
  __shared__ __attribute__((aligned(16))) __bf16 k_s1[L::ELEMS];
  __shared__ __attribute__((aligned(16))) __bf16 v_s0[L::ELEMS];
  __shared__ __attribute__((aligned(16))) __bf16 v_s1[L::ELEMS];
  __shared__ uint32_t tiles_s[kWin + 4];
  __shared__ int item_s[2];
  __shared__ int again_s;            // a wave's sums are not numbers
  __shared__ float delta_s[NW][32];  // <dO, O> of the waves' rows

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, hh = lane >> 5;
  const int N = (int)P->N;
  const float c = P->qscale;
  const float rr = EXACT ? P->rmul : 1.0f;
  auto ex2 = [&](float x) { return __builtin_amdgcn_exp2f(EXACT ? rr * x : x); };

  // ---- per-item state
  int bh, m, i;
  int64_t head_off;
  const __bf16* __restrict__ Kg;
  const __bf16* __restrict__ Vg;
  const uint64_t* __restrict__ mrow;
  bf16x8 qf[KS], dof[KS];
  // Where there is room, 16 registers hold dP's start value throughout.  (With them the instance for sharper scales kept 63-76 others in
  // scratch memory: backward of packed sequences of 4096, 139-147 us, now 117.)
  constexpr bool START_REGS = D == 64 && !EXACT;
  f32x16 dp_init, dq[DB];
  float nl_lane = 0.0f, nd_lane = 0.0f;

  // (found anew for every item, see store_slab: kept across the merge of a cut row, some of it lay in scratch memory)
  TileAddr<D> A;
  uint32_t copy_base;

  auto tile_of = [](uint32_t e) { return (int)(e & 0x7fffffffu); };
  // e0: this step's list entry, e1: the next one's (as it came from LDS: made a scalar when the step starts)
  uint32_t e0, e1_v;
  uint64_t mw_nxt = 0;
  constexpr int LPW = L::NBLK / NW;  // copy instructions of a wave per tile
  // Tile e, n = 0 .. 2*LPW-1.  Keys past N come as zeros; their tile is never full, so the mask gives them probability 0.
  auto copy_piece = [&](uint32_t e, int rows, __bf16* kd, __bf16* vd, int n) {
    const int64_t at = (int64_t)tile_of(e) * 64 * D;
    if (n < LPW)
      tile_copy_piece<D, NW>(Kg + at, rows, copy_base, kd, n, wave);
    else
      tile_copy_piece<D, NW>(Vg + at, rows, copy_base, vd, n - LPW, wave);
  };
  auto copy_all = [&](uint32_t e, __bf16* kd, __bf16* vd) __attribute__((always_inline)) {
    const int rows = rows_of_tile(tile_of(e) * 64, N);
#pragma unroll
    for (int n = 0; n < 2 * LPW; ++n) copy_piece(e, rows, kd, vd, n);
  };
  auto request_mask = [&](uint32_t e) {
    if ((e >> 31) == 0) mw_nxt = mrow[(int64_t)tile_of(e) * N];
  };

  // One tile: a chain of matrix instructions over its two 32-key halves, S0, dP0, S1, dP1, dQ0, dQ1, with everything else
  // behind them: the next tile's copies behind S0, the exponentials of a half behind its dP, dS0 behind S1, dS1 behind dQ0.
  // The mask is in the start values of the scores, -inf where it has no bit.  If the product of such a masked pair overflows
  // (rows that nobody sees may hold anything finite) the sum is no number, and nor is then any of the query's dQ: the tiles are
  // gone through again with the mask behind the product (`late`).  Behind the product at once, the mask costs 2-7 % of the
  // backward pass at D = 64 and 1-4 % at D = 128, on tiles without a mask too.  The second pass costs nothing where none is needed, as
  // long as it leaves the first one its registers: operands one ahead, start values from one register, no argument kept for it.
  auto step = [&](auto pb, auto late, int it) __attribute__((always_inline)) {
    constexpr int PB = decltype(pb)::value;
    constexpr bool LATE = decltype(late)::value != 0;
    const uint64_t mw = mw_nxt;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    __bf16* const k_cur = PB ? k_s1 : k_s0;
    __bf16* const v_cur = PB ? v_s1 : v_s0;
    __bf16* const k_oth = PB ? k_s0 : k_s1;
    __bf16* const v_oth = PB ? v_s0 : v_s1;
    // The next tile's copies go out one by one between the matrix instructions of this one: requested in one go they fill
    // the memory pipe's queue, and every wave of the work-group stands there for 700-850 cycles of a step (D = 128).  Behind
    // the last tile they copy zero rows into buffers that nobody reads any more, cheaper than a branch around each.
    const uint32_t e1 = scalar(e1_v);
    const bool more = e1 != kNoTile, partial = (e0 >> 31) == 0;
    const int rows1 = more ? rows_of_tile(tile_of(e1) * 64, N) : 0;
    if (more) request_mask(e1);
    e0 = e1;
    e1_v = tiles_s[it + 2];
    // a partial tile in which none of this wave's 32 queries sees a key contributes exact zeros: skip it
    const bool live = !partial || __ballot(mw != 0ull) != 0ull;
    if (!live && more) copy_all(e1, k_oth, v_oth);
    if (!live) return;
    constexpr int N1 = KS, N2 = 2 * KS, N3 = 3 * KS, N4 = 4 * KS, N5 = N4 + 2 * DB, N6 = N5 + 2 * DB;
    constexpr int PER = D == 128 ? 4 : 8;  // elements behind a matrix instruction
    static_assert(PER * (KS - 2) >= 16 && PER * (2 * DB - 2) >= 16, "all 16 must find room");
    f32x16 s[2], dp[2];
    uint32_t dsf[2][2][4];  // dS of [half][16-key step], pairs of bf16
    float nl = nl_lane;
    if constexpr (LATE) asm volatile("" : "+v"(nl));  // (else the compiler keeps 16 copies of it in registers throughout)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      for (int e = 0; e < 16; ++e) s[kb][e] = nl;  // the scores start at the negated log-sum-exp
    auto mask_half = [&](int kb) {
      const uint32_t w = (uint32_t)(mw >> (32 * kb)) >> (4 * hh);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t keep = (uint32_t)((int32_t)(w << (31 - (8 * (e / 4) + e % 4))) >> 31);  // all ones iff the bit is set
        s[kb][e] = __uint_as_float((__float_as_uint(s[kb][e]) & keep) | (0xff800000u & ~keep));
      }
    };
    if (!LATE && partial) mask_half(0), mask_half(1);
    auto dp_start = [&](f32x16& acc) {
      if constexpr (START_REGS && !LATE) {
        acc = dp_init;
      } else {  // registers are short: the start value is kept as one scalar per lane
        float nd = nd_lane;
        if constexpr (LATE || D == 64) asm volatile("" : "+v"(nd));
        for (int e = 0; e < 16; ++e) acc[e] = nd;
      }
    };
    auto exps = [&](int kb, int slot) {
#pragma unroll
      for (int e = slot * PER; e < min(16, (slot + 1) * PER); ++e) s[kb][e] = ex2(s[kb][e]);
    };
    auto ds = [&](int kb, int slot) {
#pragma unroll
      for (int e = slot * PER; e < min(16, (slot + 1) * PER); e += 2)
        dsf[kb][e / 8][e % 8 / 2] = pack(s[kb][e] * dp[kb][e], s[kb][e + 1] * dp[kb][e + 1]);
    };
    mfma_ring<N6, LATE ? 1 : kRing>(
        [&](auto i) {
          constexpr int n = decltype(i)::value;
          if constexpr (n < N4)
            return A.row_frag(n / KS % 2 ? v_cur : k_cur, n / N2, n % KS);
          else
            return A.tr_frag(k_cur, (n - N4) / DB, (n - N4) % DB);
        },
        [&](auto i, bf16x8 f) {
          constexpr int n = decltype(i)::value;
          if constexpr (n == N1) dp_start(dp[0]);
          if constexpr (n == N3) dp_start(dp[1]);
          if constexpr (n < N4 && n / KS % 2 == 0) {
            s[n / N2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[n % KS], s[n / N2], 0, 0, 0);
          } else if constexpr (n < N4) {
            dp[n / N2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, dof[n % KS], dp[n / N2], 0, 0, 0);
          } else {
            constexpr int m = n - N4, u = m / DB;
            dq[m % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, operand(dsf[u / 2][u % 2]), dq[m % DB], 0, 0, 0);
          }
        },
        [&](auto i) {
          constexpr int n = decltype(i)::value;
          constexpr int GAP = 2 * LPW < KS ? KS / (2 * LPW) : 1;  // matrix instructions per copy
          if constexpr (n % GAP == 0 && n / GAP < 2 * LPW) copy_piece(e1, rows1, k_oth, v_oth, n / GAP);
          // a product is complete two matrix instructions after its last one was issued
          if constexpr (LATE && (n == N1 + 2 || n == N3 + 2))
            if (partial) mask_half(n / N2);
          if constexpr (n >= N1 + 2 && n < N2) exps(0, n - N1 - 2);
          if constexpr (n >= N2 + 2 && n < N3) ds(0, n - N2 - 2);
          if constexpr (n >= N3 + 2 && n < N4) exps(1, n - N3 - 2);
          if constexpr (n >= N4 + 2 && n < N5) ds(1, n - N4 - 2);
        });
  };

  // this lane's query: Q * scale * log2(e) and dO as B operands, D = <dO, O>, the negated statistics
  // between() is run when all of it has been asked for.
  auto begin_item = [&](bool write_stats, auto between) __attribute__((always_inline)) {
    head_off = (int64_t)bh * N * D;
    int ln = lane;
    asm volatile("" : "+v"(ln));  // keeps the addresses out of the loop over items, see store_slab
    A.init(ln);
    copy_base = tile_copy_base<D, NW>(wave, ln);
    const int wrow = i * BR + wave * 32, qrow = wrow + (ln & 31);
    const bool q_ok = qrow < N;
    mrow = global(P->packed) + (int64_t)m * P->W * N + (q_ok ? qrow : 0);
    // The wave's 32 rows of Q, dO and O are contiguous pieces of memory and are fetched as such, 1 KiB an instruction: a lane
    // that picks its row up in 16-byte pieces touches 64 cache lines an instruction.  Q goes to a staging slab in the tile
    // buffers (of parity 1 while at most four waves want one), dO follows through registers, where <dO, O> is formed; chunk c of row r sits at position c ^ (r % RC).
    __bf16* const stage = (wave / 2 == 0 ? k_s1 : wave / 2 == 1 ? v_s1 : wave / 2 == 2 ? k_s0 : v_s0) + (wave % 2) * 32 * D;
    const int g_row = ln / L::RC, g_chunk = ln % L::RC, rows = max(0, min(32, N - wrow));
    // (Rows past N come as zeros, by the bounds of the buffers.)
    bf16x8 gr[32 / L::RPB], orow[32 / L::RPB];
    const int64_t slab = head_off + (int64_t)wrow * D;
    const __amdgpu_buffer_rsrc_t do_r = buffer_of(P->d_o + slab, rows * D * 2), o_r = buffer_of(P->o + slab, rows * D * 2);
    const int64_t row_at = (int64_t)bh * N + wrow;
    const uint32_t lse_bits = __builtin_amdgcn_raw_buffer_load_b32(buffer_of(P->lse + row_at, rows * 4), (ln & 31) * 4, 0, 0);
#pragma unroll
    for (int n = 0; n < 32 / L::RPB; ++n) {
      const int r = n * L::RPB + g_row, at = (r * D + g_chunk * 8) * 2;
      copy_async<16>(P->q + slab, rows * D * 2, (uint32_t)(r * D + (g_chunk ^ (r % L::RC)) * 8) * 2u, stage + n * 512);
      gr[n] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(do_r, at, 0, 0));
      orow[n] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(o_r, at, 0, 0));
    }
    between();
#pragma unroll
    for (int n = 0; n < 32 / L::RPB; ++n) {
      float x = 0.0f;
      for (int e = 0; e < 8; ++e) x += (float)gr[n][e] * (float)orow[n][e];
      x = row_sum<L::RC>(x);
      if (g_chunk == 0) delta_s[wave][n * L::RPB + g_row] = x;
    }
    __builtin_amdgcn_s_waitcnt(0);  // this wave's own copies have landed (no other wave touches its slab)
    auto frag = [&](int t) { return *reinterpret_cast<const bf16x8*>(stage + (ln & 31) * D + ((2 * t + (ln >> 5)) ^ (ln % L::RC)) * 8); };
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      qf[t] = frag(t);
      for (int e = 0; e < 8; ++e) qf[t][e] = (__bf16)((float)qf[t][e] * c);
    }
#pragma unroll
    for (int n = 0; n < 32 / L::RPB; ++n) {
      const int r = n * L::RPB + g_row;
      *reinterpret_cast<bf16x8*>(stage + r * D + (g_chunk ^ (r % L::RC)) * 8) = gr[n];
    }
#pragma unroll
    for (int t = 0; t < KS; ++t) dof[t] = frag(t);
    const float delta = delta_s[wave][ln & 31];
    const float lse_i = q_ok ? __uint_as_float(lse_bits) : -INFINITY;
    const float nl = (lse_i == -INFINITY) ? -INFINITY : -lse_i * (kLog2e / rr);
    if (write_stats && (ln >> 5) == 0) {
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(nl), buffer_of(P->nl2 + row_at, rows * 4), (ln & 31) * 4, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(-delta), buffer_of(P->ndelta + row_at, rows * 4), (ln & 31) * 4, 0, 0);
    }
    nl_lane = nl;
    nd_lane = -delta;
    if constexpr (START_REGS)
      for (int e = 0; e < 16; ++e) dp_init[e] = -delta;
#pragma unroll
    for (int db = 0; db < DB; ++db)
      for (int e = 0; e < 16; ++e) dq[db][e] = 0.0f;
  };

  // The tiles list[0 .. n_list) (the first of which, `first`, is known already) for this work-group's queries.
  auto run_list = [&](const uint32_t* __restrict__ list, int n_list, uint32_t first, bool write_stats) {
    Kg = P->k + (int64_t)bh * N * D;
    Vg = P->v + (int64_t)bh * N * D;
    static_assert(NT >= kWin, "an entry of a window a thread");
    auto ask_list = [&](int w0) __attribute__((always_inline)) { return list[w0 + max(0, min(tid, n_list - w0 - 1))]; };
    auto put_list = [&](int w0, uint32_t entry) __attribute__((always_inline)) {
      const int count = min(kWin, n_list - w0);
      if (tid < count) tiles_s[tid] = entry;
      if (tid < 3) tiles_s[count + tid] = kNoTile;
    };
    auto start_tile = [&](uint32_t e) __attribute__((always_inline)) {
      e0 = e;
      copy_all(e0, k_s0, v_s0);
    };
    constexpr bool EARLY = NW <= 4;  // the waves' slabs of Q leave the buffers of parity 0 to the first tile
    auto run = [&](auto late) __attribute__((always_inline)) {
      // The list, the rows of Q, dO and O, their log-sum-exp and the first tile are asked for in one go, by buffer.  With the list's way to
      // LDS behind the tile, the rows behind that and the log-sum-exp behind those it was three round trips to memory in series.
      // Registers are not what it saves: in scratch memory lie none at D = 128, before or now, and at D = 64, four waves, 7 instead of
      // 5 (7 instead of 9 with the sharper scale), outside the tile loop.  The whole backward pass, us: D = 128, packed sequences of
      // 3001 68.1 -> 66.3, 4096 at 64 / 128 / 256 queries a block row 272.8 -> 267.4, 256.3 -> 250.2, 274.5 -> 269.3, a dilated window over 8
      // heads of 4096 51.9 -> 49.9 at 64; D = 64, where three work-groups a CU hide most of it, packed sequences of 4096 119.4 -> 118.1,
      // 116.9 -> 115.7, 131.8 -> 129.5, a window of 2 x 8 x 8192 96.7 -> 95.7, 95.7 -> 95.6, 102.1 -> 101.6, 1 x 2 x 256 16.6 -> 16.3.
      const uint32_t ahead = ask_list(0);
      begin_item(write_stats, [&]() __attribute__((always_inline)) {
        if (EARLY && n_list > 0) start_tile(first);
      });
      if (!EARLY || n_list == 0) __syncthreads();  // .. or to the epilogue, once every wave has read its slab
      if (!EARLY && n_list > 0) start_tile(first);
      for (int w0 = 0; w0 < n_list; w0 += kWin) {
        const int count = min(kWin, n_list - w0);
        if (w0 > 0) start_tile(scalar(list[w0]));
        put_list(w0, w0 > 0 ? ask_list(w0) : ahead);
        request_mask(e0);
        __syncthreads();
        if (decltype(late)::value != 0 && tid == 0) again_s = 0;  // (everyone has read it)
        e1_v = tiles_s[1];
        for (int it = 0; it < count; it += 2) {
          step(IntC<0>{}, late, it);
          if (it + 1 < count) step(IntC<1>{}, late, it + 1);
        }
        if (decltype(late)::value == 0 && __any(is_nan(dq[0][0]))) again_s = 1;
        __builtin_amdgcn_s_waitcnt(0);  // (the zero rows that the last step copied)
        __syncthreads();  // the next window rewrites the tile list and the buffers; the epilogue stages into them
      }
    };
    run(IntC<0>{});
    if (__builtin_expect(n_list > 0 && scalar(again_s) != 0, 0)) run(IntC<1>{});
  };

  auto write_dq = [&]() {
    __bf16* const stage = ((wave >> 1) == 0 ? k_s0 : (wave >> 1) == 1 ? k_s1 : (wave >> 1) == 2 ? v_s0 : v_s1) + (wave & 1) * 32 * D;
    store_slab<D>(dq, P->scale, stage, global(P->dq) + head_off, i * BR + wave * 32, N, lane);
  };

  // ---- which block row is this work-group's own: rank-major interleave of G (batch, head) planes, as in the forward
  int own_bh, own_m, rank;
  {
    const int logical = logical_wg((int)blockIdx.x, P->total_wgs);
    const int grp = logical / (P->G * P->nbr), within = logical - grp * (P->G * P->nbr);
    const int g_planes = min(P->G, P->total_wgs / P->nbr - grp * P->G);
    rank = within / g_planes;
    own_bh = grp * P->G + (within - rank * g_planes);
    own_m = (P->Mb == 1) ? 0 : own_bh / P->H;
  }
  int own_i, list_pos, n_list, nparts_all = 0, split_T = 0x7fffffff;
  uint32_t own_first = 0;
  if (global(P->sched)) {
    const int2 hdr = *reinterpret_cast<const int2*>(global(P->sched));
    const int4 rec = *reinterpret_cast<const int4*>(global(P->sched) + bbm::sched_order_base(P->Mb, P->nbr) +
                                                    bbm::kSchedRowInts * (int64_t)(own_m * P->nbr + rank));
    nparts_all = hdr.x;
    split_T = hdr.y;
    own_i = rec.x;
    list_pos = rec.y;
    n_list = rec.z;
    own_first = (uint32_t)rec.w;
  } else {
    own_i = P->nbr - 1 - rank;
    list_pos = global(P->row_ptr)[(int64_t)own_m * (P->nbr + 1) + own_i];
    n_list = global(P->row_ptr)[(int64_t)own_m * (P->nbr + 1) + own_i + 1] - list_pos;
    if (n_list > 0) own_first = global(P->col_idx)[(int64_t)own_m * P->nbr * P->nbc + list_pos];
  }

  if (tid == 0) again_s = 0;
  // The first n_extra work-groups serve the queue of cut-row parts before their own row (nothing to do when no row was cut):
  // one loop for parts and own row, so that the tile loop is in the program once.
  const bool leading = nparts_all > 0 && (int)blockIdx.x < P->n_extra;
  const int n_items = leading ? nparts_all * P->hbp : 0;
  int item = blockIdx.x;  // the first item is the work-group's own index; later ones come from the counter
  for (;;) {
    const bool is_part = item < n_items;
    int pos = list_pos, n_run = n_list <= split_T ? n_list : 0;  // (of a row that the schedule cut only the statistics are left)
    int next_item = 0, part = 0, nparts = 0, q_first = 0, rho = 0, hb = 0;
    uint32_t first = own_first;
    if (is_part) {
      if (tid == 0) next_item = P->n_extra + atomicAdd(global(P->row_queue), 1);
      hb = item / nparts_all;
      const int32_t* seg = global(P->sched) + bbm::kSchedPartBase + (int64_t)bbm::kSchedPartInts * (item - hb * nparts_all);
      const int row = seg[0];
      pos = seg[1], n_run = seg[2], part = seg[3], nparts = seg[4], q_first = seg[5], rho = seg[6], first = (uint32_t)seg[7];
      m = row / P->nbr;
      i = row - m * P->nbr;
      bh = (P->Mb == 1) ? hb : m * P->H + hb;
    } else {
      if (leading && tid == 0 && atomicAdd(global(P->row_queue) + 1, 1) == P->n_extra - 1) {  // the last leading work-group to leave the queue
        global(P->row_queue)[0] = 0;
        global(P->row_queue)[1] = 0;
      }
      m = own_m, i = own_i, bh = own_bh;
    }
    run_list(global(P->col_idx) + (int64_t)m * P->nbr * P->nbc + pos, n_run, scalar(first), !is_part);
    if (!is_part) {
      if (n_list <= split_T) write_dq();
      return;
    }
    // park the partial sums; the last part of the row to arrive adds them all up in part order, two records' loads in flight at
    // D = 64, one's at D = 128 (registers).  With a load at a time the backward pass took 161 instead of 147 us at 2 x 8 heads of
    // 8192 tokens, window, global tokens and random blocks, D = 64, and 319 instead of 268 at 8 heads of 16384, D = 128.
    float* const rec0 = global(P->row_partials) + ((int64_t)q_first * P->hbp + hb) * (REGS * NT);
    const int64_t pstride = (int64_t)P->hbp * (REGS * NT);
    int at = tid;
    asm volatile("" : "+v"(at));  // see store_slab
    bbm::store_record<DB, NT>(bbm::record_rsrc(rec0 + part * pstride, REGS * NT), at, dq);
    bbm::hand_over();
    if (tid == 0) {
      item_s[1] = atomicAdd(global(P->row_queue) + 8 + rho * P->hbp + hb, 1);
      item_s[0] = next_item;
    }
    __syncthreads();
    if (item_s[1] == nparts - 1) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
        for (int e = 0; e < 16; ++e) dq[db][e] = 0.0f;
      bbm::for_records<DB, NT, false, D == 64 ? 2 : 1>(rec0, pstride, nparts, at, [&](const f32x16 (&x)[DB], float2) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
          for (int e = 0; e < 16; ++e) dq[db][e] += x[db][e];
      });
      write_dq();
      if (tid == 0) global(P->row_queue)[8 + rho * P->hbp + hb] = 0;  // last user of this counter: zero for the next call
    }
    item = (int)scalar((uint32_t)item_s[0]);  // (a scalar: everything that addresses the item follows from it)
    __syncthreads();  // everyone has read the item, and the staged sums, before the next item's copies and list land
  }
}

// ------------------------------------------------------------------------------------------------------------------
// dK, dV
// ------------------------------------------------------------------------------------------------------------------
// One work-group per (block column, batch, head); the first P->n_extra work-groups first serve the queue of
// the parts of cut block columns, as the dQ kernel does for cut block rows.
// Four waves, (key half) x (query half of every 64-query sub-tile): each computes all four products of its 32 keys and its 32
// queries, so P and dS never leave its registers; the sums of the two query halves meet through LDS behind the last sub-tile.
// What bounds it is the way from one phase of a sub-tile to the next, so the phases are one chain of matrix instructions with
// everything else behind them (mfma_ring): in the loop the matrix pipe is 75 % busy.  It took the place, at D = 128, of a split
// of the waves by product, P crossing through LDS behind a second barrier, where either role waited for the other (a step of
// 3620 cycles, now 2740), and at D = 64 of two waves that took one key half each.  Kernel time: 2 x 32 heads of 8192 causal
// tokens, D = 128, 2370 -> 1900-1960 us; 4 x 16 heads of 4096, D = 64, 350 -> 303 us; a 16384-token window with global tokens
// 195 -> 188; packed sequences of 4096, D = 64, 73.7 -> 72.4, of 3001, D = 128, 45.2 -> 41.9.
// Registers are what the form lives by.  D = 128: 256, two operand pieces in LDS, two waves a SIMD; one register more in scratch
// memory inside the loop costs a wait for the tile copies in flight (a form with 16 of them took 3240 us).  D = 64: 168, three.
template <int D, bool EXACT>
__global__ __launch_bounds__(256, D == 128 ? 2 : 3) void attn_bwd_dkv_kernel(const BwdParams) {
  Args P = bbm::kernel_args<BwdParams>();
  using L = TL<D>;
  constexpr int NW = 4, NT = 64 * NW;
  constexpr int NTP = 128;  // lanes that hold one of the two sums: stride of the parked records
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int REGS = DB * 16;
  constexpr int kRing = 3;
  static_assert(2 * 32 * D <= L::ELEMS, "two 32 x D output slabs must fit in a tile buffer");

  __shared__ __attribute__((aligned(16))) __bf16 t_s0[2 * L::ELEMS];  // [Q, dO] tiles, one variable per parity
  __shared__ __attribute__((aligned(16))) __bf16 t_s1[2 * L::ELEMS];
  __shared__ __attribute__((aligned(16))) float st_s0[2 * 64];  // [-lse*log2 e, -D] of the sub-tile's queries
  __shared__ __attribute__((aligned(16))) float st_s1[2 * 64];
  __shared__ __attribute__((aligned(16))) uint32_t mk_s0[2][64];  // [key half][query row of the sub-tile]
  __shared__ __attribute__((aligned(16))) uint32_t mk_s1[2][64];
  __shared__ uint32_t tiles_s[kWin + 2];  // entries past the last one are read but not used
  __shared__ int item_s[2];
  __shared__ int again_s;  // a wave's sums are not numbers
  // D = 128: the last pieces of the K operand, which find no room in the registers
  constexpr int KL = D == 128 ? 2 : 0;
  __shared__ __attribute__((aligned(16))) bf16x8 kl_s[KL ? KL : 1][NW][64];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kh = wave & 1;   // key half of the column block
  const int qh = wave >> 1;  // query half of the sub-tile; behind the last one, 0: this wave writes dV, 1: dK
  const int N = (int)P->N;
  const float c = P->qscale;
  const float rr = EXACT ? P->rmul : 1.0f;
  auto ex2 = [&](float x) { return __builtin_amdgcn_exp2f(EXACT ? rr * x : x); };

  // ---- per-item state
  int bh, m, j;
  int64_t head_off;
  const __bf16* __restrict__ Qg;
  const __bf16* __restrict__ Gg;
  const float* __restrict__ nlg;
  const float* __restrict__ ndg;
  const uint32_t* __restrict__ mcol;
  bf16x8 kf[KS - KL], vf[KS];
  f32x16 dk[DB], dv[DB];  // behind the last sub-tile dk holds this wave's output, dV or dK

  TileAddr<D> A;
  A.init(lane);
  for (int i = 0; i < 2; ++i) {  // this wave's half of the tile's rows
    A.ra[i] += qh * (32 / L::NBLK) * D;
    A.ta[i] += 2 * qh * (D == 64 ? 2 * D : D);
  }

  const int qs_shift = P->br == 64 ? 0 : P->br == 128 ? 1 : 2;  // 64-query sub-tiles per block row: 1, 2, 4
  // Copies of the 64-query sub-tile from row0 on into the buffers of one parity: Q and dO tiles, the negated statistics of its
  // queries (-lse*log2 e and -D) and, if the block is partial, the two 32-bit halves of its mask words, a wave for each of the
  // four.  Queries past N come as zeros everywhere: with Q = dO = D = 0 they add exact zeros.
  const uint32_t copy_base = tile_copy_base<D, NW>(wave, lane);
  constexpr int LPW = L::NBLK / NW;  // copy instructions of a wave per tile
  auto copy_piece = [&](int row0, int rows, __bf16* td, int n) {  // n = 0 .. 2*LPW-1
    const int64_t at = (int64_t)row0 * D;
    if (n < LPW)
      tile_copy_piece<D, NW>(Qg + at, rows, copy_base, td, n, wave);
    else
      tile_copy_piece<D, NW>(Gg + at, rows, copy_base, td + L::ELEMS, n - LPW, wave);
  };
  auto copy_stats = [&](int row0, int rows, bool partial, float* sts, uint32_t (*mkd)[64]) __attribute__((always_inline)) {
    if (qh == 0)
      copy_async<4>((kh == 0 ? nlg : ndg) + row0, rows * 4, lane_now() * 4, sts + kh * 64);
    else if (partial)  // (the words lie 8 bytes apart; this wave's half is the first or the second 4 bytes of each)
      copy_async<4>(mcol + 2 * (int64_t)row0, max(0, rows * 8 - 4), lane_now() * 8, mkd[kh]);
  };
  auto copy_all = [&](int row0, int rows, __bf16* td) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < 2 * LPW; ++n) copy_piece(row0, rows, td, n);
  };

  // Step s: list entry e0 = tiles_s[s >> qs_shift], the entry of step s + 1 is e1 (both read a step ahead).
  int n_steps = 0;
  uint32_t e0 = 0, e1 = 0;
  auto entry_of = [&](int s) { return scalar(tiles_s[s >> qs_shift]); };
  auto row_of = [&](uint32_t e, int s) { return (int)(((e & 0x7fffffffu) << qs_shift) + (s & ((1 << qs_shift) - 1))) * 64; };
  // `late`: the mask behind the product, see the dQ kernel (a sum here that is no number takes all of the key's dV with it).
  auto step = [&](auto pb, auto late, int s) __attribute__((always_inline)) {
    constexpr int PB = decltype(pb)::value;
    constexpr bool LATE = decltype(late)::value != 0;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    __bf16* const q_cur = PB ? t_s1 : t_s0;
    __bf16* const g_cur = q_cur + L::ELEMS;
    __bf16* const t_oth = PB ? t_s0 : t_s1;
    const float* const nl_cur = (PB ? st_s1 : st_s0) + 32 * qh;
    const float* const nd_cur = nl_cur + 64;
    const uint32_t* const mk_cur = &(PB ? mk_s1 : mk_s0)[kh][32 * qh];
    const bool partial = (e0 >> 31) == 0;
    // The next sub-tile's copies go out one by one between the matrix instructions of this one: requested in one go they
    // fill the memory pipe's queue, and every wave of the work-group stands there for 700-850 cycles of a step (D = 128).
    // Behind the last sub-tile they copy zero rows into buffers that nobody reads any more, cheaper than a branch around each.
    const bool more = s + 1 < n_steps;
    const int row1 = row_of(e1, s + 1), rows1 = more ? rows_of_tile(row1, N) : 0;
    if (more) copy_stats(row1, rows1, (e1 >> 31) == 0, PB ? st_s0 : st_s1, PB ? mk_s0 : mk_s1);
    e0 = e1;
    const uint32_t e2 = tiles_s[(s + 2) >> qs_shift];
    // a partial sub-tile in which none of this wave's 32 queries sees one of its 32 keys contributes exact zeros
    const bool live = !partial || __ballot(mk_cur[lane_now() & 31] != 0u) != 0ull;
    if (!live && more) copy_all(row1, rows1, t_oth);
    if (live) {
      f32x16 sc, dp;
      const int ln = lane_now(), hh4 = ln >> 5 << 2;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 x = *reinterpret_cast<const float4*>(nl_cur + 8 * g + hh4);
        sc[4 * g + 0] = x.x, sc[4 * g + 1] = x.y, sc[4 * g + 2] = x.z, sc[4 * g + 3] = x.w;
      }
      auto mask_scores = [&]() {  // -inf, i.e. P = 0, where the mask word (32 keys of a query row) has no bit
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const uint4 w = *reinterpret_cast<const uint4*>(mk_cur + 8 * g + hh4);
          const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)ww[e], ln & 31, 1);  // all ones iff bit lq is set
            sc[4 * g + e] = __uint_as_float((__float_as_uint(sc[4 * g + e]) & keep) | (0xff800000u & ~keep));
          }
        }
      };
      if (!LATE && partial) mask_scores();
      // One chain of matrix instructions, S, dP, dV, dK, with everything else behind them: the next sub-tile's copies behind
      // S, the exponentials behind dP, dS behind dV.  At D = 128 the fp32 probabilities do not outlive dP (registers): dS is
      // formed from P as the dV product consumes it, rounded to bf16.
      constexpr bool P32 = D == 64;
      constexpr int N1 = KS, N2 = 2 * KS, N3 = N2 + 2 * DB, N4 = N3 + 2 * DB;
      constexpr int PER = D == 128 ? 4 : 8;  // elements behind a matrix instruction
      static_assert(PER * (KS - 2) >= 16 && PER * (2 * DB - 2) >= 16, "all 16 must find room");
      uint32_t pf[2][4], dsf[2][4];  // pairs of bf16
      bf16x8 kl[2];
      mfma_ring<N4, LATE ? 1 : kRing>(
          [&](auto i) {
            constexpr int n = decltype(i)::value;
            if constexpr (n < N2)
              return A.row_frag(n < N1 ? q_cur : g_cur, 0, n % KS);
            else
              return A.tr_frag(n < N3 ? g_cur : q_cur, (n - N2) % (2 * DB) / DB, n % DB);
          },
          [&](auto i, bf16x8 f) {
            constexpr int n = decltype(i)::value, db = n % DB, u = (n - N2) % (2 * DB) / DB;
            static_assert(KS % DB == 0, "the two counts of column blocks start at multiples of DB");
            if constexpr (n < N1 - KL)
              sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, kf[n], sc, 0, 0, 0);
            else if constexpr (n < N1)
              sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, kl[n & 1], sc, 0, 0, 0);
            else if constexpr (n < N2)
              dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, vf[n - N1], dp, 0, 0, 0);
            else if constexpr (n < N3)
              dv[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, operand(pf[u]), dv[db], 0, 0, 0);
            else
              dk[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, operand(dsf[u]), dk[db], 0, 0, 0);
          },
          [&](auto i) {
            constexpr int n = decltype(i)::value;
            static_assert(2 * LPW == KS, "one copy behind every matrix instruction of S");
            if constexpr (n < N1) copy_piece(row1, rows1, t_oth, n);
            if constexpr (n >= N1 - KL - 2 && n < N1 - 2) kl[n & 1] = kl_s[n - (N1 - KL - 2)][wave][lane_now()];
            if constexpr (n == N1 - 2) {
              const float* const nd = nd_cur + (lane_now() >> 5 << 2);
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                const float4 x = *reinterpret_cast<const float4*>(nd + 8 * g);
                dp[4 * g + 0] = x.x, dp[4 * g + 1] = x.y, dp[4 * g + 2] = x.z, dp[4 * g + 3] = x.w;
              }
            }
            if constexpr (LATE && n == N1 + 2)
              if (partial) mask_scores();
            if constexpr (n >= N1 + 2 && n < N2) {  // S is complete two matrix instructions after its last one was issued
#pragma unroll
              for (int e = (n - N1 - 2) * PER; e < min(16, (n - N1 - 1) * PER); e += 2) {
                sc[e] = ex2(sc[e]);
                sc[e + 1] = ex2(sc[e + 1]);
                pf[e / 8][e % 8 / 2] = pack(sc[e], sc[e + 1]);
                // (hides the pair's origin: the compiler otherwise rounds each of the two once more where dS takes it apart)
                if constexpr (!P32) asm("" : "+v"(pf[e / 8][e % 8 / 2]));
              }
            }
            if constexpr (n >= N2 + 2 && n < N3) {
#pragma unroll
              for (int e = (n - N2 - 2) * PER; e < min(16, (n - N2 - 1) * PER); e += 2) {
                const uint32_t w = pf[e / 8][e % 8 / 2];
                const float p0 = P32 ? sc[e] : __uint_as_float(w << 16), p1 = P32 ? sc[e + 1] : __uint_as_float(w & 0xffff0000u);
                dsf[e / 8][e % 8 / 2] = pack(p0 * dp[e], p1 * dp[e + 1]);
              }
            }
          });
    }
    e1 = scalar(e2);
  };

  // The query blocks list[0 .. n_list) (the first of which, `first`, is known already) of this work-group's 64 keys.
  auto run_list = [&](const uint32_t* __restrict__ list, int n_list, uint32_t first) {
    head_off = (int64_t)bh * N * D;
    Qg = P->q + head_off;
    Gg = global(P->d_o) + head_off;
    nlg = global(global(P->nl2)) + (int64_t)bh * N;
    ndg = global(P->ndelta) + (int64_t)bh * N;
    // this wave's 32-bit half of the packed mask words of block column j (one word per query row)
    mcol = reinterpret_cast<const uint32_t*>(global(P->packed) + ((int64_t)m * P->W + j) * (int64_t)N) + kh;
    auto run = [&](auto late) __attribute__((always_inline)) {
      // The last column's operands end here: set in the first window only, they would be kept from item to item (56 registers at
      // D = 128, and as many of the merge's in scratch memory).
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        asm("" : "=v"(vf[t]));
        if (t < KS - KL) asm("" : "=v"(kf[t < KS - KL ? t : 0]));
      }
#pragma unroll
      for (int db = 0; db < DB; ++db)
        for (int e = 0; e < 16; ++e) dk[db][e] = dv[db][e] = 0.0f;
      for (int w0 = 0; w0 < n_list; w0 += kWin) {
        const int count = min(kWin, n_list - w0);
        e0 = w0 > 0 ? scalar(list[w0]) : first;
        const int row0 = row_of(e0, 0), rows0 = rows_of_tile(row0, N);
        copy_stats(row0, rows0, (e0 >> 31) == 0, st_s0, mk_s0);
        copy_all(row0, rows0, t_s0);
        if (w0 == 0) {
          // K and V come through the tile buffers of parity 1 as well (keys past N as zeros): straight from memory a lane would
          // pick its row up in 16-byte pieces, 64 cache lines an instruction, and stand there for 7000 cycles of a column at
          // D = 64, 12000 at D = 128.
          const int64_t at = head_off + (int64_t)j * 64 * D;
          const int keys = rows_of_tile(j * 64, N);
#pragma unroll
          for (int n = 0; n < LPW; ++n) {
            tile_copy_piece<D, NW>(P->k + at, keys, copy_base, t_s1, n, wave);
            tile_copy_piece<D, NW>(P->v + at, keys, copy_base, t_s1 + L::ELEMS, n, wave);
          }
        }
        for (int t = tid; t < count; t += NT) tiles_s[t] = list[w0 + t];
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        n_steps = count << qs_shift;
        e1 = entry_of(1);
        if (w0 == 0) {  // this lane's key: K * scale * log2(e) and V as B operands
          const int half = (kh - qh) * (32 / L::NBLK) * D;  // (A addresses this wave's query half of a tile)
#pragma unroll
          for (int t = 0; t < KS; ++t) {
            bf16x8 kt = A.row_frag(t_s1 + half, 0, t);
            vf[t] = A.row_frag(t_s1 + L::ELEMS + half, 0, t);
            for (int e = 0; e < 8; ++e) kt[e] = (__bf16)((float)kt[e] * c);
            if (t >= KS - KL)
              kl_s[t - (KS - KL)][wave][lane] = kt;  // (read back by this wave alone)
            else
              kf[t] = kt;
          }
        }
        if (decltype(late)::value != 0 && tid == 0) again_s = 0;  // (everyone has read it)
        for (int s = 0; s < n_steps; s += 2) {
          step(IntC<0>{}, late, s);
          if (s + 1 < n_steps) step(IntC<1>{}, late, s + 1);
        }
        if (decltype(late)::value == 0 && __any(is_nan(dv[0][0]))) again_s = 1;
        __builtin_amdgcn_s_waitcnt(0);  // (the zero rows that the last step copied)
        __syncthreads();  // the next window rewrites the list and the buffers; the epilogue stages into them
      }
    };
    run(IntC<0>{});
    if (__builtin_expect(n_list > 0 && scalar(again_s) != 0, 0)) run(IntC<1>{});
    // The two waves of a key half exchange: query half 0 hands over its dK and receives dV, query half 1 the other way round.
    float4* const mine = reinterpret_cast<float4*>(qh == 0 ? t_s0 : t_s1) + kh * (REGS / 4) * 64;
    const float4* const theirs = reinterpret_cast<const float4*>(qh == 0 ? t_s1 : t_s0) + kh * (REGS / 4) * 64;
    static_assert(2 * REGS * 64 * sizeof(float) <= 2 * L::ELEMS * sizeof(__bf16), "two waves' sums must fit in the tile buffers of a parity");
    int ln = lane;
    asm volatile("" : "+v"(ln));  // see store_slab
#pragma unroll
    for (int db = 0; db < DB; ++db)
      for (int g = 0; g < 4; ++g) {
        float4 x;
        x.x = qh ? dv[db][4 * g + 0] : dk[db][4 * g + 0];
        x.y = qh ? dv[db][4 * g + 1] : dk[db][4 * g + 1];
        x.z = qh ? dv[db][4 * g + 2] : dk[db][4 * g + 2];
        x.w = qh ? dv[db][4 * g + 3] : dk[db][4 * g + 3];
        mine[(db * 4 + g) * 64 + ln] = x;
      }
    __syncthreads();
#pragma unroll
    for (int db = 0; db < DB; ++db)
      for (int g = 0; g < 4; ++g) {
        const float4 x = theirs[(db * 4 + g) * 64 + ln];
        dk[db][4 * g + 0] = x.x + (qh ? dk[db][4 * g + 0] : dv[db][4 * g + 0]);
        dk[db][4 * g + 1] = x.y + (qh ? dk[db][4 * g + 1] : dv[db][4 * g + 1]);
        dk[db][4 * g + 2] = x.z + (qh ? dk[db][4 * g + 2] : dv[db][4 * g + 2]);
        dk[db][4 * g + 3] = x.w + (qh ? dk[db][4 * g + 3] : dv[db][4 * g + 3]);
      }
    __syncthreads();  // the epilogue stages into the same buffers
  };

  auto write_dkv = [&]() {
    const int row0 = j * 64 + kh * 32;
    if (qh == 0)
      store_slab<D>(dk, 1.0f, t_s0 + L::ELEMS + kh * 32 * D, global(P->dv) + head_off, row0, N, lane);
    else
      store_slab<D>(dk, P->scale, t_s0 + kh * 32 * D, global(P->dk) + head_off, row0, N, lane);
  };

  // This work-group's own block column: rank-major interleave of G (batch, head) planes as in the dQ kernel, ranks by list
  // length (longest first) from the schedule's records
  int nparts_all = 0, split_T = 0x7fffffff;
  int own_bh, own_m, own_j, own_pos, own_n;
  uint32_t own_first = 0;
  {
    const int logical = logical_wg((int)blockIdx.x, P->total_wgs);
    if (global(P->csched)) {
      const int2 hdr = *reinterpret_cast<const int2*>(global(P->csched));
      nparts_all = hdr.x;
      split_T = hdr.y;
      const int grp = logical / (P->Gc * P->nbc), within = logical - grp * (P->Gc * P->nbc);
      const int g_planes = min(P->Gc, P->total_wgs / P->nbc - grp * P->Gc);
      const int rank = within / g_planes;
      own_bh = grp * P->Gc + (within - rank * g_planes);
      own_m = (P->Mb == 1) ? 0 : own_bh / P->H;
      const int4 rec = *reinterpret_cast<const int4*>(global(P->csched) + bbm::kSchedPartBase + (int64_t)bbm::kSchedPartInts * P->Mb * P->nbc +
                                                      bbm::kSchedRowInts * (int64_t)(own_m * P->nbc + rank));
      own_j = rec.x;
      own_pos = rec.y;
      own_n = rec.z;
      own_first = (uint32_t)rec.w;
    } else {
      own_bh = logical / P->nbc;
      own_j = logical - own_bh * P->nbc;
      own_m = (P->Mb == 1) ? 0 : own_bh / P->H;
      own_pos = global(P->col_ptr)[(int64_t)own_m * (P->nbc + 1) + own_j];
      own_n = global(P->col_ptr)[(int64_t)own_m * (P->nbc + 1) + own_j + 1] - own_pos;
      if (own_n > 0) own_first = global(P->row_idx)[(int64_t)own_m * P->nbr * P->nbc + own_pos];
    }
  }

  if (tid == 0) again_s = 0;
  // The first n_extra work-groups serve the queue of cut-column parts before their own column (nothing to do when no column
  // was cut): one loop for parts and own column, so that the tile loop is in the program once.
  const bool leading = nparts_all > 0 && (int)blockIdx.x < P->n_extra;
  const int n_items = leading ? nparts_all * P->hbp : 0;
  int item = blockIdx.x;  // the first item is the work-group's own index; later ones come from the counter
  for (;;) {
    const bool is_part = item < n_items;
    int pos, n_list, next_item = 0, part = 0, nparts = 0, q_first = 0, rho = 0, hb = 0;
    uint32_t first = own_first;
    if (is_part) {
      if (tid == 0) next_item = P->n_extra + atomicAdd(global(P->col_queue), 1);
      hb = item / nparts_all;
      const int32_t* seg = global(P->csched) + bbm::kSchedPartBase + (int64_t)bbm::kSchedPartInts * (item - hb * nparts_all);
      const int col = seg[0];
      pos = seg[1], n_list = seg[2], part = seg[3], nparts = seg[4], q_first = seg[5], rho = seg[6], first = (uint32_t)seg[7];
      m = col / P->nbc;
      j = col - m * P->nbc;
      bh = (P->Mb == 1) ? hb : m * P->H + hb;
    } else {
      if (leading && tid == 0 && atomicAdd(global(P->col_queue) + 1, 1) == P->n_extra - 1) {  // the last leading work-group to leave the queue
        global(P->col_queue)[0] = 0;
        global(P->col_queue)[1] = 0;
      }
      if (own_n > split_T) return;  // a column the schedule cut belongs to the queue
      m = own_m, j = own_j, bh = own_bh, pos = own_pos, n_list = own_n;
    }
    run_list(global(P->row_idx) + (int64_t)m * P->nbr * P->nbc + pos, n_list, scalar(first));
    if (!is_part) {
      write_dkv();
      return;
    }
    float* const rec0 = global(P->col_partials) + ((int64_t)q_first * P->hbp + hb) * (2 * REGS * NTP);
    const int64_t pstride = (int64_t)P->hbp * (2 * REGS * NTP);
    int at = kh * 64 + lane;
    asm volatile("" : "+v"(at));  // see store_slab
    float* const rec = rec0 + (qh == 0 ? REGS * NTP : 0);  // a record: [dK | dV]
    bbm::store_record<DB, NTP>(bbm::record_rsrc(rec + part * pstride, REGS * NTP), at, dk);
    bbm::hand_over();
    if (tid == 0) {
      item_s[1] = atomicAdd(global(P->col_queue) + 8 + rho * P->hbp + hb, 1);
      item_s[0] = next_item;
    }
    __syncthreads();
    if (item_s[1] == nparts - 1) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
        for (int e = 0; e < 16; ++e) dk[db][e] = 0.0f;
      bbm::for_records<DB, NTP, false, D == 64 ? 2 : 1>(rec, pstride, nparts, at, [&](const f32x16 (&x)[DB], float2) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
          for (int e = 0; e < 16; ++e) dk[db][e] += x[db][e];
      });
      write_dkv();
      if (tid == 0) global(P->col_queue)[8 + rho * P->hbp + hb] = 0;
    }
    item = (int)scalar((uint32_t)item_s[0]);  // (a scalar: everything that addresses the item follows from it)
    __syncthreads();  // everyone has read the item, and the staged sums, before the next item's copies and list land
  }
}

// Leading work-groups that serve a queue of parts before their own block row / column.
constexpr int kExtraWGs = 256;

inline size_t round256(size_t n) { return (n + 255) / 256 * 256; }
inline size_t stats_bytes(int64_t B, int64_t H, int64_t N) { return round256((size_t)(B * H * N) * sizeof(float)); }
// counters of one queue: 8 + one per (cut row or column, (batch, head) of its plane); at most nb * B*H of those
inline size_t queue_bytes(int64_t B, int64_t H, int64_t nb) { return round256((size_t)(8 + B * H * nb) * sizeof(int32_t)); }
// at most Mb*nbr row parts and Mb*nbc column parts exist (the split thresholds are at least twice the mean length):
// the partial results of all parts together are one fp32 copy of dQ, and of dK plus dV, each padded to whole blocks
inline size_t row_partial_bytes(int64_t B, int64_t H, int64_t nbr, int Br, int d) { return (size_t)(B * H * nbr) * Br * d * sizeof(float); }
inline size_t col_partial_bytes(int64_t B, int64_t H, int64_t nbc, int d) { return (size_t)(B * H * nbc) * 2 * 64 * d * sizeof(float); }

template <int D, bool EXACT>
int launch_bwd(BwdParams& P, int64_t B, int64_t H, hipStream_t s) {
  P.total_wgs = (int32_t)(B * H * P.nbr);
  P.n_extra = std::min<int32_t>(P.total_wgs, kExtraWGs);
  P.G = bbm::interleaved_planes(B * H, 2 * P.N * D * (int64_t)sizeof(__bf16));
  if (P.br == 64)
    attn_bwd_dq_kernel<D, 2, EXACT><<<(unsigned)P.total_wgs, 128, 0, s>>>(P);
  else if (P.br == 128)
    attn_bwd_dq_kernel<D, 4, EXACT><<<(unsigned)P.total_wgs, 256, 0, s>>>(P);
  else
    attn_bwd_dq_kernel<D, 8, EXACT><<<(unsigned)P.total_wgs, 512, 0, s>>>(P);
  int rc = bbm::launch_status("bbm_attn_bwd (dq)");
  if (rc != BBM_OK) return rc;
  P.total_wgs = (int32_t)(B * H * P.nbc);
  P.n_extra = std::min<int32_t>(P.total_wgs, kExtraWGs);
  P.Gc = P.G;
  attn_bwd_dkv_kernel<D, EXACT><<<(unsigned)P.total_wgs, 256, 0, s>>>(P);
  return bbm::launch_status("bbm_attn_bwd (dk, dv)");
}

}  // namespace

extern "C" __attribute__((visibility("default"))) size_t bbm_attn_bwd_workspace_bytes(int64_t B, int64_t H, int64_t N, int d, int Br) {
  if (B < 1 || H < 1 || N < 1 || (d != 64 && d != 128) || (Br != 64 && Br != 128 && Br != 256)) return 0;
  const int64_t nbr = (N + Br - 1) / Br, nbc = (N + 63) / 64;
  return queue_bytes(B, H, nbr) + queue_bytes(B, H, nbc) + 2 * stats_bytes(B, H, N) + round256(row_partial_bytes(B, H, nbr, Br, d)) +
         col_partial_bytes(B, H, nbc, d);
}
extern "C" __attribute__((visibility("default"))) int bbm_attn_bwd(const void* q, const void* k, const void* v, const void* o, const void* d_o,
                                                                   const float* lse, void* dq, void* dk, void* dv, int64_t B, int64_t H,
                                                                   int64_t N, int d, float softmax_scale, int64_t Mb,
                                                                   const uint64_t* packed_mask, const bbm_index* idx, void* workspace,
                                                                   size_t workspace_bytes, void* stream) {
  using namespace bbm;
  clear_error();
  if (!q || !k || !v || !o || !d_o || !lse || !dq || !dk || !dv)
    return fail(BBM_EINVAL, "bbm_attn_bwd: q, k, v, o, d_o, lse, dq, dk, dv must not be NULL");
  if (!aligned(q, 16) || !aligned(k, 16) || !aligned(v, 16) || !aligned(o, 16) || !aligned(d_o, 16) || !aligned(dq, 16) ||
      !aligned(dk, 16) || !aligned(dv, 16))
    return fail(BBM_EINVAL, "bbm_attn_bwd: q, k, v, o, d_o, dq, dk, dv must be 16-byte aligned");
  if (!aligned(lse, 4)) return fail(BBM_EINVAL, "bbm_attn_bwd: lse must be 4-byte aligned");
  if (B < 1 || H < 1 || N < 1) return fail(BBM_EINVAL, "bbm_attn_bwd: B=%lld, H=%lld, N=%lld must be >= 1", (long long)B, (long long)H, (long long)N);
  if (!(softmax_scale > 0.0f) || !(softmax_scale < INFINITY)) return fail(BBM_EINVAL, "bbm_attn_bwd: softmax_scale must be finite and > 0");
  if (Mb != 1 && Mb != B) return fail(BBM_EINVAL, "bbm_attn_bwd: Mb=%lld must be 1 or B=%lld", (long long)Mb, (long long)B);
  if (!idx) return fail(BBM_EINVAL, "bbm_attn_bwd: idx must not be NULL");
  if (!packed_mask || !aligned(packed_mask, 8)) return fail(BBM_EINVAL, "bbm_attn_bwd: packed_mask must be a non-NULL 8-byte aligned pointer");
  if (d != 64 && d != 128) return fail(BBM_EUNSUPPORTED, "bbm_attn_bwd: d=%d has no kernel instance (64, 128)", d);
  if (idx->Bc != 64 || (idx->Br != 64 && idx->Br != 128 && idx->Br != 256))
    return fail(BBM_EUNSUPPORTED, "bbm_attn_bwd: tile (Br=%d, Bc=%d) has no kernel instance (Br in {64,128,256}, Bc = 64)", idx->Br, idx->Bc);
  const int64_t nbr = ceil_div(N, idx->Br), nbc = ceil_div(N, idx->Bc);
  if (idx->Nq != N || idx->Nk != N)
    return fail(BBM_EINVAL, "bbm_attn_bwd: index built for a mask of %lld x %lld does not match N=%lld", (long long)idx->Nq, (long long)idx->Nk,
                (long long)N);
  if (idx->Mb != Mb || idx->nbr != nbr || idx->nbc != nbc)
    return fail(BBM_EINVAL, "bbm_attn_bwd: index (Mb=%lld, nbr=%lld, nbc=%lld) does not match the problem (Mb=%lld, nbr=%lld, nbc=%lld)",
                (long long)idx->Mb, (long long)idx->nbr, (long long)idx->nbc, (long long)Mb, (long long)nbr, (long long)nbc);
  if (!idx->row_ptr || !idx->col_idx || !idx->col_ptr || !idx->row_idx)
    return fail(BBM_EINVAL, "bbm_attn_bwd: the index needs row_ptr, col_idx (block list) and col_ptr, row_idx (column list)");
  if (nbr * nbc >= (1ll << 31) || B * H * nbr >= (1ll << 31) || B * H * nbc >= (1ll << 31) || N >= (1ll << 31))
    return fail(BBM_EUNSUPPORTED, "bbm_attn_bwd: problem too large for 32-bit tile counters");
  const size_t need = bbm_attn_bwd_workspace_bytes(B, H, N, d, idx->Br);
  if (!workspace || workspace_bytes < need)
    return fail(BBM_EWORKSPACE, "bbm_attn_bwd: workspace of %zu bytes needed, %zu given", need, workspace ? workspace_bytes : (size_t)0);
  if (!aligned(workspace, 16)) return fail(BBM_EINVAL, "bbm_attn_bwd: workspace must be 16-byte aligned");

  BwdParams P;
  P.q = static_cast<const __bf16*>(q);
  P.k = static_cast<const __bf16*>(k);
  P.v = static_cast<const __bf16*>(v);
  P.o = static_cast<const __bf16*>(o);
  P.d_o = static_cast<const __bf16*>(d_o);
  P.lse = lse;
  P.dq = static_cast<__bf16*>(dq);
  P.dk = static_cast<__bf16*>(dk);
  P.dv = static_cast<__bf16*>(dv);
  // workspace: the two counter arrays first (they are what must be zero between calls), then statistics and partials
  char* ws = static_cast<char*>(workspace);
  P.row_queue = reinterpret_cast<int32_t*>(ws);
  ws += queue_bytes(B, H, nbr);
  P.col_queue = reinterpret_cast<int32_t*>(ws);
  ws += queue_bytes(B, H, nbc);
  P.nl2 = reinterpret_cast<float*>(ws);
  ws += stats_bytes(B, H, N);
  P.ndelta = reinterpret_cast<float*>(ws);
  ws += stats_bytes(B, H, N);
  P.row_partials = reinterpret_cast<float*>(ws);
  ws += round256(row_partial_bytes(B, H, nbr, idx->Br, d));
  P.col_partials = reinterpret_cast<float*>(ws);
  P.csched = idx->col_sched;
  P.hbp = (int32_t)(Mb == 1 ? B * H : H);
  P.n_extra = 0;
  P.packed = packed_mask;
  P.row_ptr = idx->row_ptr;
  P.col_idx = idx->col_idx;
  P.sched = idx->sched;
  P.col_ptr = idx->col_ptr;
  P.row_idx = idx->row_idx;
  P.N = N;
  P.H = (int32_t)H;
  P.Mb = (int32_t)Mb;
  P.nbr = (int32_t)nbr;
  P.nbc = (int32_t)nbc;
  P.W = (int32_t)ceil_div(N, 64);
  P.br = idx->Br;
  P.scale = softmax_scale;
  // the same rule as the forward (whose lse this call consumes): scales up to 1/sqrt(d) fold into the bf16 operand
  const float c = softmax_scale * kLog2e;
  const bool exact = softmax_scale * sqrtf((float)d) > 1.0f + 1.0f / 1024.0f;
  int c_exp = 0;
  (void)frexpf(c, &c_exp);
  P.qscale = exact ? ldexpf(1.0f, c_exp - 1) : c;
  P.rmul = exact ? c / P.qscale : 1.0f;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (exact) return d == 64 ? launch_bwd<64, true>(P, B, H, s) : launch_bwd<128, true>(P, B, H, s);
  return d == 64 ? launch_bwd<64, false>(P, B, H, s) : launch_bwd<128, false>(P, B, H, s);
}
