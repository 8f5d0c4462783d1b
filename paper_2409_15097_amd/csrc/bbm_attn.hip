// Stage 2: fused masked attention forward that visits only non-zero key/value tiles (paper Sec. 3 "Flash
// Attention", Sec. 4 "Binary Block Masking" / "Dense Binary Block Masking").
//
// Work decomposition.  One work-group owns one block row (Br = 32*NW query rows) of one (batch, head); each
// of its NW wavefronts owns 32 query rows.  Key/value tiles are Bc = 64 keys wide.  The kernel computes the
// TRANSPOSED products so that one lane owns one query row:
//     S^T[key][q]  = K_tile[key][:] . Q[q][:]        (A operand = K from LDS, B operand = Q in registers)
//     O^T[dcol][q] += V_tile^T[dcol][key] . P^T[key][q]  (A operand = V via transposing LDS reads, B = P)
// With the 32x32x16 bf16 MFMA the accumulator of lane l holds column q = l%32 and rows
// 8*(v/4) + 4*(l/32) + v%4, v = 0..15.  So a lane and its partner l^32 together hold all scores of one query
// row: the row maximum needs one cross-lane exchange, the rescale factor and the row sum stay in-lane, and
// the S^T accumulators are -- after rounding to bf16 -- directly the B operand of the second product (the key
// order inside a 16-key MFMA step is a fixed permutation, matched by the addresses of the V reads).
// The element mask of a 32x64 score slab is one 64-bit word per query row (word-column-major packed mask),
// tested with compile-time bit positions.
#include "bbm_internal.h"
#include "bbm_mfma.h"

#include <algorithm>
#include <cstddef>
#include <mutex>

namespace {

using bbm::bf16x2, bbm::bf16x4, bbm::bf16x8, bbm::f32x16, bbm::global, bbm::IntC, bbm::mfma_ring, bbm::partner_sum, bbm::s16x4, bbm::scalar;

constexpr int kBc = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLazy = 8.0f;  // log2 headroom before the running maximum is moved

struct AttnParams {
  const __bf16* q;
  const __bf16* k;
  const __bf16* v;
  __bf16* o;
  float* lse;
  const uint64_t* packed;  // [Mb][W][N]
  const uint8_t* bin_blk_mat;
  const int32_t* offset;
  const int32_t* total_ones;
  const int32_t* nz_lo;
  const int32_t* nz_hi;
  const int32_t* row_ptr;
  const uint32_t* col_idx;
  int64_t N;   // queries per head
  int64_t Nk;  // keys per head (= N for self-attention over one sequence)
  int32_t H, Mb, nbr, nbc, W;
  int32_t total_wgs;
  int32_t mode;
  float qscale;       // factor applied to Q before it is rounded to bf16 (see `rmul`)
  float rmul;         // factor applied to the first product's result inside the exponential (EXACT instances), else 1
  // LIST mode: schedule (read-only), work-queue state and partial results of cut rows (in the caller's workspace)
  const int32_t* sched;
  int32_t* queue;     // [0] part items handed out, [1] leading work-groups done, [8 + rho*hbp + hb] finished parts of
                      // cut row rho, in a small launch the meetings of the row's parts that one side has come to
                      // (merge_tree); all zero between calls (each call puts back the zeros it disturbed)
  float* partials;    // [(cut part)*hbp + hb][(regs + 2) * threads], layout: park
  int32_t hbp;        // (batch, head) pairs per mask plane: B*H if Mb == 1, else H
  int32_t n_extra;    // leading work-groups that serve the queue of cut-row parts (LIST mode)
  int32_t G;          // (batch, head) planes whose block rows are interleaved in launch order
  int32_t split;      // most parts per block row when the launch is too small to fill the chip, else 1
  int32_t part_cap;   // records of `partials` the workspace holds; a schedule whose parts need more is not followed
};

__device__ __forceinline__ float partner_max(float x) {
  // lanes l and l^32 exchange: swap(x, x) gives {x[l%32], x[l%32 + 32]} in some order on every lane
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// s_waitcnt until at most n of the wave's memory operations are under way (they end in the order in which they were issued)
constexpr int wait_vm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | (n >> 4) << 14; }

// A barrier behind which LDS writes are seen, and which does not wait for copies on their way there.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

constexpr int kSplitMinTiles = 8;        // list entries that a part of a row in a small launch keeps (split_parts)
constexpr int kWin = 1024;               // tiles per schedule window (block columns, or list entries)
constexpr uint32_t kNoTile = 0xffffffffu;  // sentinel after the last entry of a window
constexpr uint32_t kZeroWord = 0x40000000u;  // entry flag: the tile's mask words are all zero and are not in memory

typedef bbm::InPlace<AttnParams> Args;

// Builds, in LDS, the ascending list of tiles one block row visits inside one schedule window; entry =
// block column | (1 << 31 if the element mask can be skipped there).  Returns the number of entries (uniform).
// `win` counts windows of kWin block columns.  (BITMAP, RUNS and DENSE_BASELINE; LIST mode copies its list instead.)
// [clo, chi): the block columns this work-group is responsible for (all of them unless the block row is computed in
// parts).
template <int NW>
__device__ __forceinline__ int build_window(Args P, int m, int i, int win, uint32_t* tiles_s, int* cnt_s, int clo, int chi) {
  constexpr int NT = NW * 64;
  constexpr int CH = kWin / 64;  // 64-column chunks per window
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r = (int64_t)m * P->nbr + i;
  int count;
  if (P->mode == BBM_MODE_DENSE_BASELINE) {
    const int j0 = clo + win * kWin;
    count = min(kWin, chi - j0);
    // an empty block's packed words are never written by the block reduction: flag it, the mask word is then 0
    const uint8_t* row = global(P->bin_blk_mat) + r * P->nbc;
    for (int t = tid; t < count; t += NT) tiles_s[t] = (uint32_t)(j0 + t) | (row[j0 + t] == 0 ? kZeroWord : 0u);
  } else {
    int lo = clo, hi = chi, run_lo = 0, run_hi = 0;
    if (P->mode == BBM_MODE_RUNS) {
      lo = max(clo, global(P->nz_lo)[r]);
      hi = min(chi, global(P->nz_hi)[r]);
      run_lo = global(P->offset)[r];
      run_hi = run_lo + global(P->total_ones)[r];
    }
    const int j0 = (lo & ~63) + win * kWin;
    const uint8_t* row = global(P->bin_blk_mat) + r * P->nbc;
    uint64_t nz[(CH + NW - 1) / NW];
#pragma unroll
    for (int n = 0; n < (CH + NW - 1) / NW; ++n) {
      const int ch = wave + n * NW;
      const int j = j0 + 64 * ch + lane;
      const uint8_t v = (ch < CH && j >= lo && j < hi) ? row[j] : (uint8_t)0;
      nz[n] = __ballot(v != 0);
      if (ch < CH && lane == 0) cnt_s[ch] = __popcll(nz[n]);
    }
    __syncthreads();
    int total = 0, before = 0;
    for (int ch = 0; ch < CH; ++ch) {
      const int cn = cnt_s[ch];
      total += cn;
    }
    count = total;
#pragma unroll
    for (int n = 0; n < (CH + NW - 1) / NW; ++n) {
      const int ch = wave + n * NW;
      if (ch < CH) {
        before = 0;
        for (int c2 = 0; c2 < ch; ++c2) before += cnt_s[c2];
        if ((nz[n] >> lane) & 1ull) {
          const int j = j0 + 64 * ch + lane;
          const bool in_run = (P->mode == BBM_MODE_RUNS) && j >= run_lo && j < run_hi;
          tiles_s[before + __popcll(nz[n] & ((1ull << lane) - 1ull))] = (uint32_t)j | (in_run ? 0x80000000u : 0u);
        }
      }
    }
  }
  count = __builtin_amdgcn_readfirstlane(count);
  if (tid < 3) tiles_s[count + tid] = kNoTile;
  __syncthreads();
  return count;
}

// Number of schedule windows of the block columns [clo, chi) of one block row (uniform).
__device__ __forceinline__ int num_windows(Args P, int m, int i, int clo, int chi) {
  int lo = clo, hi = chi;
  if (P->mode == BBM_MODE_RUNS) {
    const int64_t r = (int64_t)m * P->nbr + i;
    lo = max(clo, global(P->nz_lo)[r]);
    hi = min(chi, global(P->nz_hi)[r]);
  }
  if (hi <= lo) return 0;
  if (P->mode != BBM_MODE_DENSE_BASELINE) lo &= ~63;
  return (hi - lo + kWin - 1) / kWin;
}

// One work-group per (block row, batch, head), tiles from build_window.  SCHED = 2 (a launch too small to fill the chip):
// every block row is computed in up to P->split equal parts by as many work-groups, which merge them in pairs (merge_tree).
// With SCHED = 1 (LIST mode) the first
// P->n_extra work-groups, before turning to their own block row, take the parts of the block rows which the split
// schedule cut from a queue; the work-group that completes a row's last part merges the parts in part order and
// writes the row, and the row's own work-group skips it.
//
// The softmax needs exp2(c * <q, k> - m) with c = softmax_scale * log2(e).  EXACT = false: Q is multiplied by c and
// rounded to bf16, so the first product delivers the exponent directly (no per-element multiplication; the rounding
// moves a score by up to 2^-9 * c * sum |q_d k_d|, harmless up to the usual scale 1/sqrt(d)).  EXACT = true (sharper
// scales): c = 2^k * r with r in [1, 2); Q is multiplied by 2^k, which is exact in bf16, and r multiplies the
// accumulator inside the exponential; running maxima are then kept in units of 1/r.
template <int D, int NW, int SCHED, bool EXACT>
__global__ __launch_bounds__(NW * 64, D == 64 && NW == 4 ? 3 : NW >= 4 ? 2 : 1) void attn_fwd_kernel(const AttnParams) {
  Args P = bbm::kernel_args<AttnParams>();
  constexpr int NT = NW * 64;
  constexpr int BR = NW * 32;
  // LDS tile layout ("blocks"): one asynchronous copy instruction of a wave fills one 1 KiB block with RPB rows
  // that lie NBLK rows apart: row r sits in block r % NBLK at slot r / NBLK.  Blocks are padded (K by 16 bytes, V
  // by 64) so that the 16 consecutive rows a 16-byte K read touches, and the 4 consecutive rows a transposing V
  // read touches, start in different banks.  Every read address is one per-lane register plus a constant.
  constexpr int RC = D / 8;                    // 16-byte chunks per row
  constexpr int RPB = 64 / RC;                 // rows per 1 KiB block
  constexpr int NBLK = kBc / RPB;              // blocks per tile = copy instructions per tile
  constexpr int LPW = NBLK / NW;               // copy instructions per wave and tile
  static_assert(NBLK % NW == 0, "tile must split evenly over the waves");
  constexpr int KBLK = 512 + 8;                // K block stride in elements (1 KiB + 16 B)
  constexpr int VBLK = 512 + 32;               // V block stride in elements (1 KiB + 64 B)
  constexpr int KS = D / 16;                   // MFMA k-steps of the first product
  constexpr int DB = D / 32;                   // 32-wide output-column blocks of the second product
  constexpr int REGS = DB * 16;                // fp32 accumulator registers per lane
  static_assert(2 * 32 * D <= NBLK * KBLK && NW <= 8, "two 32 x D output slabs must fit in each tile buffer");

  // separate arrays per buffer so the compiler can tell an asynchronous copy into one from reads of the other
  __shared__ __attribute__((aligned(16))) __bf16 k_s0[NBLK * KBLK];
  __shared__ __attribute__((aligned(16))) __bf16 k_s1[NBLK * KBLK];
  __shared__ __attribute__((aligned(16))) __bf16 v_s0[NBLK * VBLK];
  __shared__ __attribute__((aligned(16))) __bf16 v_s1[NBLK * VBLK];
  __shared__ uint32_t tiles_s[kWin + 4];
  __shared__ int cnt_s[kWin / 64];
  __shared__ int item_s[2];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform by construction: keep it in a scalar register
  const int64_t N = P->N, Nk = P->Nk;
  const float c = P->qscale;
  const float rr = EXACT ? P->rmul : 1.0f;
  auto ex2 = [&](float x) { return __builtin_amdgcn_exp2f(EXACT ? rr * x : x); };

  // ---- per-item state (SCHED = false: exactly one item, derived from blockIdx)
  int m, i, bh;
  const __bf16* __restrict__ Kg;
  const __bf16* __restrict__ Vg;
  int64_t head_off;
  const uint64_t* __restrict__ mrow;
  bf16x8 qf[KS];
  f32x16 oacc[DB];
  // m_run: reference maximum of the row in exponent units (score * scale * log2 e; -inf before the first visible key);
  // s_init: its negative (0 while m_run = -inf), replicated, as the start value of the score accumulators
  float m_run, l_run;
  f32x16 s_init;

  // Q through LDS needs a 32 x D staging slab per wave in the two buffers of parity 1 (two slabs each)
  constexpr bool Q_VIA_LDS = NW <= 4;
  bool q_pending = false;
  // The row's list is asked for before Q and the first tile (and Q's fragments are picked up while that tile is under way), or behind
  // them, and everything is waited for at once: then it costs a trip to memory, but Q and the tile set off earlier, which matters
  // more where other work-groups of the CU fill the waiting.  Work-groups of whole rows, forward in us on other tensors call by call,
  // list first / behind:
  //   D = 64, 64 queries a row: windows of 3 x 9 x 1500 9.75 / 9.60, of 5 x 12 x 914 10.40 / 10.13; packed sequences of 3001 15.24 / 15.40
  //   D = 64, 128 queries: windows of 3 x 9 x 1500 10.49 / 9.96, of 5 x 12 x 914 11.15 / 10.68; packed sequences of 4096 38.7 / 38.5
  //   D = 64, 256 queries: within 0.4 %
  //   D = 128, 64 queries: packed sequences of 3001 25.8 / 26.9, of 4096 101.9 / 104.8, a window of 5 x 12 x 914 19.8 / 20.7
  //   D = 128, 128 queries: a window of 3 x 9 x 1500 15.5 / 14.5; packed sequences of 3001 24.2 / 24.4, of 4096 82.1 / 82.5
  //   D = 128, 256 queries: packed sequences of 3001 29.2 / 28.8, of 4096 94.3 / 93.4
  constexpr bool LIST_FIRST = SCHED != 1 || (D == 128 && NW == 2);
  // What a lane reads and copies where.  Found anew for every item at D = 128: kept across the merge of a cut row, some of it lay in
  // scratch memory, and the own row's list was asked for only when its first tile had landed (the wait for the reload).  At D = 64
  // there is room for it (packed sequences of 3001, 64 queries a row, 13.56 -> 13.40 us), except beside the merge of small launches
  // (a window over 8 heads of 4096 11.5 us with, 11.8 without).
  int lq, hh;          // query row of the wave's 32, half of the keys
  int g_row, g_chunk;  // row and 16-byte chunk this lane moves in a 1 KiB copy
  int kaddr, vaddr;    // see k_frag, v_frag
  uint32_t g_off;      // see copy_piece
  auto lane_places = [&]() __attribute__((always_inline)) {
    int ln = lane;
    if constexpr (D == 128 || SCHED == 2) asm volatile("" : "+v"(ln));
    lq = ln & 31, hh = ln >> 5;
    g_row = ln / RC, g_chunk = ln % RC;
    kaddr = (lq % NBLK) * KBLK + (lq / NBLK) * D + hh * 8;
    const int vy = (ln & 15) >> 2, vg = (ln >> 4) & 1, vx = (ln & 3) >> 1;
    vaddr = (4 * hh + vy) * VBLK + (2 * vg + vx) * 8 + 4 * (ln & 1);
    g_off = (uint32_t)((wave + g_row * NBLK) * D + g_chunk * 8) * 2u;
  };
  auto q_stage = [&]() { return (wave / 2 == 0 ? k_s1 : v_s1) + (wave % 2) * 32 * D; };
  auto begin_item = [&]() {
    lane_places();
    head_off = (int64_t)bh * N * D;
    Kg = global(P->k) + (int64_t)bh * Nk * D;
    Vg = global(P->v) + (int64_t)bh * Nk * D;
    const int64_t qrow = (int64_t)i * BR + wave * 32 + lq;
    const bool q_ok = qrow < N;
    // packed mask words of this lane's query row (rows past N borrow row 0: their results are never stored)
    mrow = global(P->packed) + (int64_t)m * P->W * N + (q_ok ? qrow : 0);
    // The wave's 32 x D slab of Q is one contiguous piece of memory: it is copied asynchronously, 1 KiB per instruction,
    // into this wave's staging slab (tile buffer 1, idle until the second tile is requested), where the MFMA fragments are picked
    // up.  Chunk j of row r lands at chunk position j ^ (r % RC) of row r.  Eight waves find no room there and read their fragments
    // themselves.  Rows past N come as zeros (their results are never stored).  (The buffer form: the compiler takes the global
    // form of the copy for a possible access to LDS by another path, and waits for all that is under way where it needs an
    // earlier load.  This alone: packed sequences of 3001 23.7 -> 22.7 us at D = 128, 13.44 -> 13.40 at D = 64.)
    const int64_t row0 = (int64_t)i * BR + wave * 32;
    const int rows = (int)max<int64_t>(0, min<int64_t>(32, N - row0));
    const __amdgpu_buffer_rsrc_t slab = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(global(P->q)) + head_off + row0 * D, 0,
                                                                          (int)scalar(rows * D * 2), 0x00027000);
    if constexpr (Q_VIA_LDS) {
      __bf16* const stage = q_stage();
#pragma unroll
      for (int n = 0; n < 32 / RPB; ++n) {
        const int r = n * RPB + g_row;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(slab, (void __attribute__((address_space(3)))*)(stage + n * 512), 16,
                                                 (uint32_t)(r * D + ((g_chunk ^ (r % RC)) * 8)) * 2u, 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int t = 0; t < KS; ++t)
        qf[t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(slab, (lq * D + 16 * t + 8 * hh) * 2, 0, 0));
    }
    q_pending = true;
#pragma unroll
    for (int db = 0; db < DB; ++db)
      for (int e = 0; e < 16; ++e) oacc[db][e] = 0.0f;
    m_run = -INFINITY;
    l_run = 0.0f;
    for (int e = 0; e < 16; ++e) s_init[e] = 0.0f;
  };

  // Asynchronous global -> LDS copy (no registers in between).  One instruction moves 1 KiB per wave: lane l lands at
  // LDS base + 16*l, i.e. slot l / RC, chunk l % RC of the block, so it fetches row (block + NBLK * slot).  copy_piece is
  // instruction n (0 .. 2*LPW-1) of the wave for the tile of list entry e; keys past Nk (`rows` of the 64 lie below it) come as
  // zeros from the bounds check of the buffer resource: they sit in a tile that is never "full", so the element mask gives them
  // probability exactly 0, and zeros add nothing.
  auto copy_piece = [&](int jt, int rows, __bf16* kd, __bf16* vd, int n) {
    const int p = n % LPW, blk = p * NW + wave;
    const __bf16* const tile = (n < LPW ? Kg : Vg) + (int64_t)jt * (kBc * D);
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(tile), 0, (int)scalar(rows * D * 2), 0x00027000);
    uint32_t off = g_off;
    asm volatile("" : "+v"(off));  // one register throughout the tile loop, not one per block
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (void __attribute__((address_space(3)))*)(n < LPW ? kd + blk * KBLK : vd + blk * VBLK), 16,
                                             off + p * NW * D * 2, 0, 0, 0);
  };
  auto rows_of_tile = [&](int jt) { return (int)scalar((uint32_t)max(0, min(kBc, (int)Nk - jt * kBc))); };
  auto copy_all = [&](int jt, __bf16* kd, __bf16* vd) {
    const int rows = rows_of_tile(jt);
#pragma unroll
    for (int n = 0; n < 2 * LPW; ++n) copy_piece(jt, rows, kd, vd, n);
  };

  // K fragment of MFMA k-step t, key block kb: row 32*kb + lq, chunk 2t + hh.
  auto k_frag = [&](const __bf16* ks, int kb, int t) {
    return *reinterpret_cast<const bf16x8*>(ks + kaddr + kb * (32 / NBLK) * D + t * 16);
  };

  // V fragment (transposing read) of 16-key step u, half a, column block db: the lane addresses row
  // vr = 16u + 8a + 4hh + y (y = (lane%16)/4), 16-byte chunk 4db + 2g + x (g = (lane/16)%2, x = (lane%4)/2),
  // elements 4*(lane%2).. of it, and receives keys 16u + 8a + 4hh + 0..3 of column 32db + lane%32 -- the key
  // order of the bf16 probabilities taken straight from the S^T accumulators.
  auto v_frag = [&](const __bf16* vs, int u, int db) {
    s16x4 part[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      // row 16u + 8a + (4hh + y): block (row % NBLK), slot (row / NBLK)
      const int off = D == 64 ? (2 * u + a) * D + db * 32 : 8 * a * VBLK + u * D + db * 32;
      part[a] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(vs + vaddr + off));
    }
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7));
  };

  const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

  // One tile: S^T = K Q^T, mask, online softmax and O^T += V^T P^T for tile e0 whose K and V sit in buffer PB, in two chains of
  // matrix instructions with everything that can be behind them: the asynchronous copies of the next tile behind the first, the
  // exponentials of the next 16 keys behind the second.  Against the copies in one go behind the first product and the
  // compiler's own order in the second (kernel times, us): 2 x 32 heads of 8192 dense tokens, D = 128, 2075 -> 1971, 1020 -> 996
  // causal; 4 x 16 causal heads of 4096, D = 64, 195 -> 185; packed sequences 46.6 -> 42.8; tree prefill 141 -> 133.  The maximum
  // of the first 32 keys behind the products of the second 32, with the mask in the start values: 2-7 % slower everywhere.
  uint32_t e0, e1_v;  // this step's list entry, and the next one's (as it came from LDS: made a scalar when the step starts)
  uint64_t mw_nxt;
  auto step = [&](auto pb, int it) __attribute__((always_inline)) {
    constexpr int PB = decltype(pb)::value;
    const uint64_t mw = mw_nxt;
    __builtin_amdgcn_s_waitcnt(0);  // this wave's asynchronous tile copies of the previous iteration have landed
    __syncthreads();                // ... and everyone's; every wave is also done with the buffers refilled below
    __bf16* const k_cur = PB ? k_s1 : k_s0;
    __bf16* const k_oth = PB ? k_s0 : k_s1;
    __bf16* const v_cur = PB ? v_s1 : v_s0;
    __bf16* const v_oth = PB ? v_s0 : v_s1;
    // The next tile's copies go out one by one between the matrix instructions of the first product: requested in one go they
    // fill the memory pipe's queue, and every wave of the work-group stands there.  Behind the last tile they copy zero rows into
    // buffers that nobody reads any more, cheaper than a branch around each.
    const uint32_t e1 = scalar(e1_v);
    const bool more = e1 != kNoTile, partial = (e0 >> 31) == 0;
    const int jt1 = more ? (int)(e1 & 0x3fffffffu) : 0, rows1 = more ? rows_of_tile(jt1) : 0;
    if (more) mw_nxt = (e1 >> 30) == 0 ? mrow[(int64_t)jt1 * N] : 0;
    e1_v = tiles_s[it + 2];
    // a partial tile in which none of this wave's 32 queries sees a key adds exact zeros: such a wave only takes part
    // in the copies and barriers of the step (not in the dense-tile baseline, which stands for a kernel that knows
    // nothing about the mask's structure)
    const bool live = !partial || (SCHED == 0 && P->mode == BBM_MODE_DENSE_BASELINE) || __ballot(mw != 0ull) != 0ull;
    if (!live && more) copy_all(jt1, k_oth, v_oth);
    e0 = e1;
    if (live) {
      f32x16 s[2];
      // Wave priority: the two phases that feed the matrix pipe are raised above the address arithmetic, copy requests
      // and maxima of the other waves on the SIMD, so a wave that has matrix work issues it first (dense masks: d=64
      // -3 %, d=128 -1.5 %; neutral on the short rows of packed sequences).
      __builtin_amdgcn_s_setprio(2);
      s[0] = s_init;
      s[1] = s_init;
      mfma_ring<2 * KS, 4>([&](auto i) { return k_frag(k_cur, decltype(i)::value & 1, decltype(i)::value >> 1); },
                           [&](auto i, bf16x8 f) {
                             constexpr int n = decltype(i)::value;
                             s[n & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[n >> 1], s[n & 1], 0, 0, 0);
                           },
                           [&](auto i) {
                             constexpr int n = decltype(i)::value, GAP = KS / LPW;  // matrix instructions per copy
                             if constexpr (n % GAP == 0) copy_piece(jt1, rows1, k_oth, v_oth, n / GAP);
                           });
      __builtin_amdgcn_s_setprio(0);

      // ---- element mask (only where the schedule cannot rule out zeros): keep s where the bit is set, else -inf
      if (partial) {
  #pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
          const uint32_t w = (uint32_t)(mw >> (32 * kb)) >> (4 * hh);
  #pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int bit = 8 * (e / 4) + (e % 4);
            const uint32_t keep = (uint32_t)((int32_t)(w << (31 - bit)) >> 31);  // all ones iff the bit is set
            s[kb][e] = __uint_as_float((__float_as_uint(s[kb][e]) & keep) | (0xff800000u & ~keep));
          }
        }
      }

      // ---- row maximum of this lane's query row
      float mx = s[0][0];
  #pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[kb][e]);
      mx = partner_max(mx);
      // The scores arrive relative to the reference (s = exponent - m_run).  The reference only moves when some row's
      // maximum exceeds it by more than kLazy: softmax is invariant to the reference, probabilities stay <= 2^kLazy, and
      // the rescale of O -- and here also the per-element subtraction -- is skipped on almost every tile.
      if (__any(((m_run == -INFINITY) ? (mx > -INFINITY) : (mx > kLazy)) ? 1 : 0)) {
        const float m_old = (m_run == -INFINITY) ? 0.0f : m_run;       // what the accumulators started from
        const float m_new = fmaxf(m_run, m_old + mx);
        const float m_fin = (m_new == -INFINITY) ? 0.0f : m_new;
        const float alpha = ex2(m_run - m_fin);
        const float shift = m_fin - m_old;
        l_run *= alpha;
        m_run = m_new;
  #pragma unroll
        for (int e = 0; e < 16; ++e) s_init[e] = -m_fin;
  #pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          for (int e = 0; e < 16; ++e) s[kb][e] -= shift;
  #pragma unroll
        for (int db = 0; db < DB; ++db)
          for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
      }

      __builtin_amdgcn_s_setprio(1);
      // ---- O^T += V^T P^T, the exponentials of a 16-key step behind the matrix instructions of the step before
      bf16x8 pf[2];
      auto exps = [&](int u, int e0, int e1) {
#pragma unroll
        for (int e = e0; e < e1; e += 2) {
          pf[u & 1][e] = (__bf16)ex2(s[u / 2][8 * (u % 2) + e]);
          pf[u & 1][e + 1] = (__bf16)ex2(s[u / 2][8 * (u % 2) + e + 1]);
          // row sum of the ROUNDED probabilities (the same numbers the second product consumes), two per instruction
          const bf16x2 pair = {pf[u & 1][e], pf[u & 1][e + 1]};
          l_run = __builtin_amdgcn_fdot2_f32_bf16(pair, ones2, l_run, false);
        }
      };
      exps(0, 0, 8);
      mfma_ring<4 * DB, 3>([&](auto i) { return v_frag(v_cur, decltype(i)::value / DB, decltype(i)::value % DB); },
                           [&](auto i, bf16x8 f) {
                             constexpr int n = decltype(i)::value;
                             oacc[n % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pf[n / DB & 1], oacc[n % DB], 0, 0, 0);
                           },
                           [&](auto i) {
                             constexpr int n = decltype(i)::value, PER = 8 / DB;
                             if constexpr (n / DB < 3) exps(n / DB + 1, n % DB * PER, (n % DB + 1) * PER);
                           });
      __builtin_amdgcn_s_setprio(0);
    }
  };

  // What begin_item asked for stays in front of what follows: Q's copies are waited for by the number of operations behind them.
  auto q_copies_first = [&]() { __builtin_amdgcn_sched_barrier(0); };

  // Starts the asynchronous copies of a window's first tile e (into buffer 0) and asks for its mask word.
  auto start_tile0 = [&](uint32_t e) {
    e0 = scalar(e);
    const int jt = (int)(e0 & 0x3fffffffu);
    copy_all(jt, k_s0, v_s0);
    mw_nxt = (e0 >> 30) == 0 ? mrow[(int64_t)jt * N] : 0;
  };

  // Runs the tiles listed in tiles_s[0 .. count) (followed by sentinels) through the pipeline; `started` says that
  // start_tile0 was already called for tiles_s[0].
  auto run_window = [&](int count, bool started) {
    if (!started) {
      q_copies_first();
      start_tile0(tiles_s[0]);
    }
    if (q_pending) {  // first window of a block row: Q fragments
      if constexpr (Q_VIA_LDS) {
        if constexpr (LIST_FIRST) {
          __builtin_amdgcn_s_waitcnt(wait_vm(2 * LPW));  // this wave's own copies of Q have landed, behind which it asked for the first tile
          auto pick_up = [&](const __bf16* stage) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < KS; ++t) qf[t] = *reinterpret_cast<const bf16x8*>(stage + lq * D + (((2 * t + hh) ^ (lq % RC)) * 8));
          };
          // (By variable, not through a pointer to either, which the compiler would make of this without the asm: it then waits for
          // no other copies.)
          if (wave < 2) {
            pick_up(k_s1 + wave * 32 * D);
#pragma unroll
            for (int t = 0; t < KS; ++t) asm volatile("; from k_s1" : "+v"(qf[t]));
          } else {
            pick_up(v_s1 + (wave & 1) * 32 * D);
#pragma unroll
            for (int t = 0; t < KS; ++t) asm volatile("; from v_s1" : "+v"(qf[t]));
          }
        } else {
          __builtin_amdgcn_s_waitcnt(0);
          const __bf16* const stage = q_stage();
#pragma unroll
          for (int t = 0; t < KS; ++t) qf[t] = *reinterpret_cast<const bf16x8*>(stage + lq * D + (((2 * t + hh) ^ (lq % RC)) * 8));
        }
      }
#pragma unroll
      for (int t = 0; t < KS; ++t)
        for (int e = 0; e < 8; ++e) qf[t][e] = (__bf16)((float)qf[t][e] * c);
      q_pending = false;
    }
    e1_v = tiles_s[1];
    for (int it = 0; it < count; it += 2) {
      step(IntC<0>{}, it);
      if (it + 1 < count) step(IntC<1>{}, it + 1);
    }
    __builtin_amdgcn_s_waitcnt(0);  // (the zero rows that the last step copied)
    __syncthreads();  // whoever comes next rewrites the tile list and the K/V buffers
  };

  // Runs nt >= 1 consecutive list entries, the first of which is already known: its copies start before the list
  // itself has been fetched.  `ahead` is this thread's entry, from ask_list, where the list is asked for first: it does not wait
  // behind the 64 KiB of Q and the first tile, and what is left to do before the first product (list to LDS, Q's fragments) is
  // done while the tile is on its way.
  auto ask_list = [&](const uint32_t* __restrict__ list, int nt) { return LIST_FIRST ? list[max(0, min(tid, nt - 1))] : 0u; };
  auto run_list = [&](const uint32_t* __restrict__ list, int nt, uint32_t first, uint32_t ahead) {
    if constexpr (LIST_FIRST) q_copies_first();
    start_tile0(first);
    for (int w0 = 0; w0 < nt; w0 += kWin) {
      const int count = min(kWin, nt - w0);
      int t = tid;
      if (LIST_FIRST && w0 == 0) {
        tiles_s[t] = t < nt ? ahead : kNoTile;
        t += NT;
      }
      for (; t < count; t += NT) tiles_s[t] = list[w0 + t];
      if (tid < 3) tiles_s[count + tid] = kNoTile;
      lds_barrier();  // (the first tile may still be on its way)
      run_window(count, w0 == 0);
    }
  };

  // normalise, round to bf16, store; fully masked rows give O = 0, lse = -inf.  The wave's 32 x D output slab goes
  // through LDS (the tile buffers are idle here: two slabs fit in each) so that the global stores are whole rows:
  // 16-byte chunk ch of row r sits at chunk position ch ^ (r % RC) of the row.
  auto write_output = [&]() {
    if (Q_VIA_LDS && q_pending) {  // a block row without tiles: its Q copies still target the slabs staged in below
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      q_pending = false;
    }
    const float l_tot = partner_sum(l_run);
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    __bf16* const stage = ((wave >> 1) == 0 ? k_s0 : (wave >> 1) == 1 ? k_s1 : (wave >> 1) == 2 ? v_s0 : v_s1) + (wave & 1) * 32 * D;
    // lane coordinates, re-derived behind an optimisation barrier: otherwise the per-lane staging addresses are
    // hoisted to the kernel's start and occupy registers throughout the tile loop
    int lqo = lq, hho = hh, gro = g_row, gco = g_chunk;
    asm volatile("" : "+v"(lqo), "+v"(hho), "+v"(gro), "+v"(gco));
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 ov;
        for (int e = 0; e < 4; ++e) ov[e] = (__bf16)(oacc[db][4 * g + e] * inv);
        *reinterpret_cast<bf16x4*>(stage + lqo * D + (((4 * db + g) ^ (lqo % RC)) * 8) + 4 * hho) = ov;
      }
    }
    const int64_t row0 = (int64_t)i * BR + wave * 32;
    bbm::store_rows<D>(stage, global(P->o) + head_off + row0 * D, (int)max<int64_t>(0, min<int64_t>(32, N - row0)), gro, gco);
    if (row0 + lqo < N && global(P->lse) && hho == 0)
      global(P->lse)[(int64_t)bh * N + row0 + lqo] = l_tot > 0.0f ? m_run * (rr / kLog2e) + __logf(l_tot) : -INFINITY;
  };

  // A parked partial result: the accumulators, then a (maximum, sum) pair per thread.
  constexpr int RECORD = (REGS + 2) * NT;
  auto park = [&](float* rec, int at) {
    const __amdgpu_buffer_rsrc_t r = bbm::record_rsrc(rec, RECORD);
    bbm::store_record<DB, NT>(r, at, oacc);
    bbm::store_pair<DB, NT>(r, at, m_run, l_run);
  };
  auto this_thread = [&]() {
    int at = tid;
    asm volatile("" : "+v"(at));  // keeps the addresses out of the tile loop
    return at;
  };

  // Cut rows: parks the result of part `part` of `nparts` of the row whose records start at rec0, pstride apart, and -- in the
  // work-group that arrives last at `counter` -- merges all of them in part order (the result does not depend on which part
  // came last) and writes the row.  The merge is a tail that nobody else can help with, so the maxima are read eight records at a
  // time and the records two at a time: with a load at a time the forward took 144 instead of 96 us at 8 heads of 16384 tokens,
  // window, global tokens and random blocks, D = 128, and 106-111 instead of 92-100 at 16 heads, D = 64.
  auto park_and_merge = [&](float* rec0, int64_t pstride, int part, int nparts, int32_t* counter, int next_item) {
    const int at = this_thread();
    park(rec0 + part * pstride, at);
    bbm::hand_over();
    if (tid == 0) {
      item_s[1] = atomicAdd(counter, 1);
      item_s[0] = next_item;
    }
    __syncthreads();
    if (item_s[1] != nparts - 1) return;
    float m_all = -INFINITY;
#pragma unroll 1
    for (int k = 0; k < nparts; k += 8) {
      float2 ml[8];
#pragma unroll
      for (int n = 0; n < 8; ++n) ml[n] = bbm::load_pair<DB, NT>(bbm::record_rsrc(rec0 + min(k + n, nparts - 1) * pstride, RECORD), at);
#pragma unroll
      for (int n = 0; n < 8; ++n) m_all = fmaxf(m_all, ml[n].x);
    }
    const float m_fin = (m_all == -INFINITY) ? 0.0f : m_all;
#pragma unroll
    for (int db = 0; db < DB; ++db)
      for (int e = 0; e < 16; ++e) oacc[db][e] = 0.0f;
    l_run = 0.0f;
    bbm::for_records<DB, NT, true, 2>(rec0, pstride, nparts, at, [&](const f32x16 (&x)[DB], float2 ml) {
      const float wgt = ex2(ml.x - m_fin);
      l_run += wgt * ml.y;
#pragma unroll
      for (int db = 0; db < DB; ++db)
        for (int e = 0; e < 16; ++e) oacc[db][e] += wgt * x[db][e];
    });
    m_run = m_all;
    write_output();
    if (tid == 0) *counter = 0;  // last user of this counter: leave it zero for the next call
  };

  // Rows in S parts that run side by side: the parts meet in pairs, the pairs in pairs of pairs, ..  At every meeting the group
  // that comes first parks its result and leaves, the second one merges it into its own and goes on, so the work-group that comes
  // last of all reads one record per level, not all S, and parks nothing.  Which groups meet is fixed and the merge treats its two
  // sides alike, so the result does not depend on who comes when.  `met` holds one bit per meeting: set by the first to come.
  // 256 queries x 32 heads against 16640 keys, D = 128, 8 parts: with one work-group merging all records of a row behind
  // device-wide fences, parking took 16-22 us and merging 26 us of 118.
  auto merge_tree = [&](float* rec0, int64_t pstride, int part, int S, int32_t* met) {
    const int at = this_thread();
    int g = part, node0 = 0;
#pragma unroll 1
    for (int l = 0; (1 << l) < S; ++l, g >>= 1) {
      const int groups = (S + (1 << l) - 1) >> l, other = g ^ 1;
      const int32_t bit = 1 << (node0 + (g >> 1));
      node0 += (groups + 1) >> 1;
      if (other >= groups) continue;  // nobody to meet at this level
      if (tid == 0) item_s[1] = __hip_atomic_load(met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit;
      __syncthreads();
      if (item_s[1] == 0) {
        park(rec0 + ((int64_t)g << l) * pstride, at);
        bbm::hand_over();
        if (tid == 0) item_s[0] = atomicOr(met, bit) & bit;
        __syncthreads();
        if (item_s[0] == 0) return;
      }
      const __amdgpu_buffer_rsrc_t other_rec = bbm::record_rsrc(rec0 + ((int64_t)other << l) * pstride, RECORD);
      const float2 ml = bbm::load_pair<DB, NT>(other_rec, at);
      f32x16 x[DB];
      bbm::load_record<DB, NT>(other_rec, at, x);
      const float m_new = fmaxf(m_run, ml.x), m_fin = (m_new == -INFINITY) ? 0.0f : m_new;
      const float w_own = ex2(m_run - m_fin), w_other = ex2(ml.x - m_fin);
      {
#pragma clang fp contract(off)  // both products are rounded, whichever side is the one in registers
        l_run = w_own * l_run + w_other * ml.y;
#pragma unroll
        for (int db = 0; db < DB; ++db)
          for (int e = 0; e < 16; ++e) oacc[db][e] = w_own * oacc[db][e] + w_other * x[db][e];
      }
      m_run = m_new;
      __syncthreads();  // everyone has read item_s before the next level's is written
    }
    write_output();
    if (tid == 0) *met = 0;  // last user of this word: leave it zero for the next call
  };

  // ---- a launch too small to fill the chip: work-group = (block row, part), merged by merge_tree
  if constexpr (SCHED == 2) {
    int nbr = P->nbr, Mb = P->Mb, H = P->H, split = P->split, mode = P->mode;
    asm volatile("" : "+s"(nbr), "+s"(Mb), "+s"(H), "+s"(split), "+s"(mode) : "s"(P->q));  // in one go, see below
    int part = (int)blockIdx.x % split;
    const int rest = (int)blockIdx.x / split;
    int S = split;  // parts of this row
    bh = rest / nbr;
    i = nbr - 1 - (rest - bh * nbr);
    m = (Mb == 1) ? 0 : bh / H;
    const int hb = (Mb == 1) ? bh : bh - m * H;
    if (mode == BBM_MODE_LIST) {  // equal shares of the row's list, none shorter than kSplitMinTiles entries if there are several
      const int32_t* rp = global(P->row_ptr) + (int64_t)m * (nbr + 1) + i;
      const int p_row = rp[0], n_row = rp[1] - rp[0];
      S = max(1, min(S, n_row / kSplitMinTiles));
      // Work-groups go to the eight XCDs in turn: if the same ones of every row were left over, some XCDs would get no work (rows
      // of 6 to 10 entries, left whole: a window over 8 heads of 4096, D = 64, 14.3 -> 12.6 us; over one head of 16384, D = 128,
      // 25.7 -> 20.8).  Rows in all their parts keep the order in which the rows of a head read one part's keys on one XCD.
      if (S < P->split) part = (part + rest * P->split / 8) % P->split;
      if (part >= S) return;
      const int chunk = (n_row + S - 1) / S;
      const int nt = max(0, min(chunk, n_row - part * chunk));
      const int p0 = p_row + (nt > 0 ? part * chunk : 0);  // (an entry is asked for in any case: of a row without any, there is one behind it)
      const uint32_t* __restrict__ list = global(P->col_idx) + (int64_t)m * P->nbr * P->nbc + p0;
      const uint32_t first = list[0], ahead = ask_list(list, nt);
      begin_item();
      if (nt > 0) run_list(list, nt, first, ahead);
    } else {  // BITMAP, RUNS: equal shares of the block columns
      begin_item();
      const int chunk = (P->nbc + S - 1) / S;
      const int clo = part * chunk, chi = min(P->nbc, clo + chunk);
      const int nwin = num_windows(P, m, i, clo, chi);
      for (int win = 0; win < nwin; ++win) {
        const int count = build_window<NW>(P, m, i, win, tiles_s, cnt_s, clo, chi);
        if (count > 0) run_window(count, false);
      }
    }
    if (Q_VIA_LDS && q_pending) {  // nothing was computed: let the Q copies land before anyone reuses the slabs
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      q_pending = false;
    }
    const int row = m * P->nbr + i;
    merge_tree(global(P->partials) + ((int64_t)row * P->split * P->hbp + hb) * ((REGS + 2) * NT), (int64_t)P->hbp * ((REGS + 2) * NT), part, S,
               global(P->queue) + 8 + row * P->hbp + hb);
    return;
  }

  // ---- which block row is this work-group's own?  Work-groups are handed to the 8 XCDs round-robin; give each XCD a
  // contiguous range of logical ids so the row blocks of one head (which share K and V) meet in one XCD's L2.
  // Launch order inside a group of G consecutive (batch, head) planes: rank-major, i.e. rank 0 of every plane of the
  // group, then rank 1 of every plane, ...  The hardware starts work-groups in index order as slots free up, so
  // with ranks sorted by length long rows start early everywhere and the short ones fill the tail.
  // The arguments this takes are asked for in one go (hence the asm), and with them one from every cache line of the argument
  // segment, which is cold when a kernel starts.  The compiler would read each where it is needed, a trip to memory for every line
  // in turn; and since a scalar load is waited for together with all that are under way, one of them stood between the schedule's
  // header and the row's record below, which then followed each other, too.  Over 45 shapes on other tensors call by call: 1 % of the
  // forward, a dilated window of 2 x 7 x 670, D = 64, 256 queries a row, 10.41 -> 10.23 us, windows of 5 x 12 x 914, D = 128, 64 queries
  // a row, 20.3 -> 19.8.  (Header and record through the constant address space, so that they are scalar loads: no kernel that reads
  // a schedule writes one.)
  static_assert(sizeof(AttnParams) <= 256 && offsetof(AttnParams, q) / 64 == 0 && offsetof(AttnParams, H) / 64 == 1 && offsetof(AttnParams, nbr) / 64 == 2 &&
                    offsetof(AttnParams, G) / 64 == 3 && offsetof(AttnParams, split) / 64 == 3, "one argument of every line is among those below");
  int own_bh, own_m, own_rank;
  int T = P->total_wgs, G = P->G, nbr = P->nbr, Mb = P->Mb, H = P->H, hbp = P->hbp, part_cap = P->part_cap, nbc = P->nbc, n_extra = P->n_extra;
  uint64_t sched_at = reinterpret_cast<uint64_t>(P->sched);
  asm volatile("" : "+s"(T), "+s"(G), "+s"(nbr), "+s"(Mb), "+s"(H), "+s"(hbp), "+s"(part_cap), "+s"(nbc), "+s"(n_extra), "+s"(sched_at) : "s"(P->q));
  {
    const int wg = (int)blockIdx.x;
    const int xcd = wg & 7, slot = wg >> 3;
    const int per = T >> 3, rem = T & 7;
    const int logical = xcd * per + (xcd < rem ? xcd : rem) + slot;
    const int grp = logical / (G * nbr), within = logical - grp * (G * nbr);
    const int g_planes = min(G, T / nbr - grp * G);
    own_rank = within / g_planes;
    own_bh = grp * G + (within - own_rank * g_planes);
    own_m = (Mb == 1) ? 0 : own_bh / H;
  }
  // LIST mode: the schedule's header (parts, split threshold) and this work-group's row record -- which block row has
  // its rank, where its list lies and how it starts -- are requested together: one round trip, not three
  typedef int32_t int4x __attribute__((ext_vector_type(4)));
  int4x own_rec = {0, 0, 0, -1};
  int nparts_all = 0, split_T = 0;
  if (SCHED == 1) {
    const auto sched = reinterpret_cast<const int4x __attribute__((address_space(4)))*>(sched_at);
    const int4x hdr = sched[0];
    static_assert(bbm::kSchedPartBase % 4 == 0 && bbm::kSchedPartInts % 4 == 0 && bbm::kSchedRowInts == 4, "records of 16 bytes");
    own_rec = sched[bbm::sched_order_base(Mb, nbr) / 4 + own_m * nbr + own_rank];
    nparts_all = hdr[bbm::kSchedNParts];
    split_T = hdr[bbm::kSchedSplitT];
    // a workspace too small for the partial results of every (part, head) item: no row is computed in parts
    // (the same decision in every work-group: it depends on the header and the launch only)
    if ((int64_t)nparts_all * hbp > (int64_t)part_cap) {
      nparts_all = 0;
      split_T = 0x7fffffff;
    }
  }
  // ---- LIST mode, the first n_extra work-groups: before their own block row they serve the queue of cut-row parts
  // (nothing to do, and no cost, when the schedule cut no row).  The tile loop is in the program twice, here and below: with one
  // loop for parts and own row the short rows of packed sequences took 44.9 us instead of 41.8, a 16384-token window 123 instead
  // of 115 (the backward kernels, which are short of registers, gained from it).
  if (SCHED == 1 && (int)blockIdx.x < n_extra) {
    const int n_items = nparts_all * P->hbp;
    // The first item of a work-group is its own index; later ones come from the queue counter, which therefore stands
    // for "n_extra items already handed out".
    int item = blockIdx.x;
    while (item < n_items) {
      int next_item = 0;
      if (tid == 0) next_item = P->n_extra + atomicAdd(global(P->queue), 1);  // asked now, needed after this item
      const int hb = item / nparts_all;
      const int32_t* seg = global(P->sched) + bbm::kSchedPartBase + (int64_t)bbm::kSchedPartInts * (item - hb * nparts_all);
      const int row = seg[0], p0 = seg[1], nt = seg[2], part = seg[3], nparts = seg[4], q_first = seg[5], rho = seg[6];
      m = row / P->nbr;
      i = row - m * P->nbr;
      bh = (P->Mb == 1) ? hb : m * P->H + hb;
      const uint32_t* const list = global(P->col_idx) + (int64_t)m * P->nbr * P->nbc + p0;
      const uint32_t ahead = ask_list(list, nt);
      begin_item();
      run_list(list, nt, (uint32_t)seg[7], ahead);
      park_and_merge(global(P->partials) + ((int64_t)q_first * P->hbp + hb) * ((REGS + 2) * NT), (int64_t)P->hbp * ((REGS + 2) * NT), part, nparts,
                     global(P->queue) + 8 + rho * P->hbp + hb, next_item);
      item = (int)scalar((uint32_t)item_s[0]);  // (a scalar: everything that addresses the item follows from it)
      __syncthreads();  // everyone has read the item, and the staged output, before the next item's copies and list land
    }
    // the last leading work-group to leave the queue puts the two queue counters back to zero for the next call
    if (n_items > 0 && tid == 0 && atomicAdd(global(P->queue) + 1, 1) == P->n_extra - 1) {
      global(P->queue)[0] = 0;
      global(P->queue)[1] = 0;
    }
  }

  bh = own_bh;
  m = own_m;
  if (SCHED == 1) {
    i = own_rec.x;
    const int n_list = own_rec.z;
    const uint32_t* const list = global(P->col_idx) + (int64_t)m * nbr * nbc + own_rec.y;
    const uint32_t ahead = ask_list(list, n_list);
    begin_item();
    if (n_list <= split_T) {  // a row the schedule cut belongs to the queue
      if (n_list > 0) run_list(list, n_list, (uint32_t)own_rec.w, ahead);
      write_output();
    }
  } else {
    i = P->nbr - 1 - own_rank;  // from the last row up: long rows first for causal-like masks
    begin_item();
    const int nwin = num_windows(P, m, i, 0, P->nbc);
    for (int win = 0; win < nwin; ++win) {
      const int count = build_window<NW>(P, m, i, win, tiles_s, cnt_s, 0, P->nbc);
      if (count > 0) run_window(count, false);
    }
    write_output();
  }
}

// Leading work-groups that serve the queue of cut-row parts before their own block row (LIST mode).
constexpr int kExtraWGs = 256;

constexpr size_t kQueueAlign = 256;
inline size_t queue_bytes(int64_t Mb, int64_t nbr, int64_t hbp) {
  const size_t n = (size_t)(8 + Mb * nbr * hbp) * sizeof(int32_t);
  return (n + kQueueAlign - 1) / kQueueAlign * kQueueAlign;
}
// one parked partial result: the fp32 accumulators of a work-group plus its running maximum and sum
inline size_t record_bytes(int d, int Br) { return (size_t)((d / 32 * 16 + 2) * (Br * 2)) * sizeof(float); }
// Partial results of cut rows: at most Mb*nbr cut parts exist (T >= 2 * mean list length), one record per (cut part,
// head-batch); in practice a handful of rows is cut (8 parts x 16 heads = 4.4 MB on the long-context workload), so
// the workspace asked for stops at kPartialCapBytes and a schedule that would need more is not followed (the rows
// are then computed whole: slower, same results up to the rounding order of the merge).
constexpr size_t kPartialCapBytes = 32u << 20;
inline size_t partial_bytes(int64_t Mb, int64_t nbr, int64_t hbp, int d, int Br) {
  return std::min((size_t)(Mb * nbr * hbp) * record_bytes(d, Br), kPartialCapBytes);
}

// A launch of at most kSplitUpTo work-groups leaves CUs idle or with a single work-group (a few block rows of new
// tokens against a long key/value cache; one long sequence with few heads): every block row is then computed in
// split_parts() parts.  A part costs a prologue, one record parked (64 KiB at d = 128) and a share of the merge, so LIST mode
// takes as many as give every CU one work-group and leave a part kSplitMinTiles block columns, or, if that leaves a part
// kSplitLongTiles, as many as give it two, up to 8: numbers in between leave some CUs with two and some with one.  At
// d = 128 a second work-group per CU takes twice kSplitLongTiles where memory is the bound: with one block row per head, or
// from kSplitWide work-groups on.  The kernel lowers the number for rows whose list is shorter than that.
// All keys seen, us, in 1 / 2 / 4 / 8 / 16 / 32 parts.  One block row of 128 queries per head, d = 128:
//   1 head x 1024 keys 20 / 16 / 16;   x 4096 62 / 37 / 26 / 22 / 22;   x 16384 239 / 123 / 69 / 44 / 33 / 29
//   16 heads x 4096 64 / 38 / 28 / 25 / 28;   x 16384 236 / 125 / 72 / 47 / 41 / 72;   32 x 8192 121 / 69 / 45 / 39 / 60
//   64 x 8192 124 / 76 / 57 / 70;   64 x 16384 289 / 162 / 114 / 122;   128 x 4096 68 / 52 / 61;   256 x 4096 106 / 109
// and d = 64: 64 x 32768 391 / 208 / 128 / 116 / 157;   128 x 8192 100 / 61 / 54 / 83;   256 x 4096 56 / 49 / 75.
// Two block rows, d = 128: 32 heads x 8192 122 / 70 / 51 / 62;   x 16384 242 / 133 / 93 / 95 (with inputs that come from
// memory 110 in 4, 106 in 8);   x 32768 544 / 303 / 193 / 157;   64 x 8192 135 / 91 / 95;   128 x 4096 80 / 86.
// 32 block rows of one head x 32768, d = 128: 468 / 245 / 132 / 84 / 93.
// Lists are not known here.  At d = 64, 256 work-groups over 64 block columns (8 heads of 4096 queries) go from 63 to 37 us in two
// parts on a causal mask, from 61 to 41 with global tokens; rows of 6 to 12 entries, left whole, pay for 256 work-groups that leave at
// once: a window 12.8 -> 12.6, packed sequences 17.0 -> 17.1, a dilated window 16.4 -> 17.5.
// Self-attention (as many queries as keys: what a backward pass follows) over fewer than 2 * kSplitLongTiles block columns is
// left whole, as it always was: there the results, and through them the gradients, do not depend on the block height.  The number
// of parts does, so from 64 block columns on they do too.  What that costs: 2 causal heads of 4032 at d = 128 take 72 us, of 4096,
// in 4 parts, 29; cut like the rest, 1 head x 1024 would take 16 us instead of 20.
// BITMAP and RUNS, which cut the block columns into equal ranges and so do not know how long a part's list is, keep to parts of
// kSplitLongTiles columns (twice that from kSplitWide work-groups on) and at most eight.  Those limits were measured when one
// work-group merged all parts behind device-wide fences, not since.
constexpr int kSplitUpTo = 256, kSplitWide = 128, kSplitOne = 256, kSplitTwo = 512, kSplitMax = 32, kSplitLongTiles = 32;
static_assert(kSplitMax <= 32, "one bit of a 32-bit word for each of the at most kSplitMax - 1 meetings of merge_tree");
inline int split_parts(int64_t total_wgs, int64_t nbr, int64_t nbc, int d, bool list, bool self) {
  if (total_wgs > kSplitUpTo || (self && nbc < 2 * kSplitLongTiles)) return 1;
  const int64_t two = kSplitTwo / total_wgs;
  int64_t s;
  if (list) {
    const int64_t long_tiles = d == 128 && (nbr == 1 || total_wgs >= kSplitWide) ? 2 * kSplitLongTiles : kSplitLongTiles;
    s = std::min<int64_t>({kSplitMax, kSplitOne / total_wgs, nbc / kSplitMinTiles});
    if (nbc >= std::min<int64_t>(8, two) * long_tiles) s = std::max<int64_t>(s, std::min<int64_t>(8, two));
  } else {
    const int64_t min_tiles = total_wgs < kSplitWide ? kSplitLongTiles : 2 * kSplitLongTiles;
    s = std::min<int64_t>(std::min<int64_t>(8, two), nbc / min_tiles);
  }
  return s < 2 ? 1 : (int)s;
}

template <int D, int NW, bool EXACT>
int launch(AttnParams& P, int64_t Mb, void* workspace, size_t workspace_bytes, hipStream_t s) {
  const size_t qb = queue_bytes(Mb, P.nbr, P.hbp);
  const bool have_ws = workspace && bbm::aligned(workspace, 16) && workspace_bytes >= qb + record_bytes(D, NW * 32);
  const int64_t cap = have_ws ? (int64_t)std::min<size_t>((workspace_bytes - qb) / record_bytes(D, NW * 32), 0x7fffffff) : 0;
  if (have_ws) {
    P.queue = static_cast<int32_t*>(workspace);
    P.partials = reinterpret_cast<float*>(static_cast<char*>(workspace) + qb);
    P.part_cap = (int32_t)cap;
    // a launch too small to fill the chip computes every block row in parts (not the dense-tile baseline, which stands
    // for the plain one-program-per-query-block kernel)
    if (P.mode != BBM_MODE_DENSE_BASELINE) P.split = split_parts(P.total_wgs, P.nbr, P.nbc, D, P.mode == BBM_MODE_LIST, P.N == P.Nk);
    while (P.split > 1 && (int64_t)P.total_wgs * P.split > cap) --P.split;  // every (row, part, head) parks a record
  }
  if (P.split > 1) {
    attn_fwd_kernel<D, NW, 2, EXACT><<<(unsigned)(P.total_wgs * P.split), NW * 64, 0, s>>>(P);
  } else if (P.mode == BBM_MODE_LIST) {
    P.n_extra = P.total_wgs < kExtraWGs ? P.total_wgs : kExtraWGs;
    attn_fwd_kernel<D, NW, 1, EXACT><<<(unsigned)P.total_wgs, NW * 64, 0, s>>>(P);
  } else {
    attn_fwd_kernel<D, NW, 0, EXACT><<<(unsigned)P.total_wgs, NW * 64, 0, s>>>(P);
  }
  return bbm::launch_status("bbm_attn_fwd");
}

}  // namespace

extern "C" __attribute__((visibility("default"))) size_t bbm_attn_fwd_workspace_bytes(int64_t B, int64_t H, int64_t N, int d, int Br, int Bc, int mode) {
  if (B < 1 || H < 1 || N < 1 || Br < 1 || Bc < 1 || (d != 64 && d != 128)) return 0;
  if (mode != BBM_MODE_LIST && mode != BBM_MODE_AUTO && mode != BBM_MODE_BITMAP && mode != BBM_MODE_RUNS) return 0;
  // sized for the larger of the two plane counts a caller may use (Mb = 1 or Mb = B): both give Mb*hbp = B*H
  // (N counts the queries; the number of keys is not known here, so the largest split of a small launch is assumed)
  const int64_t nbr = (N + Br - 1) / Br;
  const int split = split_parts(B * H * nbr, nbr, 1 << 30, d, mode == BBM_MODE_LIST || mode == BBM_MODE_AUTO, false);
  if (split > 1) return queue_bytes(1, nbr, B * H) + (size_t)(B * H * nbr * split) * record_bytes(d, Br);
  if (mode == BBM_MODE_BITMAP || mode == BBM_MODE_RUNS) return 0;  // these only ever use it for a small launch
  return queue_bytes(1, nbr, B * H) + partial_bytes(1, nbr, B * H, d, Br);
}

// ---- Scratch of bbm_attn_fwd_static: a file-scope device array instead of a caller's workspace, for callers that
// cannot allocate.  Every GPU the library runs on holds its own copy at its own address; host code only ever uses the
// address hipGetSymbolAddress returned for the current device, never the array's name.
constexpr size_t kStaticScratchBytes = 32u << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device, kept afterwards).
int static_scratch_address(const char* fn, void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return bbm::fail(BBM_EHIP, "%s: hipGetDevice: %s", fn, hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return bbm::fail(BBM_EUNSUPPORTED, "%s: device %d is beyond the %d devices the static scratch serves", fn, dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return bbm::fail(BBM_EHIP, "%s: hipGetSymbolAddress(scratch): %s", fn, hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return BBM_OK;
}

// The queue counters at the head of the scratch must be zero when the attention kernel starts.  (A fill kernel, not a
// memset: a caller may be recording the stream into a graph.)
__global__ __launch_bounds__(256) void clear_counters_kernel(int32_t* counters, int n) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < n) counters[t] = 0;
}
}  // namespace

namespace {
int attn_fwd_impl(const char* fn, const void* q, const void* k, const void* v, void* o, float* lse, int64_t B, int64_t H, int64_t N, int64_t Nk,
                  int d, float softmax_scale, int64_t Mb, const uint64_t* packed_mask, const bbm_index* idx, int mode,
                  void* workspace, size_t workspace_bytes, void* stream, bool use_static) {
  using namespace bbm;
  clear_error();
  if (!q || !k || !v || !o) return fail(BBM_EINVAL, "%s: q, k, v, o must not be NULL", fn);
  if (!aligned(q, 16) || !aligned(k, 16) || !aligned(v, 16) || !aligned(o, 16))
    return fail(BBM_EINVAL, "%s: q, k, v, o must be 16-byte aligned", fn);
  if (lse && !aligned(lse, 4)) return fail(BBM_EINVAL, "%s: lse must be 4-byte aligned", fn);
  if (B < 1 || H < 1 || N < 1 || Nk < 1)
    return fail(BBM_EINVAL, "%s: B=%lld, H=%lld, N=%lld (queries), %lld (keys) must be >= 1", fn, (long long)B, (long long)H, (long long)N, (long long)Nk);
  if (!(softmax_scale > 0.0f) || !(softmax_scale < INFINITY)) return fail(BBM_EINVAL, "%s: softmax_scale must be finite and > 0", fn);
  if (Mb != 1 && Mb != B) return fail(BBM_EINVAL, "%s: Mb=%lld must be 1 or B=%lld", fn, (long long)Mb, (long long)B);
  if (!idx) return fail(BBM_EINVAL, "%s: idx must not be NULL", fn);
  if (!packed_mask || !aligned(packed_mask, 8)) return fail(BBM_EINVAL, "%s: packed_mask must be a non-NULL 8-byte aligned pointer", fn);
  if (d != 64 && d != 128) return fail(BBM_EUNSUPPORTED, "%s: d=%d has no kernel instance (64, 128)", fn, d);
  if (idx->Bc != kBc || (idx->Br != 64 && idx->Br != 128 && idx->Br != 256))
    return fail(BBM_EUNSUPPORTED, "%s: tile (Br=%d, Bc=%d) has no kernel instance (Br in {64,128,256}, Bc = 64)", fn, idx->Br, idx->Bc);
  const int64_t nbr = ceil_div(N, idx->Br), nbc = ceil_div(Nk, idx->Bc);
  if (idx->Nq != N || idx->Nk != Nk)
    return fail(BBM_EINVAL, "%s: index built for a mask of %lld x %lld does not match %lld queries x %lld keys", fn, (long long)idx->Nq,
                (long long)idx->Nk, (long long)N, (long long)Nk);
  if (idx->Mb != Mb || idx->nbr != nbr || idx->nbc != nbc)
    return fail(BBM_EINVAL, "%s: index (Mb=%lld, nbr=%lld, nbc=%lld) does not match the problem (Mb=%lld, nbr=%lld, nbc=%lld)", fn,
                (long long)idx->Mb, (long long)idx->nbr, (long long)idx->nbc, (long long)Mb, (long long)nbr, (long long)nbc);
  if (mode == BBM_MODE_AUTO)
    mode = (idx->row_ptr && idx->col_idx && idx->sched) ? BBM_MODE_LIST
           : (idx->bin_blk_mat && idx->offset && idx->total_ones && idx->nz_lo && idx->nz_hi) ? BBM_MODE_RUNS
                                                                                              : BBM_MODE_BITMAP;
  switch (mode) {
    case BBM_MODE_BITMAP:
      if (!idx->bin_blk_mat) return fail(BBM_EINVAL, "%s: BITMAP mode needs idx->bin_blk_mat", fn);
      break;
    case BBM_MODE_RUNS:
      if (!idx->bin_blk_mat || !idx->offset || !idx->total_ones || !idx->nz_lo || !idx->nz_hi)
        return fail(BBM_EINVAL, "%s: RUNS mode needs bin_blk_mat, offset, total_ones, nz_lo, nz_hi", fn);
      break;
    case BBM_MODE_LIST:
      if (!idx->row_ptr || !idx->col_idx || !idx->sched)
        return fail(BBM_EINVAL, "%s: LIST mode needs row_ptr, col_idx and sched", fn);
      break;
    case BBM_MODE_DENSE_BASELINE:
      // empty blocks have no packed words in memory: the kernel takes their zeros from the class bytes
      if (!idx->bin_blk_mat && !idx->blk_class) return fail(BBM_EINVAL, "%s: DENSE_BASELINE mode needs idx->bin_blk_mat or idx->blk_class", fn);
      break;
    default:
      return fail(BBM_EINVAL, "%s: unknown mode %d", fn, mode);
  }
  if (nbr * nbc >= (1ll << 31) || B * H * nbr >= (1ll << 31) || N >= (1ll << 31) || Nk >= (1ll << 31))
    return fail(BBM_EUNSUPPORTED, "%s: problem too large for 32-bit tile counters", fn);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (use_static) {
    workspace = nullptr;
    workspace_bytes = 0;
    if (mode == BBM_MODE_LIST || (mode != BBM_MODE_DENSE_BASELINE && split_parts(B * H * nbr, nbr, nbc, d, mode == BBM_MODE_LIST, N == Nk) > 1)) {
      // the counters and at least one partial result per (batch, head) must fit; what else fits decides whether cut
      // rows and small launches are computed in parts (see launch())
      const size_t floor_bytes = queue_bytes(Mb, nbr, Mb == 1 ? B * H : H) + record_bytes(d, idx->Br);
      if (floor_bytes > kStaticScratchBytes)
        return fail(BBM_EWORKSPACE, "%s: B*H*ceil(Nq/Br) = %lld block rows need %zu bytes of counters, beyond the static scratch of %zu bytes; "
                    "use bbm_attn_fwd_rect with a workspace", fn, (long long)(B * H * nbr), floor_bytes, kStaticScratchBytes);
      if (int rc = static_scratch_address(fn, &workspace)) return rc;
      workspace_bytes = kStaticScratchBytes;
      const int n_counters = (int)(8 + B * H * nbr);
      clear_counters_kernel<<<(unsigned)((n_counters + 255) / 256), 256, 0, s>>>(static_cast<int32_t*>(workspace), n_counters);
      if (int rc = launch_status(fn)) return rc;
    }
  } else {
    // LIST mode cannot do without its workspace; BITMAP and RUNS use one, if given, to compute a small launch in parts.  What
    // the parts of BITMAP and RUNS need (at most eight of a row) will do for LIST as well: launch() takes as many as find room.
    size_t need = 0;
    if (mode == BBM_MODE_LIST) {
      need = bbm_attn_fwd_workspace_bytes(B, H, N, d, idx->Br, idx->Bc, BBM_MODE_BITMAP);
      if (need == 0) need = bbm_attn_fwd_workspace_bytes(B, H, N, d, idx->Br, idx->Bc, mode);
    }
    if (need > 0 && (!workspace || workspace_bytes < need))
      return fail(BBM_EWORKSPACE, "%s: workspace of %zu bytes needed, %zu given", fn, need, workspace ? workspace_bytes : (size_t)0);
    if (need > 0 && !aligned(workspace, 16)) return fail(BBM_EINVAL, "%s: workspace must be 16-byte aligned", fn);
  }

  AttnParams P;
  P.q = static_cast<const __bf16*>(q);
  P.k = static_cast<const __bf16*>(k);
  P.v = static_cast<const __bf16*>(v);
  P.o = static_cast<__bf16*>(o);
  P.lse = lse;
  P.packed = packed_mask;
  P.bin_blk_mat = idx->bin_blk_mat ? idx->bin_blk_mat : idx->blk_class;  // either is zero exactly on empty blocks
  P.offset = idx->offset;
  P.total_ones = idx->total_ones;
  P.nz_lo = idx->nz_lo;
  P.nz_hi = idx->nz_hi;
  P.row_ptr = idx->row_ptr;
  P.col_idx = idx->col_idx;
  P.N = N;
  P.Nk = Nk;
  P.H = (int32_t)H;
  P.Mb = (int32_t)Mb;
  P.nbr = (int32_t)nbr;
  P.nbc = (int32_t)nbc;
  P.W = (int32_t)ceil_div(Nk, 64);
  P.total_wgs = (int32_t)(B * H * nbr);
  P.mode = mode;
  // scales up to the usual 1/sqrt(d) fold into the bf16 Q; sharper ones keep the non-power-of-two part in fp32
  const float c = softmax_scale * kLog2e;
  const bool exact = softmax_scale * sqrtf((float)d) > 1.0f + 1.0f / 1024.0f;
  int c_exp = 0;
  (void)frexpf(c, &c_exp);                       // c = f * 2^c_exp, f in [0.5, 1)
  P.qscale = exact ? ldexpf(1.0f, c_exp - 1) : c;
  P.rmul = exact ? c / P.qscale : 1.0f;         // in [1, 2)
  P.sched = idx->sched;
  P.queue = nullptr;
  P.partials = nullptr;
  P.hbp = (int32_t)(Mb == 1 ? B * H : H);
  P.n_extra = 0;
  P.split = 1;
  P.part_cap = 0;
  P.G = interleaved_planes(B * H, 2 * Nk * d * (int64_t)sizeof(__bf16));
  auto go = [&](auto ex) {
    constexpr bool EX = decltype(ex)::value != 0;
    if (d == 64) {
      if (idx->Br == 64) return launch<64, 2, EX>(P, Mb, workspace, workspace_bytes, s);
      if (idx->Br == 128) return launch<64, 4, EX>(P, Mb, workspace, workspace_bytes, s);
      return launch<64, 8, EX>(P, Mb, workspace, workspace_bytes, s);
    }
    if (idx->Br == 64) return launch<128, 2, EX>(P, Mb, workspace, workspace_bytes, s);
    if (idx->Br == 128) return launch<128, 4, EX>(P, Mb, workspace, workspace_bytes, s);
    return launch<128, 8, EX>(P, Mb, workspace, workspace_bytes, s);
  };
  return exact ? go(IntC<1>{}) : go(IntC<0>{});
}
}  // namespace

extern "C" __attribute__((visibility("default"))) int bbm_attn_fwd(const void* q, const void* k, const void* v, void* o, float* lse, int64_t B, int64_t H,
                            int64_t N, int d, float softmax_scale, int64_t Mb, const uint64_t* packed_mask,
                            const bbm_index* idx, int mode, void* workspace, size_t workspace_bytes, void* stream) {
  return attn_fwd_impl("bbm_attn_fwd", q, k, v, o, lse, B, H, N, N, d, softmax_scale, Mb, packed_mask, idx, mode, workspace, workspace_bytes, stream, false);
}

extern "C" __attribute__((visibility("default"))) int bbm_attn_fwd_rect(const void* q, const void* k, const void* v, void* o, float* lse, int64_t B,
                                 int64_t H, int64_t Nq, int64_t Nk, int d, float softmax_scale, int64_t Mb,
                                 const uint64_t* packed_mask, const bbm_index* idx, int mode, void* workspace,
                                 size_t workspace_bytes, void* stream) {
  return attn_fwd_impl("bbm_attn_fwd_rect", q, k, v, o, lse, B, H, Nq, Nk, d, softmax_scale, Mb, packed_mask, idx, mode, workspace, workspace_bytes,
                       stream, false);
}

extern "C" __attribute__((visibility("default"))) int bbm_attn_fwd_static(const void* q, const void* k, const void* v, void* o, float* lse, int64_t B,
                                   int64_t H, int64_t Nq, int64_t Nk, int d, float softmax_scale, int64_t Mb,
                                   const uint64_t* packed_mask, const bbm_index* idx, int mode, void* stream) {
  return attn_fwd_impl("bbm_attn_fwd_static", q, k, v, o, lse, B, H, Nq, Nk, d, softmax_scale, Mb, packed_mask, idx, mode, nullptr, 0, stream, true);
}
