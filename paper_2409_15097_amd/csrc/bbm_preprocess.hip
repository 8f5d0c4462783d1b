// Stage 1a: mask bytes -> block classes, BinBlkMat and packed mask bits (paper Sec. 4 "Binary Block
// Masking"; Appendix A, block-based summation).  The sum of a block is only ever compared with 0 and with
// Br*Bc, so the kernel carries an OR and an AND of the non-zero bits instead of a count.
//
// One work-group (8 wavefronts) owns one block row (Br mask rows) x 16*LPR mask columns.  LPR lanes of a wavefront read
// one row segment, 16 B each, so a load instruction of a wavefront covers 64 / LPR rows, with U of them in flight; each lane
// turns its 16 bytes into 16 bits and keeps a running OR / AND over the rows it sees.  The bits go to LDS as uint16
// quarters of the 64-bit words and leave word-column major, so the global writes of the packed mask are contiguous too.
#include "bbm_internal.h"
#include "bbm_line_index.h"
#include "bbm_mask_index.h"

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kMaxBr = 256;
constexpr int64_t kStreamFromBytes = 128ll << 20;
constexpr int64_t kWideFromBytes = 8ll << 20;

// 4 mask bytes -> 4 bits (bit t = byte t non-zero).
__device__ __forceinline__ uint32_t nz_nibble(uint32_t x) {
  uint32_t y = (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;  // bit 7 of each byte = byte != 0
  return (((y >> 7) * 0x00204081u) >> 21) & 0xfu;                      // gather bits 0,8,16,24 -> 0..3
}

// 16 mask bytes at any byte address: gfx950 loads 16 bytes from unaligned addresses in one instruction.
// STREAM: a streaming (non-temporal) load.  A mask is read once and never again; one that is larger than the last-level
// cache can hold anyway would only push Q, K and V out of it on its way through.
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
template <bool STREAM>
__device__ __forceinline__ u32x4_any load16(const uint8_t* p) {
  const u32x4_any* q = reinterpret_cast<const u32x4_any*>(p);
  return STREAM ? __builtin_nontemporal_load(q) : *q;
}
__device__ __forceinline__ uint32_t bits16(u32x4_any x) {
  return nz_nibble(x.x) | (nz_nibble(x.y) << 4) | (nz_nibble(x.z) << 8) | (nz_nibble(x.w) << 12);
}

// INDEX: the work-group that finishes last also writes the index of the block rows, a wave each, from the class bytes in LDS.  Nobody
// waits: the others have ended.  Classes are written through and read around the XCDs' caches and counted without a fence (a
// device-wide release makes an XCD's cache write back all it holds).  What it saves is a launch, most of it on the host: both
// stages of 256 x 256 take 16.3 -> 13.5 us of a step of 256 tokens that is submitted call by call, 61.0 -> 60.0 of a decoding step of
// 256 x 1280 (replayed from a graph 6.6 -> 6.2 and 6.9 -> 6.4, which is not taken: see `recorded`).  The last work-group works alone,
// so one pass over its waves is the limit: 10 block rows of 1280 146.0 -> 147.1 of a step; with the block columns 6.8 -> 7.8, 7.1 -> 9.9.
constexpr int kFusedBytes = 4096, kFusedRows = kWaves, kAgentScope = 16;  // sc1
struct FusedIndex {
  bbm::LineArgs rows;
  int32_t* arrivals;  // work-groups that have ended; zero between calls
};
__device__ __forceinline__ __amdgpu_buffer_rsrc_t class_rsrc(const uint8_t* blk_class, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(blk_class), 0, (int)bytes, 0x00027000);
}

template <int LPR, int U, bool STREAM, bool INDEX = false>
__global__ __launch_bounds__(kThreads) void block_reduce_kernel(const uint8_t* __restrict__ mask, int64_t Nr, int64_t N,
                                                                int64_t row_stride, int Br, int Bc, int64_t nbr,
                                                                int64_t nbc, uint8_t* __restrict__ blk_class,
                                                                uint8_t* __restrict__ bin_blk_mat,
                                                                uint64_t* __restrict__ packed, const FusedIndex fused) {
  constexpr int kCols = 16 * LPR;              // mask columns of a work-group
  constexpr int kWords = LPR / 4;              // 64-bit words of a row
  constexpr int kRowsPerLoad = kWaves * 64 / LPR;  // rows the work-group's wavefronts read with one load each
  constexpr int kBatchRows = U * kRowsPerLoad;     // rows of a batch: every lane has U independent loads in flight
  __shared__ __attribute__((aligned(8))) uint16_t stage[kWords * (kMaxBr + 1) * 4];  // [word][row in block (+1 pad)][quarter]
  __shared__ uint32_t acc[kWaves][LPR];        // per wave and 16-column chunk: any16 | all16 << 16
  __shared__ uint32_t word_any[kWords];        // per 64-column word: does any of the block row's rows set a bit?

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int chunk = lane % LPR, sub = lane / LPR;
  const int64_t c0 = (int64_t)blockIdx.x * kCols;
  const int64_t i = blockIdx.y, m = blockIdx.z;
  const int64_t r0 = i * Br;
  const int rows = (int)((r0 + Br <= Nr) ? Br : (Nr - r0));  // real (unpadded) rows of this block row (Nr mask rows, N columns)
  const int64_t col = c0 + 16 * chunk;
  const uint8_t* base = mask + (m * Nr + r0) * row_stride;
  const int BrP = Br + 1;  // padded row count: consecutive words land in different LDS banks

  // The chunk that reaches past column N is read as the row's last 16 bytes and shifted down, so nothing outside a row is
  // touched and every lane runs the same instructions; chunks wholly past N shift everything out (zero: never full).
  const int64_t at = col + 16 <= N ? col : (N >= 16 ? N - 16 : 0);
  const int shift = (int)(col - at < 31 ? col - at : 31);
  uint32_t any16 = 0, all16 = 0xffffu;
  uint16_t* const s = stage + ((chunk >> 2) * BrP) * 4 + (chunk & 3);
  // rows past the last are clamped to it: the same bits once more, neutral in OR and AND (the dispatch takes a batch no
  // longer than the block, or loads that all repeat the last row would be most of them)
  auto take = [&](int r, uint32_t b) {
    any16 |= b;
    all16 &= b;
    if (packed) s[r * 4] = (uint16_t)b;
  };
  if (N >= 16) {
    for (int rb = wave * (64 / LPR) + sub; rb - sub < rows; rb += kBatchRows) {
      u32x4_any x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = load16<STREAM>(base + (int64_t)min(rb + u * kRowsPerLoad, rows - 1) * row_stride + at);
#pragma unroll
      for (int u = 0; u < U; ++u) take(min(rb + u * kRowsPerLoad, rows - 1), bits16(x[u]) >> shift);
    }
  } else {  // masks of fewer than 16 columns: byte by byte
    for (int r = wave * (64 / LPR) + sub; r < rows; r += kRowsPerLoad) {
      uint32_t b = 0;
      for (int t = 0; t < 16; ++t)
        if (col + t < N && base[(int64_t)r * row_stride + col + t] != 0) b |= 1u << t;
      take(r, b);
    }
  }
  // a lane that saw no row of this block keeps all16 = 0xffff: it is neutral in the AND below
  if (rows < Br) all16 = 0;  // block row reaches into the zero padding below the mask
#pragma unroll
  for (int d = LPR; d < 64; d <<= 1) {  // the rows that one wavefront reads side by side
    any16 |= __shfl_xor(any16, d);
    all16 &= __shfl_xor(all16, d);
  }
  if (lane < LPR) acc[wave][lane] = any16 | (all16 << 16);
  __syncthreads();

  if (wave == 0) {
    uint32_t any_v = 0, all_v = 0xffffu;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t a = acc[w][chunk];
      any_v |= a & 0xffffu;
      all_v &= a >> 16;
    }
    {  // four lanes of 16 columns make one packed word
      uint32_t w_any = any_v | __shfl_xor(any_v, 1);
      w_any |= __shfl_xor(w_any, 2);
      if (lane < LPR && (lane & 3) == 0) word_any[lane >> 2] = w_any;
    }
    const int g = Bc / 16;  // lanes per block column (at most LPR, see the dispatch)
    for (int d = 1; d < g; d <<= 1) {
      any_v |= __shfl_xor(any_v, d);
      all_v &= __shfl_xor(all_v, d);
    }
    const int64_t j = col / Bc;
    if (lane < LPR && (lane % g) == 0 && j < nbc) {
      const uint8_t cls = any_v == 0 ? BBM_BLOCK_EMPTY : (all_v == 0xffffu ? BBM_BLOCK_FULL : BBM_BLOCK_PARTIAL);
      const int64_t o = (m * nbr + i) * nbc + j;
      if constexpr (INDEX)
        __builtin_amdgcn_raw_buffer_store_b8(cls, class_rsrc(blk_class, (int64_t)gridDim.z * nbr * nbc), (int)o, 0, kAgentScope);
      else
        blk_class[o] = cls;
      if (bin_blk_mat) bin_blk_mat[o] = cls != BBM_BLOCK_EMPTY;
    }
  }

  if (packed) {
    // Words of a (block row x 64 columns) slab without a single set bit are not written: no schedule reads them (the
    // mask-everywhere baseline takes the zero from the class byte), and on sparse masks they are most of the output.
    __syncthreads();
    const int64_t W = (N + 63) / 64;
    const int64_t w0 = c0 / 64;
    const uint64_t* stage64 = reinterpret_cast<const uint64_t*>(stage);
    if constexpr (kBatchRows >= 64) {
      constexpr int kWavesPerWord = kWords < kWaves ? kWaves / kWords : 1;
      for (int wl = wave / kWavesPerWord; wl < kWords; wl += kWaves / kWavesPerWord) {
        if (w0 + wl >= W || word_any[wl] == 0) continue;
        uint64_t* const dst = packed + (m * W + w0 + wl) * Nr + r0;
        for (int rl = (wave % kWavesPerWord) * 64 + lane; rl < rows; rl += kWavesPerWord * 64) dst[rl] = stage64[wl * BrP + rl];
      }
    } else {  // blocks of one short batch: a wavefront writes several words' rows side by side
      const int wl = threadIdx.x / kBatchRows, rl = threadIdx.x % kBatchRows;
      if (wl < kWords && w0 + wl < W && rl < rows && word_any[wl] != 0) packed[(m * W + w0 + wl) * Nr + r0 + rl] = stage64[wl * BrP + rl];
    }
  }
  if constexpr (INDEX) {
    __shared__ int arrived_s;
    __shared__ int len_s[kFusedRows];
    static_assert(sizeof(stage) >= kFusedBytes, "the class bytes take the place of the packed words");
    if (wave == 0) {  // which wrote the classes
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      // (the last one's count puts it back to zero for the next call)
      if (lane == 0) arrived_s = (int)atomicInc(reinterpret_cast<unsigned*>(fused.arrivals), gridDim.x * gridDim.y * gridDim.z - 1);
    }
    __syncthreads();
    if (arrived_s != (int)(gridDim.x * gridDim.y * gridDim.z) - 1) return;
    const int Mb = gridDim.z, bytes = Mb * (int)(nbr * nbc);
    uint8_t* const cls_s = reinterpret_cast<uint8_t*>(stage);
    const __amdgpu_buffer_rsrc_t src = class_rsrc(blk_class, bytes);
    uint8_t c[kFusedBytes / kThreads];
#pragma unroll
    for (int t = 0; t < kFusedBytes / kThreads; ++t) c[t] = __builtin_amdgcn_raw_buffer_load_b8(src, t * kThreads + threadIdx.x, 0, kAgentScope);
#pragma unroll
    for (int t = 0; t < kFusedBytes / kThreads; ++t) cls_s[t * kThreads + threadIdx.x] = c[t];
    __syncthreads();
    const int line = wave;  // (plane, block row)
    auto own_block = [&](int base) { return base + lane < (int)nbc ? cls_s[line * (int)nbc + base + lane] : (uint8_t)0; };
    if (line < Mb * (int)nbr) {
      int n = 0;
      for (int base = 0; base < (int)nbc; base += 64) n += __popcll(__ballot(own_block(base) != 0));
      if (lane == 0) len_s[line] = n;
    }
    __syncthreads();
    if (line < Mb * (int)nbr)
      bbm::emit_line<false, bbm::kLineNormal>(own_block, own_block(0), len_s, nullptr, line, 0, 1, 0, (int)nbc, Mb, (int)nbr, (int)nbc, fused.rows);
  }
}

}  // namespace

namespace {
template <int V>
struct IntC {
  static constexpr int value = V;
};

int build_block_mask_impl(const char* fn, const uint8_t* mask, int64_t Mb, int64_t Nq, int64_t Nk, int64_t row_stride_bytes, int Br, int Bc,
                          uint8_t* blk_class, uint8_t* bin_blk_mat, uint64_t* packed_mask, void* stream, FusedIndex* fused = nullptr) {
  using namespace bbm;
  clear_error();
  if (!mask || !blk_class) return fail(BBM_EINVAL, "%s: mask and blk_class must not be NULL", fn);
  if (Mb < 1 || Nq < 1 || Nk < 1)
    return fail(BBM_EINVAL, "%s: Mb=%lld, rows=%lld, columns=%lld must be >= 1", fn, (long long)Mb, (long long)Nq, (long long)Nk);
  if (row_stride_bytes < Nk) return fail(BBM_EINVAL, "%s: row_stride_bytes=%lld < columns=%lld", fn, (long long)row_stride_bytes, (long long)Nk);
  if (Br < 1 || Br > kMaxBr) return fail(BBM_EUNSUPPORTED, "%s: Br=%d outside [1, %d]", fn, Br, kMaxBr);
  if (Bc != 16 && Bc != 32 && Bc != 64 && Bc != 128 && Bc != 256) return fail(BBM_EUNSUPPORTED, "%s: Bc=%d not in {16,32,64,128,256}", fn, Bc);
  if (packed_mask && !aligned(packed_mask, 8)) return fail(BBM_EINVAL, "%s: packed_mask must be 8-byte aligned", fn);
  const int64_t nbr = ceil_div(Nq, Br), nbc = ceil_div(Nk, Bc);
  if (nbr > 65535 || Mb > 65535) return fail(BBM_EUNSUPPORTED, "%s: nbr=%lld or Mb=%lld exceeds 65535", fn, (long long)nbr, (long long)Mb);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t bytes = Mb * Nq * Nk;
  // masks from kStreamFromBytes on (half the 256 MB last-level cache) are streamed: block reduction 6 % faster on a 1 GiB mask
  // and the attention kernel behind it finds more of Q, K, V still cached (whole step -2.5 % at 1 GiB, -3.5 % at 256 MiB);
  // a 64 MiB mask that is rebuilt from the cache it still sits in loses 20 % that way
  const bool streamed = bytes >= kStreamFromBytes;
  // A recorded call does without the counter: its replays may run beside other calls, whose work-groups would be counted with theirs.
  auto recorded = [&]() {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing(s, &status) == hipSuccess;
    if (!known) (void)hipGetLastError();  // (what is wrong with the stream is for the launches to say)
    return !known || status != hipStreamCaptureStatusNone;
  };
  const bool with_index = fused && fused->arrivals && !streamed && Mb * nbr * nbc <= kFusedBytes && Mb * nbr <= kFusedRows && !recorded();
  bool index_written = false;
  auto go = [&](auto lpr, auto unroll) {
    constexpr int LPR = decltype(lpr)::value, U = decltype(unroll)::value;
    if constexpr (LPR == 16) {
      if (with_index) {
        block_reduce_kernel<LPR, U, false, true><<<dim3((unsigned)ceil_div(Nk, 16 * LPR), (unsigned)nbr, (unsigned)Mb), kThreads, 0, s>>>(
            mask, Nq, Nk, row_stride_bytes, Br, Bc, nbr, nbc, blk_class, bin_blk_mat, packed_mask, *fused);
        index_written = true;
        return;
      }
    }
    const auto kernel = streamed ? block_reduce_kernel<LPR, U, true> : block_reduce_kernel<LPR, U, false>;
    kernel<<<dim3((unsigned)ceil_div(Nk, 16 * LPR), (unsigned)nbr, (unsigned)Mb), kThreads, 0, s>>>(
        mask, Nq, Nk, row_stride_bytes, Br, Bc, nbr, nbc, blk_class, bin_blk_mat, packed_mask, FusedIndex{});
  };
  // What a work-group reads is Br rows x 16*LPR bytes.  Blocks of more than 64 rows: 256-byte segments (LPR = 16) give the most
  // work-groups and the shortest chain of loads; rows that do not start on 128-byte lines cost one line more per segment, so
  // from kWideFromBytes on those are read in 512-byte segments.  Lower blocks take longer segments, or starting work-groups
  // costs more than the reading, and a batch of loads that is no longer than the block.
  // Microseconds with LPR = 16 / 32 (in a graph, rotating over 3 masks), Br = 128: 256 x 1280 3.5 / 4.0, 2048^2 x 2 3.9 / 4.3,
  // 16384^2 53.4 / 53.3; unaligned 2001^2 4.0 / 4.7, 3000^2 5.5 / 4.6, 9001^2 21.2 / 18.6.
  // 16384^2 by height, this rule / batches of 128 rows x 256 bytes for every height: 8 rows 75 / 330, 16 rows 51 / 179, 32 rows
  // 48 / 115, 64 rows 49 / 66 (60 with batches of 64 x 256); 256 x 1280 3.1-3.4 / 3.5-3.6.
  const bool line_rows = aligned(mask, 128) && row_stride_bytes % 128 == 0;
  if (Br <= 8) go(IntC<64>{}, IntC<1>{});
  else if (Br <= 16) go(IntC<64>{}, IntC<2>{});
  else if (Br <= 32) go(IntC<64>{}, IntC<4>{});
  else if (Br <= 64) bytes > kWideFromBytes ? go(IntC<32>{}, IntC<4>{}) : go(IntC<16>{}, IntC<2>{});
  else bytes > kWideFromBytes && !line_rows ? go(IntC<32>{}, IntC<8>{}) : go(IntC<16>{}, IntC<4>{});
  if (fused && !index_written) fused->arrivals = nullptr;  // the index is left to launches of its own
  return launch_status(fn);
}
}  // namespace

extern "C" __attribute__((visibility("default"))) int bbm_build_block_mask(const uint8_t* mask, int64_t Mb, int64_t N, int64_t row_stride_bytes, int Br,
                                    int Bc, uint8_t* blk_class, uint8_t* bin_blk_mat, uint64_t* packed_mask,
                                    void* stream) {
  return build_block_mask_impl("bbm_build_block_mask", mask, Mb, N, N, row_stride_bytes, Br, Bc, blk_class, bin_blk_mat, packed_mask, stream);
}

extern "C" __attribute__((visibility("default"))) int bbm_build_block_mask_rect(const uint8_t* mask, int64_t Mb, int64_t Nq, int64_t Nk,
                                         int64_t row_stride_bytes, int Br, int Bc, uint8_t* blk_class,
                                         uint8_t* bin_blk_mat, uint64_t* packed_mask, void* stream) {
  return build_block_mask_impl("bbm_build_block_mask_rect", mask, Mb, Nq, Nk, row_stride_bytes, Br, Bc, blk_class, bin_blk_mat, packed_mask, stream);
}

extern "C" __attribute__((visibility("default"))) int bbm_build_mask_index(
    const uint8_t* mask, int64_t Mb, int64_t Nq, int64_t Nk, int64_t row_stride_bytes, int Br, int Bc, uint8_t* blk_class, uint8_t* bin_blk_mat,
    uint64_t* packed_mask, int32_t* offset, int32_t* total_ones, int32_t* nz_lo, int32_t* nz_hi, int32_t* nz_cnt, int32_t* row_ptr,
    uint32_t* col_idx, int32_t* sched, int32_t* col_ptr, uint32_t* row_idx, int32_t* col_sched, int32_t* arrivals, void* stream) {
  using namespace bbm;
  clear_error();
  const char* const fn = "bbm_build_mask_index";
  const bool columns = col_ptr || row_idx || col_sched;
  const LineArgs cols{col_ptr, row_idx, col_sched};
  FusedIndex fused{{row_ptr, col_idx, sched, offset, total_ones, nz_lo, nz_hi, nz_cnt}, columns ? nullptr : arrivals};
  if (Nq >= 1 && Nk >= 1 && Br >= 1 && Bc >= 1) {  // (otherwise the block reduction's own checks fail)
    const int64_t nbr = ceil_div(Nq, Br), nbc = ceil_div(Nk, Bc);
    int rc = check_index_args(fn, blk_class, Mb, nbr, nbc, fused.rows);
    if (rc == BBM_OK && columns) rc = check_col_index_args(fn, blk_class, Mb, nbr, nbc, cols);
    if (rc != BBM_OK) return rc;
  }
  if (arrivals && !aligned(arrivals, 4)) return fail(BBM_EINVAL, "%s: arrivals must be 4-byte aligned", fn);
  int rc = build_block_mask_impl(fn, mask, Mb, Nq, Nk, row_stride_bytes, Br, Bc, blk_class, bin_blk_mat, packed_mask, stream, &fused);
  if (rc != BBM_OK || fused.arrivals) return rc;
  const int64_t nbr = ceil_div(Nq, Br), nbc = ceil_div(Nk, Bc);
  if (columns && launch_rows_and_columns(blk_class, Mb, nbr, nbc, fused.rows, cols, static_cast<hipStream_t>(stream))) return launch_status(fn);
  rc = bbm_build_index(blk_class, Mb, nbr, nbc, offset, total_ones, nz_lo, nz_hi, nz_cnt, row_ptr, col_idx, sched, stream);
  if (rc != BBM_OK || !columns) return rc;
  return bbm_build_col_index(blk_class, Mb, nbr, nbc, col_ptr, row_idx, col_sched, stream);
}
