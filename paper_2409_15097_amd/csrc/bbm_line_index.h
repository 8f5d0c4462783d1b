// The whole index of a class matrix of ordinary size in one launch: per line (block row, or block column for the
// backward pass) the ascending list of its non-zero blocks, the schedule and, for block rows, the run index.
#pragma once
#include "bbm_internal.h"

namespace bbm {
namespace {

__device__ __forceinline__ int ctz64(uint64_t x) { return x ? __builtin_ctzll(x) : 64; }

// Longest run of FULL blocks of one block row (leftmost on ties) and the span of its non-zero blocks, fed 64 block
// columns at a time in ascending order (bit t of `full` / `nz` = block column base + t).
struct RunScan {
  int best_len = 0, best_start = 0;  // longest finished run so far
  int cur_len = 0, cur_start = 0;    // run that touches the end of the previous chunk (0 = none)
  int lo = 0, hi = 0, cnt = 0;
  __device__ __forceinline__ void feed(uint64_t full, uint64_t nz, int base) {
    if (nz) {
      if (cnt == 0) lo = base + ctz64(nz);
      hi = base + 64 - __builtin_clzll(nz);
      cnt += __popcll(nz);
    }
    if (cur_len > 0) {  // continue the run that reached the chunk boundary
      const int ones = ctz64(~full);
      cur_len += ones;
      if (ones == 64) return;
      if (cur_len > best_len) { best_len = cur_len; best_start = cur_start; }
      cur_len = 0;
      full &= ~((1ull << ones) - 1ull);
    }
    while (full) {
      const int s = ctz64(full);
      const int ones = ctz64(~(full >> s));  // full >> s has zeros shifted in, so ones <= 64 - s
      if (s + ones == 64) {                  // run reaches the chunk end: decide when it ends
        cur_start = base + s;
        cur_len = ones;
        return;
      }
      if (ones > best_len) { best_len = ones; best_start = base + s; }
      full &= ~(((1ull << ones) - 1ull) << s);
    }
  }
  __device__ __forceinline__ void finish() {
    if (cur_len > best_len) { best_len = cur_len; best_start = cur_start; }
  }
};

// Exclusive prefix sum over the 64 lanes with data-parallel-primitive moves (register to register; a shuffle goes
// through LDS): shifts by 1, 2, 4, 8 inside each row of 16 lanes (a lane without a source adds 0), then lane 15 of a
// row added to the next row (rows 1 and 3), then lane 31 to rows 2 and 3.
__device__ __forceinline__ int wave_excl_scan(int x) {
  int incl = x;
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xf, 0xf, false);  // row_shr:1
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xf, 0xf, false);  // row_shr:2
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xf, 0xf, false);  // row_shr:4
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xf, 0xf, false);  // row_shr:8
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  incl += __builtin_amdgcn_update_dpp(0, incl, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return incl - x;
}

// Sum over the 64 lanes, returned in every lane.
__device__ __forceinline__ int wave_sum(int x) { return __builtin_amdgcn_readlane(wave_excl_scan(x) + x, 63); }

// Rows per launch-order group: neighbouring rows are kept together only while rows are short (split threshold at its
// floor, i.e. mean list length <= 16); with long rows the plain longest-first order balances the tail better.
__device__ __forceinline__ int launch_group_rows(int T) { return T == kSchedMinSplit ? kSchedGroupRows : 1; }

// Largest of 64 non-negative values, returned in every lane.
__device__ __forceinline__ int wave_max(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}

// RunScan with a lane per block column: the lane at which a run starts measures it, so a chunk costs a dozen
// instructions however many runs it has.
struct WaveRunScan {
  int best_len = 0, best_start = 0;  // per lane: longest run that started and ended in a chunk at this lane
  int cur_len = 0, cur_start = 0;    // uniform: run that touches the end of the previous chunk (0 = none)
  int car_len = 0, car_start = 0;    // uniform: longest finished run that crossed a chunk boundary
  int lo = 0, hi = 0, cnt = 0;       // uniform
  __device__ __forceinline__ void feed(uint64_t full, uint64_t nz, int base, int lane) {
    if (nz) {
      if (cnt == 0) lo = base + ctz64(nz);
      hi = base + 64 - __builtin_clzll(nz);
      cnt += __popcll(nz);
    }
    uint64_t inner = full;
    if (cur_len > 0) {  // continue the run that reached the chunk boundary
      const int ones = ctz64(~full);
      cur_len += ones;
      if (ones == 64) return;
      if (cur_len > car_len) { car_len = cur_len; car_start = cur_start; }
      cur_len = 0;
      inner &= ~((1ull << ones) - 1ull);
    }
    const int tail = full == ~0ull ? 64 : __builtin_clzll(~full);  // ones at the chunk's end
    if (tail > 0) {                                                // decided when that run ends
      cur_len = tail;
      cur_start = base + 64 - tail;
      inner = tail == 64 ? 0ull : inner & ((1ull << (64 - tail)) - 1ull);
    }
    const bool starts = ((inner & ~(inner << 1)) >> lane) & 1ull;
    const int ones = ctz64(~(inner >> lane));
    if (starts && ones > best_len) { best_len = ones; best_start = base + lane; }
  }
  // longest run, leftmost on ties, uniform
  __device__ __forceinline__ void finish(int& len, int& start) {
    if (cur_len > car_len) { car_len = cur_len; car_start = cur_start; }
    len = max(wave_max(best_len), car_len);
    const int none = 0x7fffffff;
    int s = none - wave_max(best_len == len ? none - best_start : 0);
    if (car_len == len) s = min(s, car_start);
    start = len > 0 ? s : 0;
  }
};

typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(1)));

// Bytes that are not zero: 4 bytes -> 0x01 in each such byte.
__device__ __forceinline__ uint32_t nz_bytes(uint32_t w) { return ((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) >> 7) & 0x01010101u; }

// 4 class bytes -> 4 bits, 16 -> 16 (bit t = byte t not zero).
__device__ __forceinline__ uint32_t nz_bits4(uint32_t w) { return ((nz_bytes(w) * 0x10204080u) >> 28) & 0xfu; }
__device__ __forceinline__ uint32_t nz_bits16(u32x4_any x) { return nz_bits4(x.x) | (nz_bits4(x.y) << 4) | (nz_bits4(x.z) << 8) | (nz_bits4(x.w) << 12); }

// What bounds an index build is latency: kernel starts, memory round trips and serial chains over a few kilobytes.  So
// nothing is handed from one work-group to another: every work-group counts the non-zero blocks of ALL lines itself
// (16 class bytes per load) into LDS, behind one barrier, and each of its waves then produces one line from those
// counts: the line's place in its plane, the split threshold, the parts and cut lines before its own and its rank are
// sums over the counts, spread over the lanes.  One launch; the redundant reads are class bytes x work-groups out of L2.
// Microseconds a call in a graph (bench.py --stages), several launches before -> now, block rows / block columns of 0.3 density:
// 2 x 4 7.8 -> 3.9 / 5.7 -> 3.1; 2 x 260 13 -> 5.5 / 19 -> 4.7; 4 planes of 32 x 64 9.7 -> 4.9 / 11.7 -> 4.7; 128 x 256 10.7 -> 6.2 /
// 16 -> 6.0; 256 x 512 16 -> 11.4 / 39 -> 8.4.  The limits, one launch / several: rows of 300 x 450 blocks 13.1 / 15.4, 512 x 512
// 16.6 / 17.5, 1024 x 160 16.0 / 15.0, 600 x 700 31 / 21, 3 planes of 330 x 300 24.5 / 15.4, 8 of 128 x 256 14.9 / 13.8 (one plane would
// gain up to 256 KiB, several lose from 128 on); columns of 512 x 512 11.4 / 24.9, 8 planes of 181 x 181 14.7 / 13.9.
constexpr int kLineWaves = 8;
constexpr int64_t kLineMaxLines = 4096, kLineMaxBytesRows = 128 << 10, kLineMaxBytesCols = 256 << 10;  // beyond: the multi-launch paths

inline bool line_index_fits(bool cols, int64_t Mb, int64_t nbr, int64_t nbc) {
  return Mb * (cols ? nbc : nbr) <= kLineMaxLines && Mb * nbr * nbc <= (cols ? kLineMaxBytesCols : kLineMaxBytesRows);
}

// COLS = false: lines are block rows (`ptr` = row_ptr, `list` = col_idx); true: block columns (col_ptr, row_idx).
// KIND: kLineShort: class rows of fewer than 16 blocks, which are counted another way.  kLineLong: block rows of kLineLongFrom
// blocks and more whose run index is not asked for: a wave takes a strip of kLineStrip blocks of a row instead of the
// whole row, and the counts are kept by strip (one wave per row: 1 x 16384 blocks 58 us, 2 x 8192 32, 1 x 2000 10.1,
// 1 x 1024 6.9; strips: 7.0, 6.8, 6.4, 6.0).  With a run index a row is walked by one wave, which finds it on the way.
// `sched` and the five arrays of the run index (block rows only) may be NULL.
enum { kLineNormal = 0, kLineShort = 1, kLineLong = 2 };
constexpr int kLineLongFrom = 1024, kLineStrip = 512;
constexpr int kLineMaxStrips = (int)(kLineMaxBytesRows / kLineStrip + kLineMaxBytesRows / kLineLongFrom);  // whole strips + a partial one a row
using LineOut = LineArgs;

// One line, by a wave, from the counts len_s of all lines (strip_s: of all strips); own_block(base): this lane's block of the 64
// from `base` on, `next` the first of them.
template <bool COLS, int KIND, typename Block>
__device__ __forceinline__ void emit_line(Block own_block, uint8_t next, const int* len_s, const int* strip_s, int line, int seg, int S,
                                          int first_block, int past_block, int Mb, int nbr, int nbc, const LineOut& o) {
  constexpr bool LONG = KIND == kLineLong;
  const int lane = threadIdx.x & 63;
  const int L = COLS ? nbc : nbr, nlines = Mb * L, m = line / L, i = line - m * L;
  int32_t *const ptr = o.ptr, *const sched = o.sched, *const offset = o.offset;
  // ---- this wave's line: its place in the plane's list, and the split threshold (a mean over all lines)
  const int* const cp = len_s + m * L;
  const int n = cp[i];
  int above = 0, total = 0, nonempty = 0;
  for (int b = lane; b < nlines; b += 64) {
    const int x = len_s[b];
    total += x;
    nonempty += x > 0 ? 1 : 0;
    above += b >= m * L && b < line ? x : 0;
  }
  const int start = wave_sum(above);
  total = wave_sum(total);
  nonempty = wave_sum(nonempty);
  const int mean = nonempty > 0 ? (total + nonempty - 1) / nonempty : 0;
  const int T = max(COLS ? kColSchedMinSplit : kSchedMinSplit, 2 * mean);
  if (lane == 0 && seg == 0) {
    ptr[(int64_t)m * (L + 1) + i] = start;
    if (i == L - 1) ptr[(int64_t)m * (L + 1) + L] = start + n;
  }

  // parts and cut lines: before this line (lines in (plane, line) order), and in all
  const int np = n > T ? (n + T - 1) / T : 0;
  const int chunk = np > 0 ? (n + np - 1) / np : 1;
  int32_t* parts = nullptr;
  if (sched && (np > 0 || line == 0)) {
    int q = 0, rho = 0, all_parts = 0, all_cut = 0;
    for (int b = lane; b < nlines; b += 64) {
      const int x = len_s[b];
      const int np_b = x > T ? (x + T - 1) / T : 0;
      all_parts += np_b;
      all_cut += np_b > 0 ? 1 : 0;
      q += b < line ? np_b : 0;
      rho += b < line && np_b > 0 ? 1 : 0;
    }
    q = wave_sum(q);
    rho = wave_sum(rho);
    if (line == 0 && seg == 0) {
      all_parts = wave_sum(all_parts);
      all_cut = wave_sum(all_cut);
      if (lane < kSchedPartBase)
        sched[lane] = lane == kSchedNParts ? all_parts : lane == kSchedSplitT ? T : lane == kSchedNCutRows ? all_cut : 0;
    }
    parts = sched + kSchedPartBase + (int64_t)kSchedPartInts * q;
    for (int k = lane; k < (seg == 0 ? np : 0); k += 64) {
      int32_t* rec = parts + kSchedPartInts * k;
      rec[0] = line;
      rec[1] = start + k * chunk;
      rec[2] = min(chunk, n - k * chunk);
      rec[3] = k;
      rec[4] = np;
      rec[5] = q;
      rec[6] = rho;
    }
  }

  // the list; the lane that writes the entry a part starts with also leaves it in the part's record
  uint32_t* const out = o.list + (int64_t)m * nbr * nbc + start;
  int written = 0, first = -1;
  if (LONG)
    for (int k = 0; k < seg; ++k) written += strip_s[line * S + k];
  WaveRunScan rs;
#pragma unroll 1  // short code: at this length of a launch, fetching instructions is a good part of it
  for (int base = first_block; base < past_block; base += 64) {
    const uint8_t c = next;
    next = own_block(base + 64);
    const uint64_t nz = __ballot(c != BBM_BLOCK_EMPTY);
    const uint64_t full = __ballot(c == BBM_BLOCK_FULL);
    if (!COLS && offset) rs.feed(full, nz, base, lane);
    if (written == 0 && nz != 0) {  // the line's first entry (this happens once: written > 0 from here on)
      const int bit = ctz64(nz);
      first = (int)((uint32_t)(base + bit) | (((full >> bit) & 1ull) ? 0x80000000u : 0u));
    }
    if (c != BBM_BLOCK_EMPTY) {
      const int pos = written + __popcll(nz & ((1ull << lane) - 1ull));
      const uint32_t entry = (uint32_t)(base + lane) | (c == BBM_BLOCK_FULL ? 0x80000000u : 0u);
      out[pos] = entry;
      if (np > 0 && sched && pos % chunk == 0 && pos / chunk < np) parts[kSchedPartInts * (pos / chunk) + 7] = (int32_t)entry;
    }
    written += __popcll(nz);
  }
  if (!COLS && offset) {
    int run_len, run_start;
    rs.finish(run_len, run_start);
    if (lane == 0) {
      offset[line] = run_start;
      o.total_ones[line] = run_len;
      o.nz_lo[line] = rs.lo;
      o.nz_hi[line] = rs.hi;
      o.nz_cnt[line] = rs.cnt;
    }
  }
  if (!sched || (LONG && first == -1 && (n > 0 || seg > 0))) return;  // the record is left to the wave that has the line's first entry

  // launch-order record: groups of gsz lines by their longest list, longest first (ties: the higher group first); inside
  // a group the longest line first (ties: the higher line first)
  const int gsz = COLS ? 1 : launch_group_rows(T);
  const int ng = (L + gsz - 1) / gsz, g = i / gsz;
  auto group_max = [&](int gg) {
    int t = 0;
    for (int j = gg * gsz; j < min(L, (gg + 1) * gsz); ++j) t = max(t, cp[j]);
    return t;
  };
  const int longest = group_max(g);
  int before = 0;
  for (int gg = lane; gg < ng; gg += 64) {
    const int t = group_max(gg);
    before += (t > longest || (t == longest && gg > g)) ? 1 : 0;
  }
  int rank = wave_sum(before) * gsz;
  const int last = ng - 1, last_lines = L - last * gsz;  // the last group may be short
  if (last != g && group_max(last) >= longest) rank -= gsz - last_lines;
  for (int j = g * gsz; j < min(L, (g + 1) * gsz); ++j) rank += (cp[j] > n || (cp[j] == n && j > i)) ? 1 : 0;
  if (lane == 0)
    reinterpret_cast<int4*>(sched + kSchedPartBase + (int64_t)kSchedPartInts * nlines)[(int64_t)m * L + rank] = make_int4(i, start, n, first);
}

template <bool COLS, int KIND>
__device__ __forceinline__ void line_index(const uint8_t* __restrict__ cls, int wg, int* len_s, int* strip_s, int Mb, int nbr, int nbc,
                                           const LineOut& out) {
  constexpr bool SHORT = KIND == kLineShort, LONG = KIND == kLineLong;
  static_assert(!(COLS && LONG), "strips are of block rows");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = COLS ? nbc : nbr, depth = COLS ? nbr : nbc;  // lines per plane, blocks per line
  const int nlines = Mb * L;
  const int S = LONG ? (depth + kLineStrip - 1) / kLineStrip : 1;  // strips of a line
  const int unit = wg * kLineWaves + wave;      // this wave's strip, or line (waves past the last only count)
  const int line = LONG ? unit / S : unit, seg = LONG ? unit - line * S : 0;
  const int own = min(line, nlines - 1);
  const int m = own / L, i = own - m * L;
  const int first_block = LONG ? seg * kLineStrip : 0, past_block = LONG ? min(depth, first_block + kLineStrip) : depth;
  const uint8_t* const mine = cls + (int64_t)m * nbr * nbc + (COLS ? i : (int64_t)i * nbc);
  const int step = COLS ? nbc : 1;                           // bytes from one block of the line to the next
  auto own_block = [&](int base) { return base + lane < past_block ? mine[(int64_t)(base + lane) * step] : (uint8_t)0; };
  uint8_t next = own_block(first_block);  // asked for before the counting

  // ---- non-zero blocks of every line
  const int C16 = (nbc + 15) / 16;  // 16-byte chunks of a class row; the last one is read as the row's last 16 bytes
  // SHORT: 16 bytes from a row's start on, the last rows' moved back to end with the matrix; as bits, that row's first.  (A load
  // per byte took 256 planes of 15 x 15 from 14.8 to 25 us, their columns from 17.5 to 46.)
  const int bytes = nlines * depth;  // at most kLineMaxBytesCols
  auto short_rows_at = [&](int r) { return min(r * nbc, bytes - 16); };
  auto short_rows_bits = [&](u32x4_any x, int r) { return nz_bits16(x) >> (r * nbc - short_rows_at(r)); };
  const uint32_t row_bits = SHORT ? (1u << nbc) - 1u : 0xffffu;
  if (SHORT && (bytes < 16 || (!COLS && nbc <= 4 && nlines <= kLineWaves * 64))) {  // next to nothing to count
    for (int b = tid; b < nlines; b += kLineWaves * 64) {
      const int bm = b / L, bi = b - bm * L;
      int cnt = 0;
#pragma unroll 1
      for (int t = 0; t < depth; ++t) cnt += cls[(int64_t)bm * nbr * nbc + (COLS ? t * nbc + bi : bi * nbc + t)] != 0 ? 1 : 0;
      len_s[b] = cnt;
    }
  } else if (!COLS && SHORT) {
    // rows a thread takes from one load: what 16 bytes hold, but no more than it needs to have one load
    const int per = min(16 / nbc, (nlines + kLineWaves * 64 - 1) / (kLineWaves * 64)), hop = kLineWaves * 64 * per;
    constexpr int kFly = 4;
    for (int r0 = tid * per; r0 < nlines; r0 += kFly * hop) {
      u32x4_any x[kFly];
#pragma unroll
      for (int f = 0; f < kFly; ++f) x[f] = *reinterpret_cast<const u32x4_any*>(cls + short_rows_at(min(r0 + f * hop, nlines - 1)));
#pragma unroll
      for (int f = 0; f < kFly; ++f) {
        const int r = r0 + f * hop, re = min(r + per, nlines);
        uint32_t b = r < nlines ? short_rows_bits(x[f], r) : 0;
#pragma unroll 1
        for (int k = r; k < re; ++k, b >>= nbc) len_s[k] = __popc(b & row_bits);
      }
    }
  } else if (LONG) {
    constexpr int kLanes = kLineStrip / 16, kFly = 4, kPer = 64 / kLanes;  // lanes of a strip, loads in flight, strips of a load
    for (int u0 = wave * kPer + lane / kLanes; u0 - lane / kLanes < nlines * S; u0 += kFly * kLineWaves * kPer) {
      int cnt[kFly];
#pragma unroll
      for (int f = 0; f < kFly; ++f) {
        const int u = min(u0 + f * kLineWaves * kPer, nlines * S - 1), r = u / S;
        const int c = (u - r * S) * kLineStrip + 16 * (lane % kLanes), at = min(c, nbc - 16);
        const u32x4_any x = *reinterpret_cast<const u32x4_any*>(cls + r * nbc + at);
        cnt[f] = c < nbc ? __popc(nz_bits16(x) >> (c - at)) : 0;
      }
#pragma unroll
      for (int d = 1; d < kLanes; d <<= 1) {
#pragma unroll
        for (int f = 0; f < kFly; ++f) cnt[f] += __shfl_xor(cnt[f], d);
      }
      if (lane % kLanes == 0) {
#pragma unroll
        for (int f = 0; f < kFly; ++f)
          if (u0 + f * kLineWaves * kPer < nlines * S) strip_s[u0 + f * kLineWaves * kPer] = cnt[f];
      }
    }
    __syncthreads();
    for (int b = tid; b < nlines; b += kLineWaves * 64) {
      int sum = 0;
      for (int k = 0; k < S; ++k) sum += strip_s[b * S + k];
      len_s[b] = sum;
    }
  } else if (!COLS) {
    int lpr = 1;  // lanes per row
    while (lpr < C16 && lpr < 64) lpr <<= 1;
    const int rpw = 64 / lpr, sub = lane / lpr, c_first = (lane & (lpr - 1)) * 16;
    constexpr int kFly = 4;  // rows a lane has in flight
    const int hop = kLineWaves * rpw;
    for (int r0 = wave * rpw + sub; r0 - sub < nlines; r0 += kFly * hop) {
      int cnt[kFly];
#pragma unroll
      for (int f = 0; f < kFly; ++f) cnt[f] = 0;
      for (int c = c_first; c < nbc; c += lpr * 16) {
        const int at = min(c, nbc - 16);
        // bit s of byte t counts byte 4s + t of the 16; those below c belong to the chunk before
        uint32_t keep = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int skip = min(max(c - at - 4 * s, 0), 4);
          keep |= (skip < 4 ? 0x01010101u << (8 * skip) : 0u) << s;
        }
        u32x4_any x[kFly];
#pragma unroll
        for (int f = 0; f < kFly; ++f) x[f] = *reinterpret_cast<const u32x4_any*>(cls + (int64_t)min(r0 + f * hop, nlines - 1) * nbc + at);
#pragma unroll
        for (int f = 0; f < kFly; ++f)
          cnt[f] += __popc((nz_bytes(x[f].x) | (nz_bytes(x[f].y) << 1) | (nz_bytes(x[f].z) << 2) | (nz_bytes(x[f].w) << 3)) & keep);
      }
      for (int d = 1; d < lpr; d <<= 1) {
#pragma unroll
        for (int f = 0; f < kFly; ++f) cnt[f] += __shfl_xor(cnt[f], d);
      }
      if ((lane & (lpr - 1)) == 0) {
#pragma unroll
        for (int f = 0; f < kFly; ++f)
          if (r0 + f * hop < nlines) len_s[r0 + f * hop] = cnt[f];
      }
    }
  } else {
    for (int b = tid; b < nlines; b += kLineWaves * 64) len_s[b] = 0;
    __syncthreads();
    // a thread adds up 16 columns over every RG-th row of a plane, in byte counters
    const int units = Mb * C16;
    const int RG = max(1, min(nbr, kLineWaves * 64 / units));
    for (int it = tid; it < units * RG; it += kLineWaves * 64) {
      const int u = it % units, rg = it / units;
      const int pm = u / C16, c = (u - pm * C16) * 16, at = SHORT ? 0 : min(c, nbc - 16);
      const uint8_t* const plane = cls + (int64_t)pm * nbr * nbc + at;
      for (int rb = rg; rb < nbr; rb += 255 * RG) {  // a byte counter holds 255 rows
        uint32_t sum[4] = {0, 0, 0, 0};
        const int re = (int)min<int64_t>(nbr, rb + (int64_t)255 * RG);
        if (!SHORT) {
#pragma unroll 4
          for (int r = rb; r < re; r += RG) {
            const u32x4_any x = *reinterpret_cast<const u32x4_any*>(plane + (int64_t)r * nbc);
            sum[0] += nz_bytes(x.x);
            sum[1] += nz_bytes(x.y);
            sum[2] += nz_bytes(x.z);
            sum[3] += nz_bytes(x.w);
          }
        } else if (nbc <= 2) {  // one or two byte loads are cheaper than taking 16 bytes apart
#pragma unroll 4
          for (int r = rb; r < re; r += RG) {
            const uint8_t* const p = plane + (int64_t)r * nbc;
            sum[0] += p[0] != 0 ? 1u : 0u;
            if (nbc == 2) sum[0] += p[1] != 0 ? 256u : 0u;
          }
        } else {
#pragma unroll 4
          for (int r = rb; r < re; r += RG) {
            const int row = pm * nbr + r;
            const uint32_t b = short_rows_bits(*reinterpret_cast<const u32x4_any*>(cls + short_rows_at(row)), row) & row_bits;
#pragma unroll
            for (int g = 0; g < 4; ++g) sum[g] += (((b >> (4 * g)) & 0xfu) * 0x00204081u) & 0x01010101u;  // 4 bits -> 4 bytes
          }
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const int n = (int)((sum[t >> 2] >> (8 * (t & 3))) & 0xffu);
          if (n != 0 && at + t >= c) atomicAdd(&len_s[pm * nbc + at + t], n);  // columns below c belong to the chunk before
        }
      }
    }
  }
  __syncthreads();
  if (line >= nlines) return;

  emit_line<COLS, KIND>(own_block, next, len_s, strip_s, line, seg, S, first_block, past_block, Mb, nbr, nbc, out);
}

// The index of block rows (COLS = false) or block columns in a launch of its own.
template <bool COLS, int KIND>
__global__ __launch_bounds__(kLineWaves * 64) void line_index_kernel(const uint8_t* __restrict__ cls, int Mb, int nbr, int nbc, const LineOut out) {
  __shared__ int len_s[KIND == kLineLong ? kLineMaxBytesRows / kLineLongFrom : kLineMaxLines];
  __shared__ int strip_s[KIND == kLineLong ? kLineMaxStrips : 1];
  line_index<COLS, KIND>(cls, (int)blockIdx.x, len_s, strip_s, Mb, nbr, nbc, out);
}

// Both in one launch: the first row_wgs work-groups take the rows.  Block reduction + both, us from a graph, in three launches / two:
// 1 plane of 2 x 4 blocks 9.3 / 6.8, 10 x 20 10.5 / 7.3, 32 x 64 12.2 / 8.7, 4 planes of it 23.2 / 18.5, 64 x 128 23.2 / 18.3.  The
// training step of packed sequences of 3001 124.8 -> 118.9, of 4 x 4096 195.6 -> 192.3.
template <int KIND>
__global__ __launch_bounds__(kLineWaves * 64) void line_index_both_kernel(const uint8_t* __restrict__ cls, int Mb, int nbr, int nbc, int row_wgs,
                                                                          const LineOut rows, const LineOut cols) {
  __shared__ int len_s[kLineMaxLines];
  if ((int)blockIdx.x < row_wgs)
    line_index<false, KIND>(cls, (int)blockIdx.x, len_s, len_s, Mb, nbr, nbc, rows);
  else
    line_index<true, KIND>(cls, (int)blockIdx.x - row_wgs, len_s, len_s, Mb, nbr, nbc, cols);
}

}  // namespace
}  // namespace bbm
