// Stage 1b / 1c: run index of the "Dense" variant (paper Sec. 4: total_ones / offset per block row) and the
// compact per-row list of non-zero blocks.  Both read only the small [Mb][nbr][nbc] class matrix; one
// wavefront owns one block row and works on 64 classes at a time through wave-wide ballots.
#include "bbm_internal.h"
#include "bbm_line_index.h"

namespace {

constexpr int kWavesPerWG = 4;

using bbm::RunScan;
using bbm::ctz64;
using bbm::launch_group_rows;
using bbm::wave_excl_scan;
using bbm::wave_sum;

// One wave per block row.  With `row_ptr` (rows per plane: nbr) the row's count of non-zero blocks is also left at
// row_ptr[m][i+1], which is pass 1 of the list: the index stage in one call then needs no list_count_kernel.
__global__ __launch_bounds__(kWavesPerWG * 64) void runs_kernel(const uint8_t* __restrict__ cls, int64_t rows_total,
                                                                int64_t nbc, int32_t* __restrict__ offset,
                                                                int32_t* __restrict__ total_ones,
                                                                int32_t* __restrict__ nz_lo, int32_t* __restrict__ nz_hi,
                                                                int32_t* __restrict__ nz_cnt, int32_t* __restrict__ row_ptr,
                                                                int64_t nbr) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * kWavesPerWG + (threadIdx.x >> 6);
  if (row >= rows_total) return;
  const uint8_t* c = cls + row * nbc;
  RunScan rs;
  for (int64_t base = 0; base < nbc; base += 64) {
    const uint8_t v = (base + lane < nbc) ? c[base + lane] : (uint8_t)0;
    rs.feed(__ballot(v == BBM_BLOCK_FULL), __ballot(v != BBM_BLOCK_EMPTY), (int)base);
  }
  rs.finish();
  if (lane == 0) {
    offset[row] = rs.best_start;
    total_ones[row] = rs.best_len;
    nz_lo[row] = rs.lo;
    nz_hi[row] = rs.hi;
    nz_cnt[row] = rs.cnt;
    if (row_ptr) {
      const int64_t m = row / nbr, i = row - m * nbr;
      row_ptr[m * (nbr + 1) + i + 1] = rs.cnt;
    }
  }
}

// Pass 1 of the list: row_ptr[m][i+1] <- number of non-zero blocks of row i (one wave per row).
__global__ __launch_bounds__(kWavesPerWG * 64) void list_count_kernel(const uint8_t* __restrict__ cls, int64_t Mb,
                                                                      int64_t nbr, int64_t nbc,
                                                                      int32_t* __restrict__ row_ptr) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * kWavesPerWG + (threadIdx.x >> 6);
  if (row >= Mb * nbr) return;
  const uint8_t* c = cls + row * nbc;
  int cnt = 0;
  for (int64_t base = 0; base < nbc; base += 64) {
    const uint8_t v = (base + lane < nbc) ? c[base + lane] : (uint8_t)0;
    cnt += __popcll(__ballot(v != BBM_BLOCK_EMPTY));
  }
  const int64_t m = row / nbr, i = row - m * nbr;
  if (lane == 0) row_ptr[m * (nbr + 1) + i + 1] = cnt;
}

// Pass 2: in-place inclusive scan of row_ptr[m][1..nbr], one wave per plane, 64 rows per step.
__global__ __launch_bounds__(64) void list_scan_kernel(int64_t nbr, int32_t* __restrict__ row_ptr) {
  const int lane = threadIdx.x;
  int32_t* p = row_ptr + (int64_t)blockIdx.x * (nbr + 1);
  int carry = 0;
  for (int64_t base = 0; base < nbr; base += 64) {
    int x = (base + lane < nbr) ? p[base + lane + 1] : 0;
    x += wave_excl_scan(x);
    x += carry;
    if (base + lane < nbr) p[base + lane + 1] = x;
    carry = __shfl(x, 63);
  }
  if (lane == 0) p[0] = 0;
}

// Pass 3: write the ascending list of each row at row_ptr[m][i] (one wave per row).  With `counts` ([Mb][nbr] list
// lengths, as the runs kernel leaves them in nz_cnt) pass 2 is done here as well: the wave adds up the counts of the
// rows above its own -- a few hundred integers -- and writes its entry of row_ptr itself.
__global__ __launch_bounds__(kWavesPerWG * 64) void list_fill_kernel(const uint8_t* __restrict__ cls, int64_t Mb,
                                                                     int64_t nbr, int64_t nbc,
                                                                     int32_t* __restrict__ row_ptr,
                                                                     const int32_t* __restrict__ counts,
                                                                     uint32_t* __restrict__ col_idx) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * kWavesPerWG + (threadIdx.x >> 6);
  if (row >= Mb * nbr) return;
  const int64_t m = row / nbr, i = row - m * nbr;
  const uint8_t* c = cls + row * nbc;
  int start;
  if (counts) {
    const int32_t* cp = counts + m * nbr;
    int part = 0;
    for (int64_t b = lane; b < i; b += 64) part += cp[b];
    start = __builtin_amdgcn_readlane(wave_excl_scan(part) + part, 63);
    if (lane == 0) {
      row_ptr[m * (nbr + 1) + i] = start;
      if (i == nbr - 1) row_ptr[m * (nbr + 1) + nbr] = start + cp[i];
    }
  } else {
    start = row_ptr[m * (nbr + 1) + i];
  }
  uint32_t* out = col_idx + m * nbr * nbc + start;
  int written = 0;
  for (int64_t base = 0; base < nbc; base += 64) {
    const uint8_t v = (base + lane < nbc) ? c[base + lane] : (uint8_t)0;
    const uint64_t nz = __ballot(v != BBM_BLOCK_EMPTY);
    if (v != BBM_BLOCK_EMPTY) {
      const int pos = written + __popcll(nz & ((1ull << lane) - 1ull));
      out[pos] = (uint32_t)(base + lane) | (v == BBM_BLOCK_FULL ? 0x80000000u : 0u);
    }
    written += __popcll(nz);
  }
}

// Position of block row i in the launch order of its plane.  len[0 .. nbr) = list lengths of the plane's rows,
// gmax[0 .. ceil(nbr/gsz)) = longest list of every group of gsz consecutive rows.  Order: the group holding the longest
// row first (ties: higher rows first); inside a group the longest row first (ties: higher row first).
__device__ __forceinline__ int launch_rank(const int* len, const int* gmax, int nbr, int gsz, int i) {
  const int ng = (nbr + gsz - 1) / gsz, g = i / gsz;
  const int mine = gmax[g];
  int before = 0;  // groups that go first
  for (int gg = 0; gg < ng; ++gg) {
    const int t = gmax[gg];
    before += (t > mine) || (t == mine && gg > g);
  }
  int rank = before * gsz;
  // the last group may be short; it is among the groups that go first iff its turn comes before g's
  const int last = ng - 1, last_rows = nbr - last * gsz;
  if (last != g && (gmax[last] > mine || gmax[last] == mine)) rank -= gsz - last_rows;
  const int c = len[i];
  for (int j = g * gsz; j < min(nbr, (g + 1) * gsz); ++j) rank += (len[j] > c) || (len[j] == c && j > i);
  return rank;
}

// list_fill_kernel and sched_kernel in one launch, for index stages that already have every row's list length
// (`counts` = the runs kernel's nz_cnt, [Mb][nbr]) and at most kFuseSchedRows block rows over all planes: the wave that
// fills a row's list also writes the row's launch-order record, and the records of its parts if the schedule cuts the row.
// Everything a wave needs beyond its own row -- the split threshold (a mean over all rows), the parts and cut rows
// before its own, its rank among the rows of its plane -- it counts itself from `counts` (a few hundred to a few
// thousand integers), so no wave waits for another.  Same schedule, bit for bit, as sched_kernel writes.
constexpr int64_t kFuseSchedRows = 4096;
__global__ __launch_bounds__(kWavesPerWG * 64) void list_fill_sched_kernel(const uint8_t* __restrict__ cls, int Mb, int nbr, int nbc,
                                                                           int32_t* __restrict__ row_ptr,
                                                                           const int32_t* __restrict__ counts,
                                                                           uint32_t* __restrict__ col_idx, int32_t* __restrict__ sched) {
  using namespace bbm;
  const int lane = threadIdx.x & 63;
  const int row = (int)blockIdx.x * kWavesPerWG + (int)(threadIdx.x >> 6);
  const int nrows = Mb * nbr;
  if (row >= nrows) return;
  const int m = row / nbr, i = row - m * nbr;
  const int32_t* cp = counts + (int64_t)m * nbr;
  const int c = cp[i];

  // position of the row's list in its plane, and the totals the split threshold is made of
  int above = 0, total = 0, nonempty = 0;
  for (int b = lane; b < i; b += 64) above += cp[b];
  for (int b = lane; b < nrows; b += 64) {
    const int x = counts[b];
    total += x;
    nonempty += x > 0 ? 1 : 0;
  }
  const int start = wave_sum(above);
  total = wave_sum(total);
  nonempty = wave_sum(nonempty);
  const int mean = nonempty > 0 ? (total + nonempty - 1) / nonempty : 0;
  const int T = max(kSchedMinSplit, 2 * mean);
  if (lane == 0) {
    row_ptr[(int64_t)m * (nbr + 1) + i] = start;
    if (i == nbr - 1) row_ptr[(int64_t)m * (nbr + 1) + nbr] = start + c;
  }

  // parts and cut rows: before this row (rows in (plane, block row) order), and in all
  int q = 0, rho = 0, all_parts = 0, all_cut = 0;
  for (int b = lane; b < nrows; b += 64) {
    const int x = counts[b];
    const int np_b = x > T ? (x + T - 1) / T : 0;
    all_parts += np_b;
    all_cut += np_b > 0 ? 1 : 0;
    if (b < row) {
      q += np_b;
      rho += np_b > 0 ? 1 : 0;
    }
  }
  q = wave_sum(q);
  rho = wave_sum(rho);
  if (row == 0) {
    all_parts = wave_sum(all_parts);
    all_cut = wave_sum(all_cut);
    if (lane < kSchedPartBase)
      sched[lane] = lane == kSchedNParts ? all_parts : lane == kSchedSplitT ? T : lane == kSchedNCutRows ? all_cut : 0;
  }
  const int np = c > T ? (c + T - 1) / T : 0;
  const int chunk = np > 0 ? (c + np - 1) / np : 1;
  int32_t* const parts = sched + kSchedPartBase + (int64_t)kSchedPartInts * q;
  for (int k = lane; k < np; k += 64) {
    int32_t* rec = parts + kSchedPartInts * k;
    rec[0] = row;
    rec[1] = start + k * chunk;
    rec[2] = min(chunk, c - k * chunk);
    rec[3] = k;
    rec[4] = np;
    rec[5] = q;
    rec[6] = rho;
  }

  // the list; the lane that writes the entry a part starts with also leaves it in the part's record
  const uint8_t* cl = cls + (int64_t)row * nbc;
  uint32_t* out = col_idx + (int64_t)m * nbr * nbc + start;
  int written = 0, first = -1;
  for (int base = 0; base < nbc; base += 64) {
    const uint8_t v = (base + lane < nbc) ? cl[base + lane] : (uint8_t)0;
    const uint64_t nz = __ballot(v != BBM_BLOCK_EMPTY);
    const uint64_t full = __ballot(v == BBM_BLOCK_FULL);
    if (written == 0 && nz != 0) {  // the row's first entry (this happens once: written > 0 from here on)
      const int bit = ctz64(nz);
      first = (int)((uint32_t)(base + bit) | (((full >> bit) & 1ull) ? 0x80000000u : 0u));
    }
    if (v != BBM_BLOCK_EMPTY) {
      const int pos = written + __popcll(nz & ((1ull << lane) - 1ull));
      const uint32_t entry = (uint32_t)(base + lane) | (v == BBM_BLOCK_FULL ? 0x80000000u : 0u);
      out[pos] = entry;
      if (np > 0 && pos % chunk == 0 && pos / chunk < np) parts[kSchedPartInts * (pos / chunk) + 7] = (int32_t)entry;
    }
    written += __popcll(nz);
  }

  // launch-order record: rank among the rows of the plane (launch_rank's order, counted over the lanes)
  const int gsz = launch_group_rows(T);
  const int ng = (nbr + gsz - 1) / gsz, g = i / gsz;
  auto group_max = [&](int gg) {
    int t = 0;
    for (int j = gg * gsz; j < min(nbr, (gg + 1) * gsz); ++j) t = max(t, cp[j]);
    return t;
  };
  const int mine = group_max(g);
  int before = 0;
  for (int gg = lane; gg < ng; gg += 64) {
    const int t = group_max(gg);
    before += (t > mine || (t == mine && gg > g)) ? 1 : 0;
  }
  before = wave_sum(before);
  int rank = before * gsz;
  const int last = ng - 1, last_rows = nbr - last * gsz;
  if (last != g && group_max(last) >= mine) rank -= gsz - last_rows;
  for (int j = g * gsz; j < min(nbr, (g + 1) * gsz); ++j) rank += (cp[j] > c || (cp[j] == c && j > i)) ? 1 : 0;
  if (lane == 0)
    reinterpret_cast<int4*>(sched + sched_order_base(Mb, nbr))[(int64_t)m * nbr + rank] = make_int4(i, start, c, first);
}

// Split schedule of LIST mode (layout in bbm_internal.h).  Work-group 0 writes the header and the parts table: every
// thread owns a contiguous range of block rows; pass 1 counts, per thread, the parts and the cut rows; an exclusive
// scan over the threads turns the counts into positions; pass 2 writes the parts in (row, part) order, so the
// result does not depend on the thread count.  Work-group 1 + m writes the row records of plane m in launch order,
// ranking by counting over the list lengths staged in LDS.
constexpr int kSchedThreads = 256;

__global__ __launch_bounds__(kSchedThreads) void sched_kernel(const int32_t* __restrict__ row_ptr,
                                                              const uint32_t* __restrict__ col_idx, int Mb, int nbr,
                                                              int64_t plane_entries, int32_t* __restrict__ sched) {
  using namespace bbm;
  __shared__ int pre[2][kSchedThreads + 1];
  __shared__ int red[2][kSchedThreads];
  __shared__ int len_s[kSchedMaxSortRows];
  __shared__ int gmax_s[kSchedMaxSortRows];
  const int tid = threadIdx.x;
  const int nrows = Mb * nbr;
  const int per = (nrows + kSchedThreads - 1) / kSchedThreads;
  const int r_lo = min(nrows, tid * per), r_hi = min(nrows, r_lo + per);
  auto first_entry = [&](int r) {
    const int m = r / nbr, i = r - m * nbr;
    return row_ptr + (int64_t)m * (nbr + 1) + i;
  };

  // split threshold from the mean list length of the non-empty rows (every work-group needs it)
  int total = 0, nonempty = 0;
  for (int r = r_lo; r < r_hi; ++r) {
    const int32_t* rp = first_entry(r);
    const int c = rp[1] - rp[0];
    total += c;
    nonempty += c > 0;
  }
  red[0][tid] = total;
  red[1][tid] = nonempty;
  __syncthreads();
  for (int s = kSchedThreads / 2; s > 0; s >>= 1) {
    if (tid < s) {
      red[0][tid] += red[0][tid + s];
      red[1][tid] += red[1][tid + s];
    }
    __syncthreads();
  }
  total = red[0][0];
  nonempty = red[1][0];
  const int mean = nonempty > 0 ? (total + nonempty - 1) / nonempty : 0;
  const int T = max(kSchedMinSplit, 2 * mean);

  if (blockIdx.x > 0) {
    const int m = blockIdx.x - 1;
    const int32_t* rp = row_ptr + (int64_t)m * (nbr + 1);
    const uint32_t* list = col_idx + (int64_t)m * plane_entries;
    int4* rec = reinterpret_cast<int4*>(sched + sched_order_base(Mb, nbr)) + (int64_t)m * nbr;
    const bool sorted = nbr <= kSchedMaxSortRows;
    const int gsz = launch_group_rows(T);
    if (sorted) {
      for (int j = tid; j < nbr; j += kSchedThreads) len_s[j] = rp[j + 1] - rp[j];
      __syncthreads();
      for (int g = tid; g * gsz < nbr; g += kSchedThreads) {
        int t = 0;
        for (int j = g * gsz; j < min(nbr, (g + 1) * gsz); ++j) t = max(t, len_s[j]);
        gmax_s[g] = t;
      }
      __syncthreads();
    }
    for (int i = tid; i < nbr; i += kSchedThreads) {
      const int p0 = rp[i], c = rp[i + 1] - p0;
      const int rank = sorted ? launch_rank(len_s, gmax_s, nbr, gsz, i) : nbr - 1 - i;
      rec[rank] = make_int4(i, p0, c, c > 0 ? (int)list[p0] : -1);
    }
    return;
  }

  int nparts = 0, ncut = 0;
  for (int r = r_lo; r < r_hi; ++r) {
    const int32_t* rp = first_entry(r);
    const int c = rp[1] - rp[0];
    if (c > T) {
      nparts += (c + T - 1) / T;
      ncut += 1;
    }
  }
  // exclusive scan over the threads: inside each wave with register moves, then the four wave totals through LDS
  const int lane = tid & 63, wave = tid >> 6;
  const int q_in_wave = wave_excl_scan(nparts), rho_in_wave = wave_excl_scan(ncut);
  if (lane == 63) {
    pre[0][wave] = q_in_wave + nparts;
    pre[1][wave] = rho_in_wave + ncut;
  }
  __syncthreads();
  int q = q_in_wave, rho = rho_in_wave, all_parts = 0, all_cut = 0;
  for (int w = 0; w < kSchedThreads / 64; ++w) {
    q += w < wave ? pre[0][w] : 0;
    rho += w < wave ? pre[1][w] : 0;
    all_parts += pre[0][w];
    all_cut += pre[1][w];
  }
  if (tid == 0) {
    sched[kSchedNParts] = all_parts;
    sched[kSchedSplitT] = T;
    sched[kSchedNCutRows] = all_cut;
    for (int x = 3; x < kSchedPartBase; ++x) sched[x] = 0;
  }
  for (int r = r_lo; r < r_hi; ++r) {
    const int32_t* rp = first_entry(r);
    const int c = rp[1] - rp[0];
    if (c <= T) continue;
    const uint32_t* list = col_idx + (int64_t)(r / nbr) * plane_entries;
    const int np = (c + T - 1) / T;
    const int chunk = (c + np - 1) / np;
    for (int k = 0; k < np; ++k) {
      int32_t* rec = sched + kSchedPartBase + (int64_t)kSchedPartInts * (q + k);
      rec[0] = r;
      rec[1] = rp[0] + k * chunk;
      rec[2] = min(chunk, c - k * chunk);
      rec[3] = k;
      rec[4] = np;
      rec[5] = q;
      rec[6] = rho;
      rec[7] = (int32_t)list[rp[0] + k * chunk];
    }
    q += np;
    rho += 1;
  }
}

}  // namespace

namespace {

int check_runs_args(const char* fn, const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, const int32_t* offset,
                    const int32_t* total_ones, const int32_t* nz_lo, const int32_t* nz_hi, const int32_t* nz_cnt) {
  using namespace bbm;
  if (!blk_class || !offset || !total_ones || !nz_lo || !nz_hi || !nz_cnt) return fail(BBM_EINVAL, "%s: NULL pointer argument", fn);
  if (Mb < 1 || nbr < 1 || nbc < 1)
    return fail(BBM_EINVAL, "%s: Mb=%lld, nbr=%lld, nbc=%lld must be >= 1", fn, (long long)Mb, (long long)nbr, (long long)nbc);
  if (nbc > (1ll << 30) || Mb * nbr > (1ll << 31) * kWavesPerWG - 1) return fail(BBM_EUNSUPPORTED, "%s: index too large", fn);
  return BBM_OK;
}

int check_list_args(const char* fn, const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, const int32_t* row_ptr,
                    const uint32_t* col_idx, const int32_t* sched) {
  using namespace bbm;
  if (!blk_class || !row_ptr || !col_idx) return fail(BBM_EINVAL, "%s: NULL pointer argument", fn);
  if (Mb < 1 || nbr < 1 || nbc < 1)
    return fail(BBM_EINVAL, "%s: Mb=%lld, nbr=%lld, nbc=%lld must be >= 1", fn, (long long)Mb, (long long)nbr, (long long)nbc);
  if (nbr * nbc >= (1ll << 31) || Mb * nbr >= (1ll << 24))
    return fail(BBM_EUNSUPPORTED, "%s: needs nbr*nbc=%lld < 2^31 and Mb*nbr=%lld < 2^24", fn, (long long)(nbr * nbc), (long long)(Mb * nbr));
  if (sched && !aligned(sched, 32)) return fail(BBM_EINVAL, "%s: sched must be 32-byte aligned", fn);
  return BBM_OK;
}

int launch_runs(const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, int32_t* offset, int32_t* total_ones,
                int32_t* nz_lo, int32_t* nz_hi, int32_t* nz_cnt, int32_t* row_ptr_counts, hipStream_t s) {
  const int64_t rows = Mb * nbr;
  runs_kernel<<<(unsigned)bbm::ceil_div(rows, kWavesPerWG), kWavesPerWG * 64, 0, s>>>(blk_class, rows, nbc, offset, total_ones,
                                                                                    nz_lo, nz_hi, nz_cnt, row_ptr_counts, nbr);
  return bbm::launch_status("bbm_build_runs");
}

// One launch for class matrices of ordinary size; returns false if this one is larger.
bool launch_one_kernel(const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, int32_t* row_ptr, uint32_t* col_idx,
                       int32_t* sched, int32_t* offset, int32_t* total_ones, int32_t* nz_lo, int32_t* nz_hi, int32_t* nz_cnt,
                       hipStream_t s) {
  if (!bbm::line_index_fits(false, Mb, nbr, nbc)) return false;
  const bool strips = !offset && nbc >= bbm::kLineLongFrom;
  const auto kernel = strips ? bbm::line_index_kernel<false, bbm::kLineLong>
                      : nbc < 16 ? bbm::line_index_kernel<false, bbm::kLineShort> : bbm::line_index_kernel<false, bbm::kLineNormal>;
  const int64_t units = Mb * nbr * (strips ? bbm::ceil_div(nbc, bbm::kLineStrip) : 1);
  kernel<<<(unsigned)bbm::ceil_div(units, bbm::kLineWaves), bbm::kLineWaves * 64, 0, s>>>(
      blk_class, (int)Mb, (int)nbr, (int)nbc, bbm::LineOut{row_ptr, col_idx, sched, offset, total_ones, nz_lo, nz_hi, nz_cnt});
  return true;
}

// `counts`: per-row list lengths [Mb][nbr] already on the stream (the runs kernel's nz_cnt), or NULL.  With them the
// count launch is not needed, nor -- up to kScanInFillRows block rows per plane -- the scan launch.
constexpr int64_t kScanInFillRows = 1024;
int launch_list(const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, int32_t* row_ptr, uint32_t* col_idx,
                int32_t* sched, const int32_t* counts, bool counts_in_row_ptr, hipStream_t s) {
  using namespace bbm;
  if (!counts && launch_one_kernel(blk_class, Mb, nbr, nbc, row_ptr, col_idx, sched, nullptr, nullptr, nullptr, nullptr, nullptr, s))
    return launch_status("bbm_build_sparse_index(one launch)");
  const unsigned grid = (unsigned)ceil_div(Mb * nbr, kWavesPerWG);
  int rc = BBM_OK;
  const bool scan_in_fill = counts && nbr <= kScanInFillRows;
  if (!scan_in_fill) {
    if (!counts_in_row_ptr) {
      list_count_kernel<<<grid, kWavesPerWG * 64, 0, s>>>(blk_class, Mb, nbr, nbc, row_ptr);
      rc = launch_status("bbm_build_sparse_index(count)");
      if (rc) return rc;
    }
    list_scan_kernel<<<(unsigned)Mb, 64, 0, s>>>(nbr, row_ptr);
    rc = launch_status("bbm_build_sparse_index(scan)");
    if (rc) return rc;
  }
  if (scan_in_fill && sched && Mb * nbr <= kFuseSchedRows) {  // list and schedule in one launch
    list_fill_sched_kernel<<<grid, kWavesPerWG * 64, 0, s>>>(blk_class, (int)Mb, (int)nbr, (int)nbc, row_ptr, counts, col_idx, sched);
    return launch_status("bbm_build_sparse_index(fill and schedule)");
  }
  list_fill_kernel<<<grid, kWavesPerWG * 64, 0, s>>>(blk_class, Mb, nbr, nbc, row_ptr, scan_in_fill ? counts : nullptr, col_idx);
  rc = launch_status("bbm_build_sparse_index(fill)");
  if (rc || !sched) return rc;
  sched_kernel<<<(unsigned)(1 + Mb), kSchedThreads, 0, s>>>(row_ptr, col_idx, (int)Mb, (int)nbr, nbr * nbc, sched);
  return launch_status("bbm_build_sparse_index(schedule)");
}

}  // namespace

extern "C" __attribute__((visibility("default"))) int bbm_build_runs(const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, int32_t* offset,
                              int32_t* total_ones, int32_t* nz_lo, int32_t* nz_hi, int32_t* nz_cnt, void* stream) {
  bbm::clear_error();
  const int rc = check_runs_args("bbm_build_runs", blk_class, Mb, nbr, nbc, offset, total_ones, nz_lo, nz_hi, nz_cnt);
  if (rc) return rc;
  return launch_runs(blk_class, Mb, nbr, nbc, offset, total_ones, nz_lo, nz_hi, nz_cnt, nullptr, static_cast<hipStream_t>(stream));
}

extern "C" __attribute__((visibility("default"))) size_t bbm_sched_bytes(int64_t Mb, int64_t nbr) {
  if (Mb < 1 || nbr < 1) return 0;
  return (size_t)bbm::sched_ints(Mb, nbr) * sizeof(int32_t);
}

extern "C" __attribute__((visibility("default"))) int bbm_build_sparse_index(const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc,
                                      int32_t* row_ptr, uint32_t* col_idx, int32_t* sched, void* stream) {
  bbm::clear_error();
  const int rc = check_list_args("bbm_build_sparse_index", blk_class, Mb, nbr, nbc, row_ptr, col_idx, sched);
  if (rc) return rc;
  return launch_list(blk_class, Mb, nbr, nbc, row_ptr, col_idx, sched, nullptr, false, static_cast<hipStream_t>(stream));
}

extern "C" __attribute__((visibility("default"))) int bbm_build_index(const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, int32_t* offset,
                               int32_t* total_ones, int32_t* nz_lo, int32_t* nz_hi, int32_t* nz_cnt, int32_t* row_ptr,
                               uint32_t* col_idx, int32_t* sched, void* stream) {
  using namespace bbm;
  clear_error();
  int rc = check_runs_args("bbm_build_index", blk_class, Mb, nbr, nbc, offset, total_ones, nz_lo, nz_hi, nz_cnt);
  if (rc) return rc;
  rc = check_list_args("bbm_build_index", blk_class, Mb, nbr, nbc, row_ptr, col_idx, sched);
  if (rc) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (launch_one_kernel(blk_class, Mb, nbr, nbc, row_ptr, col_idx, sched, offset, total_ones, nz_lo, nz_hi, nz_cnt, s))
    return launch_status("bbm_build_index(one launch)");
  // the runs kernel's counts are pass 1 of the list: in nz_cnt for the fill kernel, and in row_ptr where a scan launch follows
  const bool scan_launch = nbr > kScanInFillRows;
  rc = launch_runs(blk_class, Mb, nbr, nbc, offset, total_ones, nz_lo, nz_hi, nz_cnt, scan_launch ? row_ptr : nullptr, s);
  if (rc) return rc;
  return launch_list(blk_class, Mb, nbr, nbc, row_ptr, col_idx, sched, nz_cnt, scan_launch, s);
}

namespace bbm {
int check_index_args(const char* fn, const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, const LineArgs& rows) {
  int rc = check_runs_args(fn, blk_class, Mb, nbr, nbc, rows.offset, rows.total_ones, rows.nz_lo, rows.nz_hi, rows.nz_cnt);
  return rc ? rc : check_list_args(fn, blk_class, Mb, nbr, nbc, rows.ptr, rows.list, rows.sched);
}

bool launch_rows_and_columns(const uint8_t* blk_class, int64_t Mb, int64_t nbr, int64_t nbc, const LineArgs& rows, const LineArgs& cols, hipStream_t s) {
  if (!line_index_fits(false, Mb, nbr, nbc) || !line_index_fits(true, Mb, nbr, nbc)) return false;
  const int64_t row_wgs = ceil_div(Mb * nbr, kLineWaves), col_wgs = ceil_div(Mb * nbc, kLineWaves);
  const auto kernel = nbc < 16 ? line_index_both_kernel<kLineShort> : line_index_both_kernel<kLineNormal>;
  kernel<<<(unsigned)(row_wgs + col_wgs), kLineWaves * 64, 0, s>>>(blk_class, (int)Mb, (int)nbr, (int)nbc, (int)row_wgs, rows, cols);
  return true;
}
}  // namespace bbm
