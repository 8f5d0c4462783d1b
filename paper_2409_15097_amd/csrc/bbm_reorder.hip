// Reverse Cuthill-McKee reordering of a sparse attention mask on the GPU (paper Sec. 4 "Binary Block Masking with
// Reverse Cuthill-McKee (RCM)": the mask is treated as a graph and reordered so that fewer blocks are non-zero), and the
// gathers that apply the permutation to the mask and to Q/K/V/O rows.
//
// The ordering is the published algorithm with every choice fixed (the library header states them): neighbours of node
// i are the non-zero entries of mask row i, a component starts at its unvisited node of minimum degree (ties: smallest
// index), each breadth-first level is ordered by (position of the earliest parent, degree, index), the result is
// reversed.  One kernel packs the mask rows to bits and counts degrees; the levels are then walked by a kernel each, which ranks a
// level and finds the next one at the same time, with no host round trip and no grid-wide barrier, every node's row being scanned
// once; a last kernel of one work-group walks whatever the fixed number of them left.
#include "bbm_internal.h"

#include <algorithm>
#include <climits>

namespace {

constexpr int kMaxNodes = 65536;            // visited set and one mask row must fit in LDS
constexpr size_t kLdsBytes = 160 * 1024;
constexpr int kOrderThreads = 1024;
constexpr int kPackThreads = 256;
constexpr int kRounds = 48;                 // parallel rounds, a breadth-first level each
constexpr int kRankChunk = 2048;            // keys of a level staged in LDS at a time
constexpr int kRankPerThread = 4;           // keys a thread ranks per sweep
constexpr int kBatch = 8;                   // row words a thread of the level walk has in flight
constexpr int64_t kSmallMaskBytes = 512 * 512;  // masks up to here are permuted a byte per lane

// 4 mask bytes -> 4 bits (bit t = byte t non-zero).
__device__ __forceinline__ uint32_t nz_nibble(uint32_t x) {
  uint32_t y = (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;
  return (((y >> 7) * 0x00204081u) >> 21) & 0xfu;
}

// Four words as a 4 x 4 byte matrix, transposed: out[i] holds byte i of a, b, c, d.
__device__ __forceinline__ void transpose4x4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&out)[4]) {
  const uint32_t ab_lo = __builtin_amdgcn_perm(b, a, 0x05010400u), ab_hi = __builtin_amdgcn_perm(b, a, 0x07030602u);  // a0 b0 a1 b1, a2 b2 a3 b3
  const uint32_t cd_lo = __builtin_amdgcn_perm(d, c, 0x05010400u), cd_hi = __builtin_amdgcn_perm(d, c, 0x07030602u);
  out[0] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u);
  out[1] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u);
  out[2] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u);
  out[3] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u);
}

// The level walk in the workspace: two records that the rounds use in turn, one read and one written, so no kernel resets what
// another may still be reading.  The node numbers are cut into regions of kRegCols; a record holds whether the walk has
// ended, how many nodes are placed, and per region the nodes of the level to come that lie in it (how many; the list itself
// has an array of its own) and its unvisited node of minimum (degree, index).
constexpr int kRegWords = 8, kRegCols = 64 * kRegWords, kMaxRegs = kMaxNodes / kRegCols;
enum { kStDone = 0, kStPlaced = 1, kStInts = 4 };
struct WalkRecord {
  int32_t* state;        // [kStInts]
  int32_t* count;        // [regions]
  uint64_t* lowest;      // [regions] degree << 32 | node, ~0 where every node is visited
  uint32_t* list;        // [regions][kRegCols] node | parent << 16, nodes in ascending order
};

typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(1)));  // 16 bytes at any address: one instruction

// One work-group per mask row: bits[row][w] (row-major, bits past N zero), degree[row], parent_pos[row] = "none".
// Bound by the mask's bytes (N = 32768: 0.20 ms, 6.0 TB/s read and written): a lane reads 16 of them, neighbouring lanes
// neighbouring pieces, four loads in flight, and writes the 16 bits as one piece of a word.  The loads are streaming ones at
// every size although the permutation reads the mask again: with ordinary loads, here or in the permutation or in both,
// ordering + permutation + index of 8192 nodes take 286-294 us (streaming 293), of 16384 490-500 (483), of 32768 1214-1261 (1178).  The piece that reaches past
// column N is read as the row's last 16 bytes and shifted down, so rows of any length and alignment run the same
// instructions.
__global__ __launch_bounds__(kPackThreads) void rcm_pack_kernel(const uint8_t* __restrict__ mask, int N, int64_t row_stride, int W,
                                                                uint16_t* __restrict__ bits, int32_t* __restrict__ degree,
                                                                int32_t* __restrict__ parent_pos) {
  __shared__ int red_s[kPackThreads / 64];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const uint8_t* __restrict__ src = mask + (int64_t)row * row_stride;
  uint16_t* __restrict__ dst = bits + (int64_t)row * W * 4;
  const int pieces = 4 * W;
  int count = 0;
  if (N >= 16) {
    constexpr int kUnroll = 4;
    for (int p0 = tid; p0 < pieces; p0 += kUnroll * kPackThreads) {
      u32x4_any x[kUnroll];
      int shift[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int col = 16 * (p0 + u * kPackThreads), at = min(col, N - 16);
        shift[u] = min(col - at, 31);
        x[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(src + at));
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const uint32_t b = (nz_nibble(x[u].x) | (nz_nibble(x[u].y) << 4) | (nz_nibble(x[u].z) << 8) | (nz_nibble(x[u].w) << 12)) >> shift[u];
        if (p0 + u * kPackThreads < pieces) {
          dst[p0 + u * kPackThreads] = (uint16_t)b;
          count += __popc(b);
        }
      }
    }
  } else if (tid < pieces) {  // fewer than 16 columns: one word of four pieces
    uint32_t b = 0;
    for (int t = 0; t < 16; ++t)
      if (16 * tid + t < N && src[16 * tid + t] != 0) b |= 1u << t;
    dst[tid] = (uint16_t)b;
    count = __popc(b);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) count += __shfl_xor(count, d);
  if (lane == 0) red_s[tid >> 6] = count;
  __syncthreads();
  if (tid == 0) {
    int total = 0;
    for (int w = 0; w < kPackThreads / 64; ++w) total += red_s[w];
    degree[row] = total;
    parent_pos[row] = INT_MAX;
  }
}

__device__ __forceinline__ uint64_t level_key(int parent, int degree, int v) {
  return ((uint64_t)(uint32_t)parent << 40) | ((uint64_t)(uint32_t)degree << 20) | (uint64_t)(uint32_t)v;
}

// Ranks the L distinct keys by counting and calls place(rank, node) for each; the keys pass through LDS in chunks and
// a thread ranks up to kRankPerThread keys per sweep.  All kOrderThreads threads of the work-group must call it.
template <typename Place>
__device__ __forceinline__ void rank_level(const uint64_t* keys, int L, uint64_t* chunk_s, int tid, Place place) {
  for (int c0 = 0; c0 < L; c0 += kRankPerThread * kOrderThreads) {
    uint64_t mine[kRankPerThread];
    int r[kRankPerThread];
#pragma unroll
    for (int t = 0; t < kRankPerThread; ++t) {
      const int c = c0 + t * kOrderThreads + tid;
      mine[t] = c < L ? keys[c] : 0;
      r[t] = 0;
    }
    for (int j0 = 0; j0 < L; j0 += kRankChunk) {
      const int n = min(kRankChunk, L - j0);
      __syncthreads();  // the previous chunk has been read
      for (int j = tid; j < n; j += kOrderThreads) chunk_s[j] = keys[j0 + j];
      __syncthreads();
      for (int j = 0; j < n; ++j) {
        const uint64_t kj = chunk_s[j];
#pragma unroll
        for (int t = 0; t < kRankPerThread; ++t) r[t] += kj < mine[t] ? 1 : 0;
      }
    }
#pragma unroll
    for (int t = 0; t < kRankPerThread; ++t)
      if (c0 + t * kOrderThreads + tid < L) place(r[t], (int)(mine[t] & 0xfffffull));
  }
}

// The unvisited node of minimum (degree, index), or -1: every one of the work-group's THREADS threads gets the result.
// A thread looks at four neighbouring nodes at a time, with kFly such groups in flight: the scan is a chain of loads.
template <int THREADS, typename Visited>
__device__ __forceinline__ int min_degree_unvisited(const int32_t* __restrict__ degree, int N, Visited visited_word,
                                                    unsigned long long* min_s, int tid) {
  constexpr int kFly = 4;
  const int lane = tid & 63, wave = tid >> 6;
  unsigned long long best = ~0ull;
  const int last4 = (N - 1) & ~3;  // degree is 16-byte aligned and padded to whole 256 bytes: groups of four are readable
  for (int i0 = 4 * tid; i0 < N; i0 += 4 * kFly * THREADS) {
    int4 dg[kFly];
    uint64_t vw[kFly];
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      const int i = min(i0 + 4 * u * THREADS, last4);  // past the end: the last group once more
      dg[u] = *reinterpret_cast<const int4*>(degree + i);
      vw[u] = visited_word(i >> 6) >> (i & 63);
    }
#pragma unroll
    for (int u = 0; u < kFly; ++u) {
      const int i = min(i0 + 4 * u * THREADS, last4);
      const int d4[4] = {dg[u].x, dg[u].y, dg[u].z, dg[u].w};
#pragma unroll
      for (int t = 0; t < 4; ++t)  // nodes past N count as visited
        if (!((vw[u] >> t) & 1ull)) best = min(best, ((unsigned long long)(uint32_t)d4[t] << 32) | (uint32_t)(i + t));
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) best = min(best, (unsigned long long)__shfl_xor(best, d));
  __syncthreads();  // min_s may still be read from an earlier call
  if (lane == 0) min_s[wave] = best;
  __syncthreads();
  best = min_s[0];
  for (int w = 1; w < THREADS / 64; ++w) best = min(best, min_s[w]);
  return best == ~0ull ? -1 : (int)(best & 0xffffffffull);
}

constexpr int kLevelThreads = 1024, kLevelWaves = kLevelThreads / 64;
constexpr int kLevelStage = 4096;    // keys of a level staged in LDS at a time
// Ranking work-groups of a round.  A CU holds one work-group of this kernel: with the expanding ones, one a region, all start at once
// up to 64 regions (32768 nodes).  Above, the last of at most 320 start when others end.
constexpr int kRankWGs = 192;
constexpr int kRankSlice = (kMaxNodes + kRankWGs - 1) / kRankWGs;

__device__ __forceinline__ uint64_t wave_min64(uint64_t x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x = min(x, (uint64_t)__shfl_xor((unsigned long long)x, d));
  return x;
}

// One round of the walk: the current level (the lists `in` holds, or, when those are empty, the start of the next component) is
// ranked and expanded side by side.  What makes that possible: which parent of a node comes first is a comparison of the
// parents' keys, not of their places, so the expansion does not wait for the ranking; the places it leaves are needed a round
// later, for the keys of the level found now.
//   work-group < regions: expands the whole level into the nodes of its own region.  Every bit row of the level is read once over
//     all regions, 8 words of it here; a node's earliest parent is a minimum in LDS, so there are no atomics on memory, and the
//     list, the visited words and the region's unvisited minimum are this work-group's alone.
//   the others: a node's place in the level is the number of smaller keys, counted by a wave, of which every work-group stages all.
// What bounds it is the chain of dependent round trips: counts, list, places and degrees, bit rows, results; the ranking is done
// before the expansion is, and the minima in LDS are 0.5 us of it.  Before, a round was an expanding kernel (atomics on memory, a
// candidate list behind one counter) and a ranking one: a level of 1700 nodes of the 32768-node power-law graph took 8 + 9 us, now
// 12.4.  The whole ordering, of which 200 us are the packing at 32768 nodes, us: 1000 nodes 259-348 -> 140-154, 8192 335-395 ->
// 166-180, 16000 364-407 -> 236-246, 32768 623 -> 467; 65536, where the launch is larger than the chip, 1608 -> 1487.  Large levels, of random
// graphs of 16 to 512 edges a node: 8192 nodes 295 -> 170, 32768 930-1000 -> 490-540, 65536 2240-2340 -> 1860-2160; stars of 32768 and
// 65536 1005 -> 540, 2342 -> 2188; a band of 8192 nodes (many small levels) 428 -> 327.  Thousands of components, which the last kernel
// walks, take what they took (32768 nodes with 4 edges each 31.4 ms).  Regions of 4 words instead of 8 (32768 nodes): 554.  All levels in one launch
// whose work-groups wait for each other's flags: 105, 152, 230, 481; not worth the waiting.  Every region's first 64 nodes asked
// for along with the counts: no difference.
__global__ __launch_bounds__(kLevelThreads) void rcm_level_kernel(const uint64_t* __restrict__ bits, const int32_t* __restrict__ degree,
                                                                  uint64_t* __restrict__ visited, int32_t* pos, int32_t* __restrict__ perm,
                                                                  const WalkRecord in, const WalkRecord out, int N, int W, int regions) {
  __shared__ uint64_t key_s[kLevelStage];
  __shared__ unsigned long long best_s[kRegCols];  // the smallest parent's key
  __shared__ uint64_t own_s[kRankSlice];
  __shared__ int rank_s[kRankSlice];
  __shared__ int first_s[kMaxRegs + 1];  // place of a region's list in the level
  __shared__ int found_s[kRegWords];
  __shared__ uint64_t lowest_s[kRegWords];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool done = in.state[kStDone] != 0;
  const int placed = in.state[kStPlaced];
  // every wave: the regions' counts, kPer a lane, added up
  constexpr int kPer = kMaxRegs / 64;
  int c[kPer], own = 0;
#pragma unroll
  for (int t = 0; t < kPer; ++t) c[t] = kPer * lane + t < regions ? in.count[kPer * lane + t] : 0;
  if (done) {
    if (blockIdx.x == 0 && tid == 0) out.state[kStDone] = 1;
    return;
  }
#pragma unroll
  for (int t = 0; t < kPer; ++t) own += c[t];
  int upto = own;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int other = __shfl_up(upto, d);
    if (lane >= d) upto += other;
  }
  int L = __shfl(upto, 63), start = -1;
  if (L == 0) {  // the next component starts at its unvisited node of minimum (degree, index)
    uint64_t low = ~0ull;
    for (int reg = lane; reg < regions; reg += 64) low = min(low, in.lowest[reg]);
    low = wave_min64(low);
    if (low == ~0ull) {
      if (blockIdx.x == 0 && tid == 0) out.state[kStDone] = 1;
      return;
    }
    start = (int)(low & 0xffffffffull);
    L = 1;
  }
  if (blockIdx.x == 0 && tid == 0) {
    out.state[kStDone] = 0;
    out.state[kStPlaced] = placed + L;
  }
  if (wave == 0) {
    int at = upto - own;
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      first_s[kPer * lane + t] = at;
      at += c[t];
    }
    if (lane == 63) first_s[kMaxRegs] = upto;
  }

  // Keys [from, to) of the level into dst (all threads; barriers on both sides).  A wave takes every 16th region, the first 64
  // nodes of each with all loads in flight.
  auto stage = [&](int from, int to, uint64_t* dst) {
    __syncthreads();
    if (start >= 0) {
      if (tid == 0) dst[0] = (uint64_t)start;
    } else {
      constexpr int kFly = kMaxRegs / kLevelWaves;
      uint32_t e[kFly];
      int at[kFly], ps[kFly], dg[kFly];
#pragma unroll
      for (int t = 0; t < kFly; ++t) {
        const int r = wave + t * kLevelWaves;
        at[t] = first_s[r] + lane;
        if (at[t] >= first_s[r + 1] || at[t] < from || at[t] >= to) at[t] = -1;
        e[t] = at[t] >= 0 ? in.list[r * kRegCols + lane] : 0;
      }
#pragma unroll
      for (int t = 0; t < kFly; ++t) {
        ps[t] = pos[e[t] >> 16];
        dg[t] = degree[e[t] & 0xffffu];
      }
#pragma unroll
      for (int t = 0; t < kFly; ++t)
        if (at[t] >= 0) dst[at[t] - from] = level_key(ps[t], dg[t], (int)(e[t] & 0xffffu));
      for (int r = wave; r < regions; r += kLevelWaves)
        for (int a = first_s[r] + 64 + lane; a < min(first_s[r + 1], to); a += 64)
          if (a >= from) {
            const uint32_t x = in.list[r * kRegCols + a - first_s[r]];
            dst[a - from] = level_key(pos[x >> 16], degree[x & 0xffffu], (int)(x & 0xffffu));
          }
    }
    __syncthreads();
  };

  if ((int)blockIdx.x < regions) {
    // neighbouring regions, which share the cache lines of the bit rows, on one XCD
    constexpr int kShare = 16 / kRegWords;
    int reg = blockIdx.x;
    if ((reg | (8 * kShare - 1)) < regions) reg = (reg & ~(8 * kShare - 1)) | ((reg & 7) * kShare) | ((reg >> 3) & (kShare - 1));
    const int own_word = lane & (kRegWords - 1), w = reg * kRegWords + own_word;
    uint64_t before = w < W ? visited[w] : ~0ull;
    if (start >= 0 && (start >> 6) == w) before |= 1ull << (start & 63);
    const int col = reg * kRegCols + tid, dg_own = tid < kRegCols && col < N ? degree[col] : 0;
    if (tid < kRegCols) best_s[tid] = ~0ull;
    const uint64_t* const base = bits + min(w, W - 1);
    for (int j0 = 0; j0 < L; j0 += kLevelStage) {
      const int n = min(kLevelStage, L - j0);
      stage(j0, j0 + n, key_s);
      constexpr int kFly = 16, kNodes = kLevelThreads / kRegWords;  // loads of a lane in flight, nodes of a load
      for (int f0 = tid / kRegWords; f0 < n; f0 += kFly * kNodes) {
        uint64_t word[kFly];
#pragma unroll
        for (int t = 0; t < kFly; ++t) word[t] = base[(int64_t)(key_s[min(f0 + t * kNodes, n - 1)] & 0xfffffull) * W];
#pragma unroll
        for (int t = 0; t < kFly; ++t) {
          uint64_t b = f0 + t * kNodes < n ? word[t] & ~before : 0;
          while (b) {
            atomicMin(&best_s[own_word * 64 + __builtin_ctzll(b)], (unsigned long long)key_s[f0 + t * kNodes]);
            b &= b - 1;
          }
        }
      }
    }
    __syncthreads();
    uint64_t best = ~0ull, fresh = 0;
    if (wave < kRegWords) {  // a wave per word
      best = best_s[tid];
      fresh = __ballot(best != ~0ull);
      const uint64_t after = (uint64_t)__shfl((unsigned long long)before, wave) | fresh;
      if (lane == 0 && reg * kRegWords + wave < W) visited[reg * kRegWords + wave] = after;
      const uint64_t low = wave_min64((after >> lane) & 1ull ? ~0ull : (uint64_t)(uint32_t)dg_own << 32 | (uint32_t)col);
      if (lane == 0) {
        found_s[wave] = __popcll(fresh);
        lowest_s[wave] = low;
      }
    }
    __syncthreads();
    if (wave < kRegWords) {
      int at = __popcll(fresh & ((1ull << lane) - 1ull));
      for (int t = 0; t < wave; ++t) at += found_s[t];
      if (best != ~0ull) out.list[reg * kRegCols + at] = (uint32_t)col | (uint32_t)(best & 0xffffull) << 16;
    }
    if (tid == 0) {
      int total = 0;
      uint64_t low = ~0ull;
      for (int t = 0; t < kRegWords; ++t) {
        total += found_s[t];
        low = min(low, lowest_s[t]);
      }
      out.count[reg] = total;
      out.lowest[reg] = low;
    }
  } else {
    const int slices = (int)gridDim.x - regions, len = (L + slices - 1) / slices;
    const int lo = ((int)blockIdx.x - regions) * len, hi = min(L, lo + len);
    if (lo >= hi) return;
    for (int t = tid; t < hi - lo; t += kLevelThreads) rank_s[t] = 0;
    if (L > kLevelStage) stage(lo, hi, own_s);
    for (int j0 = 0; j0 < L; j0 += kLevelStage) {
      const int n = min(kLevelStage, L - j0);
      stage(j0, j0 + n, key_s);
      for (int c = wave; c < hi - lo; c += kLevelWaves) {
        const uint64_t mine = L > kLevelStage ? own_s[c] : key_s[lo + c];
        int r = 0;
#pragma unroll 8
        for (int j = lane; j < n; j += 64) r += key_s[j] < mine ? 1 : 0;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) r += __shfl_xor(r, d);
        if (lane == 0) rank_s[c] += r;  // (this wave's alone)
        if (lane == 0 && j0 + n == L) {
          const int v = (int)(mine & 0xfffffull), p = placed + rank_s[c];
          pos[v] = p;
          perm[N - 1 - p] = v;
        }
      }
    }
  }
}

// What the first round reads: nothing placed, no level, every region's node of minimum (degree, index).
__global__ __launch_bounds__(kRegCols) void rcm_start_kernel(const int32_t* __restrict__ degree, uint64_t* __restrict__ visited,
                                                             const WalkRecord out, int N, int W) {
  __shared__ uint64_t lowest_s[kRegWords];
  const int reg = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, col = reg * kRegCols + tid;
  const uint64_t low = wave_min64(col < N ? (uint64_t)(uint32_t)degree[col] << 32 | (uint32_t)col : ~0ull);
  if ((tid & 63) == 0) {
    const int w = reg * kRegWords + wave;
    lowest_s[wave] = low;
    if (w < W) visited[w] = w == W - 1 && (N & 63) ? ~0ull << (N & 63) : 0ull;  // nodes past N count as visited
  }
  __syncthreads();
  if (tid == 0) {
    uint64_t all = ~0ull;
    for (int t = 0; t < kRegWords; ++t) all = min(all, lowest_s[t]);
    out.count[reg] = 0;
    out.lowest[reg] = all;
    if (reg == 0) {
      out.state[kStDone] = 0;
      out.state[kStPlaced] = 0;
    }
  }
}

// The finisher, one work-group: whatever the rounds left (nothing, for graphs of few levels and components) is walked
// here with the expansion done by the same work-group.  Global arrays written
// by some threads and read by others are separated by an agent-scope fence and a barrier.
__global__ __launch_bounds__(kOrderThreads) void rcm_finish_kernel(const uint64_t* __restrict__ bits, const int32_t* __restrict__ degree,
                                                                   int32_t* parent_pos, int32_t* order, int32_t* cand, uint64_t* keys,
                                                                   const uint64_t* __restrict__ visited_g, const WalkRecord left, int N, int W,
                                                                   int regions, int32_t* __restrict__ perm) {
  __shared__ uint64_t visited[kMaxNodes / 64];
  __shared__ uint64_t claimed[kMaxNodes / 64];  // nodes some frontier node has reached (they become visited within the level)
  __shared__ uint64_t chunk_s[kRankChunk];
  __shared__ unsigned long long min_s[kOrderThreads / 64];
  __shared__ int count_s;
  __shared__ int first_s[kMaxRegs + 1];
  const int tid = threadIdx.x;
  auto sync_global = [&]() {
    __threadfence();
    __syncthreads();
  };
  if (left.state[kStDone]) return;
  int n_done = left.state[kStPlaced];
  // the level that the last round found: listed and marked visited, not ranked (its parents' places are where `order` will be)
  if (tid == 0) {
    int sum = 0;
    for (int r = 0; r < regions; ++r) {
      first_s[r] = sum;
      sum += left.count[r];
    }
    first_s[regions] = sum;
  }
  __syncthreads();
  for (int r = tid >> 6; r < regions; r += kOrderThreads / 64)
    for (int c = first_s[r] + (tid & 63); c < first_s[r + 1]; c += 64) {
      const uint32_t e = left.list[r * kRegCols + c - first_s[r]];
      keys[c] = level_key(order[e >> 16], degree[e & 0xffffu], (int)(e & 0xffffu));
    }
  sync_global();
  rank_level(keys, first_s[regions], chunk_s, tid, [&](int r, int v) {
    order[n_done + r] = v;
    perm[N - 1 - n_done - r] = v;
  });
  int lvl_lo = n_done, lvl_hi = n_done + first_s[regions];
  n_done = lvl_hi;
  sync_global();
  {
    for (int w = tid; w < kMaxNodes / 64; w += kOrderThreads) {
      visited[w] = w < W ? visited_g[w] : ~0ull;  // nodes past N were marked visited when the set was initialised
      claimed[w] = 0;
    }
    if (tid == 0) count_s = 0;
    __syncthreads();
    while (true) {
      // ---- breadth-first levels of the current component
      while (lvl_lo < lvl_hi) {
        const int64_t total = (int64_t)(lvl_hi - lvl_lo) * W;
        for (int64_t x0 = tid; x0 < total; x0 += kBatch * kOrderThreads) {
          uint64_t word[kBatch];
          int f[kBatch], w[kBatch];
#pragma unroll
          for (int t = 0; t < kBatch; ++t) {
            const int64_t x = x0 + (int64_t)t * kOrderThreads;
            word[t] = 0;
            f[t] = w[t] = 0;
            if (x < total) {
              f[t] = lvl_lo + (int)(x / W);
              w[t] = (int)(x % W);
              word[t] = bits[(int64_t)order[f[t]] * W + w[t]] & ~visited[w[t]];
            }
          }
#pragma unroll
          for (int t = 0; t < kBatch; ++t) {
            uint64_t b = word[t];
            while (b) {
              const int v = 64 * w[t] + __builtin_ctzll(b);
              b &= b - 1;
              atomicMin(&parent_pos[v], f[t]);  // result unused: a thread's atomics pipeline instead of each waiting for its return
              const unsigned long long bit = 1ull << (v & 63);
              if (!(atomicOr(reinterpret_cast<unsigned long long*>(&claimed[v >> 6]), bit) & bit)) cand[atomicAdd(&count_s, 1)] = v;
            }
          }
        }
        sync_global();
        const int L = count_s;
        for (int c = tid; c < L; c += kOrderThreads) {
          const int v = cand[c];
          keys[c] = level_key(parent_pos[v], degree[v], v);
        }
        sync_global();
        rank_level(keys, L, chunk_s, tid, [&](int r, int v) {
          order[n_done + r] = v;
          perm[N - 1 - n_done - r] = v;
          atomicOr(reinterpret_cast<unsigned long long*>(&visited[v >> 6]), 1ull << (v & 63));
        });
        if (tid == 0) count_s = 0;
        lvl_lo = lvl_hi;
        lvl_hi = n_done + L;
        n_done += L;
        sync_global();
      }
      // ---- next component
      const int start = min_degree_unvisited<kOrderThreads>(degree, N, [&](int w) { return visited[w]; }, min_s, tid);
      if (start < 0) break;
      if (tid == 0) {
        order[n_done] = start;
        perm[N - 1 - n_done] = start;
        visited[start >> 6] |= 1ull << (start & 63);
      }
      lvl_lo = n_done;
      lvl_hi = n_done + 1;
      n_done += 1;
      sync_global();
    }
  }
}

// out[m][i][j] = mask[m][perm[i]][perm[j]], a byte per lane, for masks that are all latency: two dependent reads and a store.
__global__ __launch_bounds__(256) void permute_small_mask_kernel(const uint8_t* __restrict__ mask, int N, int64_t row_stride,
                                                                 const int32_t* __restrict__ perm, uint8_t* __restrict__ out) {
  const int j = blockIdx.x * 64 + (threadIdx.x & 63), i = blockIdx.y * 4 + (threadIdx.x >> 6);
  const int64_t m = blockIdx.z;
  if (i >= N || j >= N) return;
  // entries of perm outside [0, N) are clamped: a wrong permutation gives a wrong mask, never a wild access
  const int pi = min(max(perm[i], 0), N - 1), pj = min(max(perm[j], 0), N - 1);
  out[(m * N + i) * N + j] = mask[(m * N + pi) * row_stride + pj];
}

// The same for N >= 16.  One work-group per R output rows: it stages the R source rows in LDS, byte c of
// all R rows side by side, so that one LDS read delivers column perm[j] of all of them, then gathers 16 columns per lane
// and turns the R-byte columns into 16-byte pieces of R rows.  Rows of any length and alignment: the last piece of a row
// is moved back to end with the row (bytes handled twice get the same value).
// With one LDS read per byte (R = 1) the random reads and their bank conflicts bound the kernel, not memory: N = 32768
// 705 us.  R = 2: 404 us; R = 4: 384 us (5.6 TB/s).  Odd sizes, which were copied byte by byte: N = 20001 170 us (R = 2: 181).
template <int R>
__global__ __launch_bounds__(1024) void permute_mask_kernel(const uint8_t* __restrict__ mask, int N, int64_t row_stride,
                                                            const int32_t* __restrict__ perm, uint8_t* __restrict__ out) {
  extern __shared__ __attribute__((aligned(16))) uint8_t rows_s[];  // [N rounded up to 16][R]
  typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
  const int i0 = blockIdx.x * R, tid = threadIdx.x, NT = blockDim.x;
  const int64_t m = blockIdx.y;
  const uint8_t* src[R];
#pragma unroll
  for (int r = 0; r < R; ++r)  // entries of perm outside [0, N) are clamped: a wrong permutation gives a wrong mask, never a wild access
    src[r] = mask + (m * N + min(max(perm[min(i0 + r, N - 1)], 0), N - 1)) * row_stride;
  uint8_t* const dst = out + (m * N + i0) * (int64_t)N;
  for (int c = 16 * tid; c < N; c += 16 * NT) {
    const int at = min(c, N - 16);
    u32x4_any x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(src[r] + at));
    if constexpr (R == 4) {
      uint32_t* const d = reinterpret_cast<uint32_t*>(rows_s) + at;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint32_t col[4];
        transpose4x4(x[0][g], x[1][g], x[2][g], x[3][g], col);
        if (at == c)
          *reinterpret_cast<uint4*>(d + 4 * g) = make_uint4(col[0], col[1], col[2], col[3]);
        else
          for (int t = 0; t < 4; ++t) d[4 * g + t] = col[t];
      }
    } else if constexpr (R == 2) {
      uint16_t* const d = reinterpret_cast<uint16_t*>(rows_s) + at;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t lo = __builtin_amdgcn_perm(x[1][g], x[0][g], 0x05010400u), hi = __builtin_amdgcn_perm(x[1][g], x[0][g], 0x07030602u);
        if (at == c) {
          *reinterpret_cast<uint2*>(d + 4 * g) = make_uint2(lo, hi);
        } else {
          d[4 * g] = (uint16_t)lo, d[4 * g + 1] = (uint16_t)(lo >> 16);
          d[4 * g + 2] = (uint16_t)hi, d[4 * g + 3] = (uint16_t)(hi >> 16);
        }
      }
    }
  }
  __syncthreads();
  for (int c = 16 * tid; c < N; c += 16 * NT) {
    const int at = min(c, N - 16);
    u32x4_any y[R];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const i32x4_any p = *reinterpret_cast<const i32x4_any*>(perm + at + 4 * g);
      if constexpr (R == 4) {
        uint32_t v[4], o[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = reinterpret_cast<const uint32_t*>(rows_s)[min(max(p[t], 0), N - 1)];
        transpose4x4(v[0], v[1], v[2], v[3], o);
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r][g] = o[r];
      } else if constexpr (R == 2) {
        uint32_t v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = reinterpret_cast<const uint16_t*>(rows_s)[min(max(p[t], 0), N - 1)];
        const uint32_t a = v[0] | (v[1] << 16), b = v[2] | (v[3] << 16);  // (r0, r1) of columns 0, 1 and of columns 2, 3
        y[0][g] = __builtin_amdgcn_perm(b, a, 0x06040200u);
        y[1][g] = __builtin_amdgcn_perm(b, a, 0x07050301u);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (i0 + r < N) *reinterpret_cast<u32x4_any*>(dst + r * (int64_t)N + at) = y[r];
  }
}

// Rows of a [BH][N][d] bf16 tensor: gather (out[k] = in[perm[k]]) or scatter (out[perm[k]] = in[k]); 16 bytes per lane.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4* __restrict__ in, const int32_t* __restrict__ perm, uint4* __restrict__ out,
                                                          int64_t N, int chunks, int64_t total, int inverse) {
  const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (bh, k, chunk)
  if (x >= total) return;
  const int ch = (int)(x % chunks);
  const int64_t k = (x / chunks) % N, bh = x / chunks / N;
  const int64_t p = min<int64_t>(max(perm[k], 0), N - 1);  // clamped: never a wild access
  const int64_t from = inverse ? k : p, to = inverse ? p : k;
  out[(bh * N + to) * chunks + ch] = in[(bh * N + from) * chunks + ch];
}

inline size_t round256(size_t n) { return (n + 255) / 256 * 256; }
struct RcmLayout {
  size_t bits, degree, parent, order, cand, keys, visited, walk, state, total;
  explicit RcmLayout(int64_t N) {
    const size_t W = (size_t)((N + 63) / 64);
    size_t o = 0;
    bits = o;
    o += round256((size_t)N * W * 8);
    degree = o;
    o += round256((size_t)N * 4);
    parent = o;
    o += round256((size_t)N * 4);
    order = o;
    o += round256((size_t)N * 4);
    cand = o;
    o += round256((size_t)N * 4);
    keys = o;
    o += round256((size_t)N * 8);
    visited = o;
    o += round256(W * 8);
    walk = o;  // 24 bytes a region of 8 words: the two records' counts and minima
    o += round256(W * 8);
    state = o;
    o += round256(2 * kStInts * 4);
    total = o;
  }
};

}  // namespace

extern "C" __attribute__((visibility("default"))) size_t bbm_rcm_workspace_bytes(int64_t N) {
  if (N < 1 || N > kMaxNodes) return 0;
  return RcmLayout(N).total;
}

extern "C" __attribute__((visibility("default"))) int bbm_rcm_order(const uint8_t* mask, int64_t N, int64_t row_stride_bytes, int32_t* perm,
                                                                   void* workspace, size_t workspace_bytes, void* stream) {
  using namespace bbm;
  clear_error();
  if (!mask || !perm) return fail(BBM_EINVAL, "bbm_rcm_order: mask and perm must not be NULL");
  if (N < 1) return fail(BBM_EINVAL, "bbm_rcm_order: N=%lld must be >= 1", (long long)N);
  if (N > kMaxNodes) return fail(BBM_EUNSUPPORTED, "bbm_rcm_order: N=%lld exceeds %d", (long long)N, kMaxNodes);
  if (row_stride_bytes < N) return fail(BBM_EINVAL, "bbm_rcm_order: row_stride_bytes=%lld < N=%lld", (long long)row_stride_bytes, (long long)N);
  if (!aligned(perm, 4)) return fail(BBM_EINVAL, "bbm_rcm_order: perm must be 4-byte aligned");
  const RcmLayout lay(N);
  if (!workspace || workspace_bytes < lay.total)
    return fail(BBM_EWORKSPACE, "bbm_rcm_order: workspace of %zu bytes needed, %zu given", lay.total, workspace ? workspace_bytes : (size_t)0);
  if (!aligned(workspace, 16)) return fail(BBM_EINVAL, "bbm_rcm_order: workspace must be 16-byte aligned");
  char* ws = static_cast<char*>(workspace);
  uint64_t* bits = reinterpret_cast<uint64_t*>(ws + lay.bits);
  int32_t* degree = reinterpret_cast<int32_t*>(ws + lay.degree);
  int32_t* parent = reinterpret_cast<int32_t*>(ws + lay.parent);
  int32_t* order = reinterpret_cast<int32_t*>(ws + lay.order);
  int32_t* cand = reinterpret_cast<int32_t*>(ws + lay.cand);
  uint64_t* keys = reinterpret_cast<uint64_t*>(ws + lay.keys);
  const int W = (int)ceil_div(N, 64);
  hipStream_t s = static_cast<hipStream_t>(stream);
  uint64_t* visited = reinterpret_cast<uint64_t*>(ws + lay.visited);
  const int regions = (int)ceil_div(W, kRegWords);
  uint64_t* const lowest = reinterpret_cast<uint64_t*>(ws + lay.walk);
  int32_t* const count = reinterpret_cast<int32_t*>(lowest + 2 * regions);
  int32_t* const state = reinterpret_cast<int32_t*>(ws + lay.state);
  // while the rounds last, the places of the nodes are kept where the finisher's order will be, the two lists where its candidates
  // and keys will be
  const WalkRecord rec[2] = {{state, count, lowest, reinterpret_cast<uint32_t*>(cand)},
                             {state + kStInts, count + regions, lowest + regions, reinterpret_cast<uint32_t*>(keys)}};
  rcm_pack_kernel<<<(unsigned)N, kPackThreads, 0, s>>>(mask, (int)N, row_stride_bytes, W, reinterpret_cast<uint16_t*>(bits), degree, parent);
  int rc = launch_status("bbm_rcm_order (pack)");
  if (rc != BBM_OK) return rc;
  // kRounds rounds of a level each; the finisher walks whatever is left.  Kernels that find the walk finished return at once.
  rcm_start_kernel<<<(unsigned)regions, kRegCols, 0, s>>>(degree, visited, rec[0], (int)N, W);
  const int rank_wgs = (int)std::min<int64_t>(kRankWGs, ceil_div(N, kLevelWaves));
  static_assert(kRounds % 2 == 0, "the finisher's record and list are those of the last round");
  for (int r = 0; r < kRounds; ++r)
    rcm_level_kernel<<<(unsigned)(regions + rank_wgs), kLevelThreads, 0, s>>>(bits, degree, visited, order, perm, rec[r & 1], rec[~r & 1], (int)N, W, regions);
  rc = launch_status("bbm_rcm_order (rounds)");
  if (rc != BBM_OK) return rc;
  rcm_finish_kernel<<<1, kOrderThreads, 0, s>>>(bits, degree, parent, order, cand, keys, visited, rec[0], (int)N, W, regions, perm);
  return launch_status("bbm_rcm_order");
}

extern "C" __attribute__((visibility("default"))) int bbm_permute_mask(const uint8_t* mask, int64_t Mb, int64_t N, int64_t row_stride_bytes,
                                                                      const int32_t* perm, uint8_t* out, void* stream) {
  using namespace bbm;
  clear_error();
  if (!mask || !perm || !out) return fail(BBM_EINVAL, "bbm_permute_mask: mask, perm, out must not be NULL");
  if (mask == out) return fail(BBM_EINVAL, "bbm_permute_mask: out must not be the input");
  if (Mb < 1 || N < 1) return fail(BBM_EINVAL, "bbm_permute_mask: Mb=%lld, N=%lld must be >= 1", (long long)Mb, (long long)N);
  if (N > kMaxNodes || Mb > 65535) return fail(BBM_EUNSUPPORTED, "bbm_permute_mask: N=%lld exceeds %d or Mb=%lld exceeds 65535", (long long)N, kMaxNodes, (long long)Mb);
  if (row_stride_bytes < N) return fail(BBM_EINVAL, "bbm_permute_mask: row_stride_bytes=%lld < N=%lld", (long long)row_stride_bytes, (long long)N);
  hipStream_t s = static_cast<hipStream_t>(stream);
  // a byte per lane / rows staged in LDS, us: 250^2 2.2 / 2.8, 512^2 2.3 / 2.7, 700^2 2.7 / 2.8, 1024^2 3.2 / 2.8
  if (N < 16 || Mb * N * N <= kSmallMaskBytes) {
    permute_small_mask_kernel<<<dim3((unsigned)ceil_div(N, 64), (unsigned)ceil_div(N, 4), (unsigned)Mb), 256, 0, s>>>(mask, (int)N, row_stride_bytes, perm, out);
    return launch_status("bbm_permute_mask");
  }
  // four rows a work-group as long as they fit the 160 KiB of LDS (up to 40960 columns), two up to kMaxNodes: see the kernel
  const size_t cols = (size_t)(N + 15) / 16 * 16;
  const unsigned threads = (unsigned)std::min<size_t>(1024, (cols / 16 + 63) / 64 * 64);
  if (4 * cols <= kLdsBytes)
    permute_mask_kernel<4><<<dim3((unsigned)ceil_div(N, 4), (unsigned)Mb), threads, 4 * cols, s>>>(mask, (int)N, row_stride_bytes, perm, out);
  else
    permute_mask_kernel<2><<<dim3((unsigned)ceil_div(N, 2), (unsigned)Mb), threads, 2 * cols, s>>>(mask, (int)N, row_stride_bytes, perm, out);
  return launch_status("bbm_permute_mask");
}

extern "C" __attribute__((visibility("default"))) int bbm_gather_rows(const void* in, const int32_t* perm, void* out, int64_t BH, int64_t N, int d,
                                                                     int inverse, void* stream) {
  using namespace bbm;
  clear_error();
  if (!in || !perm || !out) return fail(BBM_EINVAL, "bbm_gather_rows: in, perm, out must not be NULL");
  if (in == out) return fail(BBM_EINVAL, "bbm_gather_rows: out must not be the input");
  if (!aligned(in, 16) || !aligned(out, 16)) return fail(BBM_EINVAL, "bbm_gather_rows: in and out must be 16-byte aligned");
  if (BH < 1 || N < 1 || d < 8 || d % 8 != 0) return fail(BBM_EINVAL, "bbm_gather_rows: BH=%lld, N=%lld >= 1 and d=%d a multiple of 8 required", (long long)BH, (long long)N, d);
  const int chunks = d / 8;
  const int64_t total = BH * N * chunks;
  if (ceil_div(total, 256) >= (1ll << 31)) return fail(BBM_EUNSUPPORTED, "bbm_gather_rows: tensor too large");
  gather_rows_kernel<<<(unsigned)ceil_div(total, 256), 256, 0, static_cast<hipStream_t>(stream)>>>(
      static_cast<const uint4*>(in), perm, static_cast<uint4*>(out), N, chunks, total, inverse ? 1 : 0);
  return launch_status("bbm_gather_rows");
}
