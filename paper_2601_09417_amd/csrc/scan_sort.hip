// Stable LSD radix sorts (gfx950, wave64): one-sweep passes of 512-thread blocks, and one block of 1024 for few
// elements.
//
// One histogram kernel counts the digits of every pass in one read of the
// keys, then each pass is a single kernel over tiles of 8192 keys (4096 or 2048 for few keys) that ranks equal digits
// inside each wave with ballots (a lane's rank = set bits of its digit-match mask below it) and across a
// wave's rounds through per-wave LDS counters, learns the earlier tiles' digit counts by
// decoupled look-back, partitions the tile in LDS, and writes it out in digit order (coalesced
// runs).
#include <hip/hip_runtime.h>

#include <utility>

#include "block_scan.h"
#include "common.h"

namespace vbm {

namespace {

constexpr int kItems = 16;            // keys per thread of a pass over many keys
constexpr int kChunk = 256 * kItems;  // keys of a histogram block's step and of the smallest depth or pair tile

__device__ __forceinline__ bool aligned16(const void* p) {
  return (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
}

__device__ __forceinline__ int64_t active_count(int64_t n_max, const uint32_t* n_dev) {
  if (!n_dev) return n_max;
  int64_t n = static_cast<int64_t>(*n_dev);
  return n < n_max ? n : n_max;
}

__global__ __launch_bounds__(256) void k_clear_words(ClearList c) {
  const int64_t first = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
  for (int k = 0; k < c.count; ++k)
    for (int64_t i = first; i < c.n[k]; i += stride) c.p[k][i] = 0u;
}

// ------------------------------------------------------------------ radix sort
// One-sweep LSD radix sort (after Adinets and Garland's Onesweep, built on Merrill and Garland's
// decoupled look-back): one histogram kernel adds the digit counts of every pass into digit totals in a
// single read of the keys, and then every pass is one kernel.  A pass block ranks its tile's keys, publishes
// the tile's digit counts, and finds how many keys of each digit the earlier tiles
// hold by walking back over their published counts (a tile that has already found its own prefix
// publishes that, so the walk stops there).  No per-pass histogram or scan launch and no per-tile
// digit offsets in memory.
//
// A sparse sort begins from one key per element, 0 meaning absent: its first pass reads all of them, takes the
// element's index as the value and moves only the keys that are there, so a compaction before the sort (a
// scan of the flags and a scattered copy) is not needed; it also writes how many there are.
constexpr int kUpThreads = 512;       // histogram block
constexpr int kUpBlocksMax = 256;     // histogram grid: enough loads in flight to stream at the HBM rate
constexpr int kMaxPasses = 8;         // 32-bit keys with digits of at least 4 bits
constexpr uint32_t kFlagAgg = 1u << 30;   // status word: the tile's own count of the digit
constexpr uint32_t kFlagInc = 2u << 30;   // status word: the count in this tile and every earlier one
constexpr uint32_t kCountMask = kFlagAgg - 1u;
constexpr int kFallbackRounds = 128;  // look-back rounds that find a tile unpublished before counting it directly
constexpr int kLookback = 8;          // earlier tiles' status words read per look-back round
// Threads of a one-sweep pass block (kItems keys each in a large sort, so 8192-key tiles): at workload H the pass
// time per step was 0.435 ms with 4096-key tiles, 0.404 ms with 8192 and 0.461 ms with 16384 (one
// block per CU); fewer tiles shorten the look-back chain and lengthen each digit's output run.
constexpr int kSweepThreads = 512;

// Exclusive scan of one value per thread across a block of NT threads (NT a multiple of 64);
// block total in *total.  Every thread of the block must call it (it synchronises).
template <int NT, class T>
__device__ __forceinline__ T block_excl_scan_n(T v, T* total) {
  __shared__ T s_wave[NT / 64];
  const int w = threadIdx.x >> 6;
  T incl = wave_incl_scan(v);
  if (lane_id() == 63) s_wave[w] = incl;
  __syncthreads();
  T base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    T x = s_wave[i];
    if (i < w) base += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return base + incl - v;
}

__device__ __forceinline__ uint32_t status_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void status_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Keys of digit d in the full tile j of CH keys (the look-back's fallback for a tile whose block has
// not published its counts).
template <int CH, bool kSparse>
__device__ uint32_t count_digit(const uint32_t* __restrict__ kin, int64_t j, int shift, uint32_t mask, uint32_t d) {
  const uint32_t* src = kin + j * CH;
  uint32_t c = 0;
  for (int i = 0; i < CH; ++i) c += (!kSparse || src[i] != 0u) && ((src[i] >> shift) & mask) == d ? 1u : 0u;
  return c;
}

// Digit counts of every pass in one read of the keys.  Block b takes 4096-key chunks b, b + G, ...
// and adds its counts to tot[passes * 256] (cleared by an earlier kernel; at most 256 additions
// to an address); lane l adds into LDS copy l & 3, so equal digits within a wave (the top digits of clustered
// keys) contend four ways less.  The block also clears its share of the passes' look-back status words.
template <bool kSparse>
__global__ __launch_bounds__(kUpThreads) void k_radix_upsweep(const uint32_t* __restrict__ keys, int64_t n_max,
                                                              const uint32_t* n_dev, int end_bit, int digit_bits,
                                                              int passes, uint32_t* __restrict__ tot,
                                                              uint32_t* __restrict__ clear, int64_t clear_n) {
  __shared__ uint32_t s_h[4][kMaxPasses * 256];
  const int R = passes * 256;
  for (int i = threadIdx.x; i < 4 * R; i += kUpThreads) s_h[i / R][i % R] = 0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * kUpThreads + threadIdx.x; i < clear_n;
       i += static_cast<int64_t>(gridDim.x) * kUpThreads)
    clear[i] = 0u;
  __syncthreads();
  const int64_t n = active_count(n_max, n_dev);
  uint32_t* h = s_h[threadIdx.x & 3];
  constexpr int kPer = kChunk / kUpThreads;   // 8 keys per thread and chunk
  for (int64_t c = blockIdx.x; c * kChunk < n; c += gridDim.x) {
    const int64_t base = c * kChunk;
    uint32_t k[kPer];
    bool ok[kPer];
    if (base + kChunk <= n && aligned16(keys)) {
      // two 16-byte loads per thread, consecutive across the block
      const uint4* src = reinterpret_cast<const uint4*>(keys + base);
#pragma unroll
      for (int r = 0; r < kPer / 4; ++r) {
        const uint4 q = src[r * kUpThreads + threadIdx.x];
        k[4 * r] = q.x;
        k[4 * r + 1] = q.y;
        k[4 * r + 2] = q.z;
        k[4 * r + 3] = q.w;
      }
#pragma unroll
      for (int r = 0; r < kPer; ++r) ok[r] = !kSparse || k[r] != 0u;
    } else {
#pragma unroll
      for (int r = 0; r < kPer; ++r) {
        const int64_t i = base + r * kUpThreads + threadIdx.x;
        k[r] = i < n ? keys[i] : 0u;
        ok[r] = i < n && (!kSparse || k[r] != 0u);
      }
    }
    for (int p = 0; p < passes; ++p) {
      const int shift = p * digit_bits;
      const int bits = end_bit - shift < digit_bits ? end_bit - shift : digit_bits;
      const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
      for (int r = 0; r < kPer; ++r)
        if (ok[r]) atomicAdd(&h[p * 256 + ((k[r] >> shift) & mask)], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < R; i += kUpThreads) {
    const uint32_t c = (s_h[0][i] + s_h[1][i]) + (s_h[2][i] + s_h[3][i]);
    if (c) atomicAdd(&tot[i], c);
  }
}

// Coarse length key of a tile's list: the longest first, one step per 8 entries, lists of 2040 or more share
// the first (the longest list's own length goes to the forward's counters).
__device__ __forceinline__ uint32_t length_key(uint2 r) { return 255u - min(255u, (r.y - r.x) >> 3); }

// The length key below which a tile's list is composited by four waves: lists of kSplitLeast entries or more,
// and of pairs / share or more (TileLists says which shares).  No list where that is more than the 2040 entries up to
// which the keys tell lengths apart: from 4.2M pairs in the backward, from 16.7M in the forward of many tiles.
constexpr uint32_t kSplitLeast = 16;
__device__ __forceinline__ uint32_t split_key(uint32_t pairs, uint32_t share) {
  const uint32_t steps = max(kSplitLeast, pairs / share) >> 3;   // lists of 8 steps entries or more
  return steps > 255u ? 0u : 256u - steps;
}
// Of n such lists the number shared in the backward.
__device__ __forceinline__ uint32_t split_backward(uint32_t n, uint32_t pairs, uint32_t longest) {
  return n <= kSplitFew || longest >= pairs / kSplitUneven ? n : 0u;
}

// One stable pass over tiles of NT x I keys.  Wave w of a tile owns keys [64 I w, 64 I (w + 1))
// and ranks them in I rounds of 64 against its own LDS digit counters: a lane's rank among the
// round's equal digits comes from ballots, and the wave's LDS operations complete in issue order,
// so a round reads its digits' counters before its leaders advance them with no barrier in
// between.  The per-wave counts give the tile's digit counts (published for the later tiles) and
// per-wave bases; the look-back gives the keys of each digit in the earlier tiles; the tile is
// partitioned in LDS and written out in digit order, so consecutive lanes store to consecutive
// addresses of a digit's output run.  kSparse: the first pass of a sparse sort (see above).
// kRanges: the last pass of the pair sort.  Its input is in order of the lower digits, so the partitioned
// tile is in order of the whole key and equal keys are neighbours; their first and last places go
// to ranges[key] as (~first, last + 1), both by maximum from 0, since a key's run can span tiles.
// kOrder: the tile order's pass (sparse); it also writes the number of split tiles.
enum SweepKind { kPlainPass, kSparsePass, kRangesPass, kOrderPass };
// I: keys per thread.  16 move the most keys a second, but up to kSmallSweep keys such tiles are fewer than the CUs or
// hardly more, and a pass takes as long as a tile: us a pass with 16 / 8 / 4 (keys): 14.5 / 10.5 / 9 (about 100,000),
// 16.4 / 13.3 / 13.1 (360,000), 22 / 19.5 / 21.5 (1.1M), 25.3 / 25.3 / 28.6 (2.4M), 58 / 66 / 87 (7.9M).  The tile
// order's pass has at most some ten thousand keys: 12.4 / 8.1 / 6.4 for 8,160 tiles, 14.7 / 10.5 / 9.1 for 65,280.
constexpr int kSmallItems = 8, kOrderItems = 4;
constexpr int64_t kSmallSweep = 2 << 20;
template <int NT, int I, SweepKind kKind>
__global__ __launch_bounds__(NT) void k_radix_onesweep(const uint32_t* __restrict__ kin,
                                                       const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
                                                       uint32_t* __restrict__ vout,
                                                       const uint32_t* __restrict__ totals,
                                                       uint32_t* __restrict__ status, int64_t n_max,
                                                       const uint32_t* n_dev, int shift, int bits,
                                                       uint32_t* __restrict__ count_out, uint2* __restrict__ ranges,
                                                       TileLists lists) {
  constexpr bool kSparse = kKind == kSparsePass || kKind == kOrderPass, kRanges = kKind == kRangesPass;
  constexpr int CH = NT * I;          // keys per tile
  constexpr int NW = NT / 64;
  constexpr int kPerWave = CH / NW;
  __shared__ uint32_t s_key[CH];
  __shared__ uint32_t s_val[CH];
  __shared__ uint32_t s_cnt[NW][256];       // per-wave digit counts, then per-wave digit bases
  __shared__ uint32_t s_start[256];         // start of each digit in the partitioned tile
  __shared__ uint32_t s_glob[256];          // global start of this tile's run of each digit
  const int64_t n = active_count(n_max, n_dev);
  const int64_t tile = blockIdx.x;
  const int64_t base = tile * CH;
  if (base >= n) return;  // uniform per block; no tile waits on a later one
  for (int x = threadIdx.x; x < NW * 256; x += NT) (&s_cnt[0][0])[x] = 0;
  const int in_tile = static_cast<int>(min(static_cast<int64_t>(CH), n - base));
  int count = in_tile;   // keys to move
  const int radix = 1 << bits;
  const uint32_t mask = static_cast<uint32_t>(radix - 1);
  const int w = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  uint32_t keys[I];
  uint32_t vals[I];
#pragma unroll
  for (int r = 0; r < I; ++r) {
    const int li = w * kPerWave + r * 64 + lane;
    keys[r] = li < in_tile ? kin[base + li] : 0u;
    vals[r] = kSparse ? static_cast<uint32_t>(base + li) : li < in_tile ? vin[base + li] : 0u;
  }
  __syncthreads();
  uint32_t slot[I];   // rank among the wave's keys of the same digit
#pragma unroll
  for (int r = 0; r < I; ++r) {
    const bool valid = kSparse ? keys[r] != 0u : w * kPerWave + r * 64 + lane < in_tile;
    const uint32_t d = (keys[r] >> shift) & mask;
    uint64_t m = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      m &= bit ? bb : ~bb;
    }
    const uint32_t rank = popc_below(m);
    const uint32_t before = s_cnt[w][d];
    if (valid && rank == 0) s_cnt[w][d] = before + static_cast<uint32_t>(__popcll(m));
    slot[r] = before + rank;
  }
  __syncthreads();
  const bool has = static_cast<int>(threadIdx.x) < radix;
  const bool dig = threadIdx.x < 256;   // the threads that own a digit's bookkeeping
  {
    uint32_t c[NW], t = 0;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      c[ww] = dig ? s_cnt[ww][threadIdx.x] : 0u;
      t += c[ww];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan_n<NT>(t, &tot);
    if (kSparse) count = static_cast<int>(tot);
    if (dig) {
      s_start[threadIdx.x] = run;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        s_cnt[ww][threadIdx.x] = run;
        run += c[ww];
      }
    }
    // keys of lower digits in the whole input: the exclusive scan of the digit totals
    uint32_t all;
    const uint32_t below = block_excl_scan_n<NT>(has ? totals[threadIdx.x] : 0u, &all);
    if (kKind == kSparsePass && tile == 0 && threadIdx.x == 0) *count_out = all;
    if (kKind == kOrderPass && tile == 0) {
      uint32_t* counters = lists.counters;
      // tiles with a lower key are split
      const uint32_t n_split = min(below, static_cast<uint32_t>(kMaxSplit));
      if (threadIdx.x == split_key(counters[1], lists.split_fwd)) counters[kSplitCounter] = n_split;
      if (threadIdx.x == split_key(counters[1], lists.split_bwd))
        counters[kSplitCounter + 1] = split_backward(n_split, counters[1], counters[kLongestCounter]);
    }
    if (has) {
      uint32_t* mine = status + tile * radix + threadIdx.x;
      uint32_t excl = 0;
      if (tile == 0) {
        status_store(mine, kFlagInc | t);
      } else {
        status_store(mine, kFlagAgg | t);
        // Walk back over windows of kLookback earlier tiles, their status words read together
        // (one memory round trip per window rather than per tile): add the counts nearest
        // first until a tile that holds its inclusive count; a window that meets a tile that has
        // published nothing yet is read again from that tile.  Nothing here assumes that the
        // earlier tiles' blocks are running: after kFallbackRounds such rounds the thread counts
        // its digit in that tile's keys itself and walks on, so every wait ends.
        int64_t j = tile - 1;
        int rounds = 0;
        for (;;) {
          uint32_t v[kLookback];
#pragma unroll
          for (int k = 0; k < kLookback; ++k)
            v[k] = j - k >= 0 ? status_load(status + (j - k) * radix + threadIdx.x) : kFlagInc;
          int k = 0;
          bool done = false;
#pragma unroll
          for (int q = 0; q < kLookback; ++q) {
            if (!done && k == q) {
              if ((v[q] & ~kCountMask) == 0u) continue;   // not published yet: stop here
              excl += v[q] & kCountMask;
              done = (v[q] & kFlagInc) != 0u;
              k = q + 1;
            }
          }
          if (done) break;
          j -= k;
          if (k < kLookback) {
            if (++rounds > kFallbackRounds) {
              excl += count_digit<CH, kSparse>(kin, j, shift, mask, threadIdx.x);   // tile j < tile is full
              --j;
              rounds = 0;
            } else {
              __builtin_amdgcn_s_sleep(1);
            }
          }
        }
        status_store(mine, kFlagInc | (excl + t));
      }
      s_glob[threadIdx.x] = below + excl;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < I; ++r) {
    if (kSparse ? keys[r] != 0u : w * kPerWave + r * 64 + lane < in_tile) {
      const uint32_t pos = s_cnt[w][(keys[r] >> shift) & mask] + slot[r];
      s_key[pos] = keys[r];
      s_val[pos] = vals[r];
    }
  }
  __syncthreads();
  // write out in digit order
#pragma unroll
  for (int r = 0; r < I; ++r) {
    const int lp = r * NT + threadIdx.x;
    if (lp < count) {
      const uint32_t key = s_key[lp];
      const uint32_t d = (key >> shift) & mask;
      const uint32_t gp = s_glob[d] + (static_cast<uint32_t>(lp) - s_start[d]);
      kout[gp] = key;
      vout[gp] = s_val[lp];
      if (kRanges) {
        if (lp == 0 || s_key[lp - 1] != key) atomicMax(&ranges[key].x, ~gp);
        if (lp + 1 == count || s_key[lp + 1] != key) atomicMax(&ranges[key].y, gp + 1u);
      }
    }
  }
}

// ------------------------------------------------------------------ one-block sort
// Up to kBlockSort elements are sorted by one block in LDS, all passes in one launch: at these sizes a pass of the
// one-sweep sort is its launch and the latency of one tile (about 8 us), however few keys there are.
// 2,048 items and 2,079 pairs (64 tiles): sorts, ranges and tile order 75 us in 13 launches before, 24 us in two
// now.  The line: a render of 4,000 items and 6,787 pairs with room for 8,192 / 12,288 / 16,384 elements in the block
// takes 74 / 76 / 76 us, 8,000 and 13,625: 91 / 94 / 106, 10,000 and 16,968: 106 / 101 / 117, 16,384 and 27,803: 108 /
// 107 / 131.
constexpr int kBlockSortThreads = 1024;
constexpr int kBlockSortItems = static_cast<int>(kBlockSort / kBlockSortThreads);
constexpr int kBlockSortWaves = kBlockSortThreads / 64;

__device__ __forceinline__ void write_status(const uint32_t* __restrict__ counters, int32_t* __restrict__ status) {
  status[0] = static_cast<int32_t>(counters[2]);
  status[1] = static_cast<int32_t>(counters[1]);
  status[2] = static_cast<int32_t>(counters[0]);
  status[3] += counters[2] ? 1 : 0;
}

// Stable places of a block's elements by an 8-bit digit.  Element r of a lane is (wave * rounds + r) * 64 + lane;
// digit 256 or more: not there.  Afterwards slot[r] is its place, and the number of elements is returned.
__device__ __forceinline__ uint32_t block_places(const uint32_t (&digit)[kBlockSortItems], int rounds,
                                                 uint32_t (*__restrict__ s_cnt)[256],
                                                 uint32_t (&slot)[kBlockSortItems]) {
  const int w = threadIdx.x >> 6;
  // a wave's own counts, which no other has touched since the last barrier
  reinterpret_cast<uint4*>(s_cnt[w])[lane_id()] = make_uint4(0u, 0u, 0u, 0u);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int r = 0; r < kBlockSortItems; ++r) {
    if (r >= rounds) break;
    const uint32_t d = digit[r];
    const bool valid = d < 256u;
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      m &= bit ? bb : ~bb;
    }
    const uint32_t rank = popc_below(m);
    const uint32_t before = s_cnt[w][d & 255u];
    if (valid && rank == 0) s_cnt[w][d] = before + static_cast<uint32_t>(__popcll(m));
    slot[r] = before + rank;
  }
  __syncthreads();
  uint32_t c[kBlockSortWaves], t = 0;
#pragma unroll
  for (int ww = 0; ww < kBlockSortWaves; ++ww) {
    c[ww] = threadIdx.x < 256 ? s_cnt[ww][threadIdx.x] : 0u;
    t += c[ww];
  }
  uint32_t total;
  uint32_t run = block_excl_scan_n<kBlockSortThreads>(t, &total);
  if (threadIdx.x < 256) {
#pragma unroll
    for (int ww = 0; ww < kBlockSortWaves; ++ww) {
      s_cnt[ww][threadIdx.x] = run;
      run += c[ww];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kBlockSortItems; ++r) {
    if (r >= rounds) break;
    slot[r] += s_cnt[w][digit[r] & 255u];
  }
  return total;
}

// OR over the wave's lanes, by all of them.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr by 1, 2, 4, 8, then the rows' last lanes
  v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  return __builtin_amdgcn_readlane(v, 15) | __builtin_amdgcn_readlane(v, 31) | __builtin_amdgcn_readlane(v, 47) |
         __builtin_amdgcn_readlane(v, 63);
}

// Maximum over the wave's lanes, by all of them.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true)));   // as in wave_or
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true)));
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true)));
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true)));
  const uint32_t a = __builtin_amdgcn_readlane(v, 15), b = __builtin_amdgcn_readlane(v, 31);
  const uint32_t c = __builtin_amdgcn_readlane(v, 47), d = __builtin_amdgcn_readlane(v, 63);
  return max(max(a, b), max(c, d));
}

// kSparse: the depth sort (see radix_sort_sparse).  kPairs: the pair sort with what follows it, the
// tiles' ranges (cleared beforehand), launch order and the caller's status.  The output may be the input.
template <bool kSparse, bool kPairs>
__global__ __launch_bounds__(kBlockSortThreads) void k_sort_block(const uint32_t* kin, const uint32_t* vin,
                                                                  uint32_t* kout, uint32_t* vout, int64_t n_max,
                                                                  const uint32_t* n_dev, int end_bit,
                                                                  uint32_t* __restrict__ count_out, TileLists lists) {
  __shared__ uint32_t s_key[kBlockSort];
  __shared__ uint32_t s_val[kBlockSort];
  __shared__ uint32_t s_cnt[kBlockSortWaves][256];   // per-wave digit counts, then per-wave digit bases
  __shared__ uint2 s_bits[kBlockSortWaves];          // kSparse: the bits in which keys differ; kPairs: longest list (x)
  int n = static_cast<int>(active_count(n_max, n_dev));
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t keys[kBlockSortItems], vals[kBlockSortItems], digit[kBlockSortItems], slot[kBlockSortItems];
  // wave w owns elements [64 rounds w, 64 rounds (w + 1))
  int rounds = (n + kBlockSortThreads - 1) / kBlockSortThreads;
#pragma unroll
  for (int r = 0; r < kBlockSortItems; ++r) {
    const int i = (w * rounds + r) * 64 + lane;
    const bool in = r < rounds && i < n;
    keys[r] = in ? kin[i] : 0u;
    vals[r] = kSparse ? static_cast<uint32_t>(i) : in ? vin[i] : 0u;
  }
  int shift0 = 0;
  if (kSparse) {
    // Only the bits in which the keys differ are sorted by: a scene's depths share most of their exponent, so that a
    // pass of four is saved.  At least one pass leaves the absent ones behind.
    uint32_t ones = 0, zeros = 0;
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r) {
      ones |= keys[r];
      zeros |= keys[r] ? ~keys[r] : 0u;
    }
    ones = wave_or(ones);
    zeros = wave_or(zeros);
    if (lane == 0) s_bits[w] = make_uint2(ones, zeros);
    __syncthreads();
    const uint2 b = s_bits[lane % kBlockSortWaves];
    const uint32_t differ = wave_or(b.x) & wave_or(b.y);
    end_bit = min(end_bit, differ ? 32 - __builtin_clz(differ) : 1);
    shift0 = min(differ ? __builtin_ctz(differ) : 0, end_bit - 1);
  }
  for (int shift = shift0; shift < end_bit; shift += 8) {
    const uint32_t mask = (1u << min(8, end_bit - shift)) - 1u;
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r) {
      const bool valid = (w * rounds + r) * 64 + lane < n && (!kSparse || keys[r] != 0u);
      digit[r] = valid ? (keys[r] >> shift) & mask : 256u;
    }
    const int total = static_cast<int>(block_places(digit, rounds, s_cnt, slot));
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r) {
      if (r >= rounds) break;
      if (digit[r] < 256u) {
        s_key[slot[r]] = keys[r];
        s_val[slot[r]] = vals[r];
      }
    }
    __syncthreads();
    n = total;   // (a sparse sort's first pass leaves the absent ones behind)
    rounds = (n + kBlockSortThreads - 1) / kBlockSortThreads;
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r) {
      if (r >= rounds) break;
      const int i = (w * rounds + r) * 64 + lane;
      keys[r] = i < n ? s_key[i] : 0u;
      vals[r] = i < n ? s_val[i] : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < kBlockSortItems; ++r) {
    if (r >= rounds) break;
    const int i = (w * rounds + r) * 64 + lane;
    if (i >= n) continue;
    kout[i] = keys[r];
    vout[i] = vals[r];
  }
  if (kSparse && threadIdx.x == 0) *count_out = static_cast<uint32_t>(n);
  if (kPairs) {
    // The runs' ends through LDS, in the sorted keys' and values' place (there are at most as many tiles).
    uint32_t first = 0, last = 0;   // a bit per round
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r) {
      const int i = (w * rounds + r) * 64 + lane;
      if (r >= rounds || i >= n) continue;   // (a batch of one tile has no digits and one run)
      first |= (i == 0 || (end_bit != 0 && s_key[i - 1] != keys[r]) ? 1u : 0u) << r;
      last |= (i + 1 == n || (end_bit != 0 && s_key[i + 1] != keys[r]) ? 1u : 0u) << r;
    }
    const int tiles = static_cast<int>(lists.n_tiles);
    __syncthreads();
    for (int t = threadIdx.x; t < tiles; t += kBlockSortThreads) s_key[t] = s_val[t] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r) {
      const uint32_t i = static_cast<uint32_t>((w * rounds + r) * 64 + lane);
      if ((first >> r) & 1u) s_key[keys[r]] = i;
      if ((last >> r) & 1u) s_val[keys[r]] = i + 1u;
    }
    __syncthreads();
    rounds = (tiles + kBlockSortThreads - 1) / kBlockSortThreads;
    uint32_t longest = 0;
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r) {
      const int i = (w * rounds + r) * 64 + lane;
      digit[r] = 256u;
      if (r < rounds && i < tiles) {
        const uint2 range = make_uint2(s_key[i], s_val[i]);
        lists.ranges[i] = range;
        digit[r] = length_key(range);
        longest = max(longest, range.y - range.x);
      }
    }
    longest = wave_max(longest);
    if (lane == 0) s_bits[w].x = longest;
    block_places(digit, rounds, s_cnt, slot);
#pragma unroll
    for (int r = 0; r < kBlockSortItems; ++r)
      if (r < rounds && digit[r] < 256u) lists.order[slot[r]] = static_cast<uint32_t>((w * rounds + r) * 64 + lane);
    if (threadIdx.x == 0) {
      // the first wave's base of a length key is the key's: the tiles with a lower one
      const uint32_t pairs = lists.counters[1], most = kMaxSplit;
      for (int ww = 1; ww < kBlockSortWaves; ++ww) longest = max(longest, s_bits[ww].x);
      lists.counters[kLongestCounter] = longest;
      lists.counters[kSplitCounter] = min(s_cnt[0][split_key(pairs, lists.split_fwd)], most);
      lists.counters[kSplitCounter + 1] =
          split_backward(min(s_cnt[0][split_key(pairs, lists.split_bwd)], most), pairs, longest);
      write_status(lists.counters, lists.status);
    }
  }
}

// Tile order of larger batches: this kernel turns the last sort pass's (~first, last + 1) into ranges (an
// untouched tile keeps (0, 0)), writes each tile's length key with bit 8 set and their counts and the longest list's
// length, and clears the look-back words of the sparse sort pass that follows; block 0 writes the caller's status.
__global__ __launch_bounds__(256) void k_tile_keys(TileLists lists, int64_t capacity, int one_tile,
                                                   uint32_t* __restrict__ keys, uint32_t* __restrict__ hist,
                                                   uint32_t* __restrict__ clear, int64_t clear_n) {
  __shared__ uint32_t s_hist[256];
  __shared__ uint32_t s_longest[4];
  s_hist[threadIdx.x] = 0u;
  __syncthreads();
  uint32_t longest = 0;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  for (int64_t i = t; i < clear_n; i += static_cast<int64_t>(gridDim.x) * 256) clear[i] = 0u;
  if (t < lists.n_tiles) {
    uint2 r = lists.ranges[t];
    if (one_tile) {   // nothing was sorted
      r = make_uint2(0u, static_cast<uint32_t>(min(static_cast<int64_t>(lists.counters[1]), capacity)));
    } else {
      r.x = r.y ? ~r.x : 0u;
    }
    lists.ranges[t] = r;
    const uint32_t key = length_key(r);
    keys[t] = key | 256u;
    atomicAdd(&s_hist[key], 1u);
    longest = r.y - r.x;
  }
  longest = wave_max(longest);
  if (lane_id() == 0) s_longest[threadIdx.x >> 6] = longest;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(&lists.counters[kLongestCounter], max(max(s_longest[0], s_longest[1]), max(s_longest[2], s_longest[3])));
  if (s_hist[threadIdx.x]) atomicAdd(&hist[threadIdx.x], s_hist[threadIdx.x]);
  if (t == 0) write_status(lists.counters, lists.status);
}

}  // namespace

vbm_status clear_words(const ClearList& c, hipStream_t s) {
  int64_t most = 1;
  for (int k = 0; k < c.count; ++k) most = c.n[k] > most ? c.n[k] : most;
  const int64_t blocks = ceil_div(most, 256 * 4);
  hipLaunchKernelGGL(k_clear_words, dim3(blocks < 1024 ? blocks : 1024), dim3(256), 0, s, c);
  VBM_LAUNCH_CHECK("clear_words");
  return VBM_OK;
}

namespace {
// Scratch of one sort: a head of kRadixHead bytes that the sort leaves alone (the renderer keeps the tile-order
// counts there), digit totals, then the look-back status words of every pass, which the histogram kernel clears.
struct RadixLayout {
  int64_t nb;        // 4096-key tiles (status words are sized for them, twice what a pass over tiles of 8192 uses)
  int passes_max;    // passes of a 32-bit key
  int radix;         // 1 << digit width
  int G;             // histogram blocks
  size_t off_tot, off_status, bytes;
};

RadixLayout radix_layout(int64_t n_max, int digit_bits) {
  RadixLayout L;
  L.nb = ceil_div(n_max > 0 ? n_max : 1, kChunk);
  L.passes_max = static_cast<int>(ceil_div(32, digit_bits));
  L.radix = 1 << digit_bits;
  L.G = static_cast<int>(L.nb < kUpBlocksMax ? L.nb : kUpBlocksMax);
  L.off_tot = kRadixHead;
  L.off_status = align_up(L.off_tot + static_cast<size_t>(L.passes_max) * 256 * 4, 256);
  L.bytes = align_up(L.off_status + static_cast<size_t>(L.passes_max) * L.nb * L.radix * 4, 256);
  return L;
}

vbm_status check_digits(int end_bit, int digit_bits) {
  if (digit_bits < 4 || digit_bits > 8) {
    set_error("radix digit width %d outside 4..8", digit_bits);
    return VBM_ERR_INVALID;
  }
  if (end_bit > 32) {
    set_error("radix sort over %d key bits (at most 32)", end_bit);
    return VBM_ERR_INVALID;
  }
  return VBM_OK;
}

// Passes first .. passes - 1 of a sort whose histogram has run, ping-ponging from (k0, v0); with ranges, the
// last one also records the runs of equal keys.
vbm_status sweep(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, int64_t n_max, const uint32_t* n_dev,
                 int end_bit, int digit_bits, int first, const RadixLayout& L, char* scratch, uint2* ranges,
                 hipStream_t s) {
  uint32_t* tot = reinterpret_cast<uint32_t*>(scratch + L.off_tot);
  uint32_t* status = reinterpret_cast<uint32_t*>(scratch + L.off_status);
  const int passes = static_cast<int>(ceil_div(end_bit, digit_bits));
  const bool small = n_max <= kSmallSweep;
  const dim3 grid(static_cast<unsigned>(ceil_div(n_max, kSweepThreads * (small ? kSmallItems : kItems))));
  for (int p = first; p < passes; ++p) {
    const int shift = p * digit_bits;
    const int bits = (end_bit - shift) < digit_bits ? (end_bit - shift) : digit_bits;
    auto launch = [&](auto kernel, uint2* r) {
      hipLaunchKernelGGL(kernel, grid, dim3(kSweepThreads), 0, s, k0, v0, k1, v1, tot + p * 256,
                         status + p * L.nb * L.radix, n_max, n_dev, shift, bits, static_cast<uint32_t*>(nullptr), r,
                         TileLists());
    };
    if (ranges && p == passes - 1)
      launch(small ? k_radix_onesweep<kSweepThreads, kSmallItems, kRangesPass>
                   : k_radix_onesweep<kSweepThreads, kItems, kRangesPass>, ranges);
    else
      launch(small ? k_radix_onesweep<kSweepThreads, kSmallItems, kPlainPass>
                   : k_radix_onesweep<kSweepThreads, kItems, kPlainPass>, static_cast<uint2*>(nullptr));
    VBM_LAUNCH_CHECK("radix_onesweep");
    std::swap(k0, k1);
    std::swap(v0, v1);
  }
  return VBM_OK;
}
}  // namespace

size_t radix_scratch_bytes(int64_t n_max, int digit_bits) {
  if (digit_bits < 4) digit_bits = 4;
  return radix_layout(n_max, digit_bits).bytes;
}

uint32_t* radix_totals(int64_t n_max, int digit_bits, void* scratch) {
  return reinterpret_cast<uint32_t*>(static_cast<char*>(scratch) + radix_layout(n_max, digit_bits).off_tot);
}

vbm_status radix_sort_sparse(const uint32_t* keys, int64_t n, uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1,
                             int end_bit, int digit_bits, uint32_t* count_dev, void* scratch, hipStream_t s) {
  if (n <= 0 || end_bit <= 0) return VBM_OK;
  VBM_TRY(check_digits(end_bit, digit_bits));
  const int passes = static_cast<int>(ceil_div(end_bit, digit_bits));
  if (n <= kBlockSort) {
    hipLaunchKernelGGL((k_sort_block<true, false>), dim3(1), dim3(kBlockSortThreads), 0, s, keys,
                       static_cast<const uint32_t*>(nullptr), passes % 2 ? k0 : k1, passes % 2 ? v0 : v1, n,
                       static_cast<const uint32_t*>(nullptr), end_bit, count_dev, TileLists());
    VBM_LAUNCH_CHECK("sort_block");
    return VBM_OK;
  }
  const RadixLayout L = radix_layout(n, digit_bits);
  char* base = static_cast<char*>(scratch);
  uint32_t* tot = reinterpret_cast<uint32_t*>(base + L.off_tot);
  uint32_t* status = reinterpret_cast<uint32_t*>(base + L.off_status);
  hipLaunchKernelGGL(k_radix_upsweep<true>, dim3(L.G), dim3(kUpThreads), 0, s, keys, n,
                     static_cast<const uint32_t*>(nullptr), end_bit, digit_bits, passes, tot, status,
                     static_cast<int64_t>(passes) * L.nb * L.radix);
  VBM_LAUNCH_CHECK("radix_upsweep");
  const bool small = n <= kSmallSweep;
  hipLaunchKernelGGL((small ? k_radix_onesweep<kSweepThreads, kSmallItems, kSparsePass>
                            : k_radix_onesweep<kSweepThreads, kItems, kSparsePass>),
                     dim3(ceil_div(n, kSweepThreads * (small ? kSmallItems : kItems))), dim3(kSweepThreads), 0, s, keys,
                     static_cast<const uint32_t*>(nullptr), k0, v0, tot, status, n,
                     static_cast<const uint32_t*>(nullptr), 0, end_bit < digit_bits ? end_bit : digit_bits, count_dev,
                     static_cast<uint2*>(nullptr), TileLists());
  VBM_LAUNCH_CHECK("radix_onesweep");
  return sweep(k0, v0, k1, v1, n, count_dev, end_bit, digit_bits, 1, L, base, nullptr, s);
}

int sort_pairs_first(int64_t n_max, int64_t n_tiles, int end_bit, int digit_bits) {
  if (n_max <= kBlockSort && n_tiles <= kBlockSort) return 0;
  return static_cast<int>(ceil_div(end_bit, digit_bits)) % 2;
}

vbm_status sort_pairs_by_tile(uint32_t* const k[2], uint32_t* const v[2], int first, int64_t capacity, int64_t n_max,
                              const uint32_t* n_dev, int end_bit, int digit_bits, const TileLists& lists,
                              void* scratch, hipStream_t s) {
  if (n_max > 0 && n_max <= kBlockSort && lists.n_tiles <= kBlockSort) {
    hipLaunchKernelGGL((k_sort_block<false, true>), dim3(1), dim3(kBlockSortThreads), 0, s, k[first], v[first], k[0],
                       v[0], n_max, n_dev, end_bit, static_cast<uint32_t*>(nullptr), lists);
    VBM_LAUNCH_CHECK("sort_block");
    return VBM_OK;
  }
  if (n_max > 0 && end_bit > 0) {
    VBM_TRY(check_digits(end_bit, digit_bits));
    const RadixLayout L = radix_layout(n_max, digit_bits);
    char* base = static_cast<char*>(scratch);
    const int passes = static_cast<int>(ceil_div(end_bit, digit_bits));
    hipLaunchKernelGGL(k_radix_upsweep<false>, dim3(L.G), dim3(kUpThreads), 0, s, k[first], n_max, n_dev, end_bit,
                       digit_bits, passes, reinterpret_cast<uint32_t*>(base + L.off_tot),
                       reinterpret_cast<uint32_t*>(base + L.off_status),
                       static_cast<int64_t>(passes) * L.nb * L.radix);
    VBM_LAUNCH_CHECK("radix_upsweep");
    VBM_TRY(sweep(k[first], v[first], k[1 - first], v[1 - first], n_max, n_dev, end_bit, digit_bits, 0, L, base,
                  lists.ranges, s));
  }
  // The pair sort's scratch is free again: the order's look-back words take its place.
  const int64_t NT = lists.n_tiles;
  const RadixLayout L = radix_layout(NT, 8);
  uint32_t* hist = tile_order_counts(scratch);
  uint32_t* look = reinterpret_cast<uint32_t*>(static_cast<char*>(scratch) + L.off_status);
  hipLaunchKernelGGL(k_tile_keys, dim3(static_cast<unsigned>(ceil_div(NT, 256))), dim3(256), 0, s, lists, capacity,
                     end_bit == 0 ? 1 : 0, lists.keys, hist, look, ceil_div(NT, kSweepThreads * kOrderItems) * L.radix);
  VBM_LAUNCH_CHECK("tile_keys");
  hipLaunchKernelGGL((k_radix_onesweep<kSweepThreads, kOrderItems, kOrderPass>),
                     dim3(static_cast<unsigned>(ceil_div(NT, kSweepThreads * kOrderItems))), dim3(kSweepThreads), 0, s,
                     lists.keys, static_cast<const uint32_t*>(nullptr), lists.keys + NT, lists.order, hist, look, NT,
                     static_cast<const uint32_t*>(nullptr), 0, 8, static_cast<uint32_t*>(nullptr),
                     static_cast<uint2*>(nullptr), lists);
  VBM_LAUNCH_CHECK("tile_order");
  return VBM_OK;
}

}  // namespace vbm
