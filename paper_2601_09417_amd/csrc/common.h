// Internal declarations shared by the libvbm translation units (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "../../include/vbm.h"

namespace vbm {

// ------------------------------------------------------------------ errors
void set_error(const char* fmt, ...);
vbm_status hip_check(hipError_t e, const char* what);
#define VBM_LAUNCH_CHECK(name)                                         \
  do {                                                                 \
    hipError_t _e = hipGetLastError();                                 \
    if (_e != hipSuccess) return ::vbm::hip_check(_e, name);           \
  } while (0)
#define VBM_TRY(expr)                                                  \
  do {                                                                 \
    vbm_status _s = (expr);                                            \
    if (_s != VBM_OK) return _s;                                       \
  } while (0)

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Bump allocator over a caller-provided workspace (sizing pass when base == nullptr).
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base(static_cast<char*>(b)) {}
  template <class T>
  T* take(size_t count) {
    off = align_up(off, 256);
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

// ------------------------------------------------------------------ device view table
// One record per view, written by vbm_plan_make on the host and read by every render kernel.
struct DevView {
  float R[9];            // world->camera rotation, row-major
  float t[3];
  float fx, fy, cx, cy;
  float near_plane;
  float bg[3];
  int32_t width, height, tiles_x, tiles_y;
  int32_t item_offset;   // first item of this view
  int32_t gauss_offset;  // first Gaussian of the view's scene
  int32_t n_gauss;       // Gaussians in the view's scene
  int32_t tile_offset;   // first global tile of this view
  int32_t pixel_offset;  // first pixel of this view
  int32_t scene;
  float lim_x, lim_y;    // FOV clamp of the projection Jacobian: 1.3 (0.5 W / fx), 1.3 (0.5 H / fy) in float32
};
static_assert(sizeof(DevView) % 16 == 0, "DevView must stay 16-byte aligned");

// Scene table appended after the views in the device view table.
struct DevScene {
  int32_t gauss_offset, n_gauss;
};

// ------------------------------------------------------------------ limits
constexpr int kMaxViewSide = 16384;                                             // pixels; checked by the plan
constexpr int64_t kMaxRectTiles = int64_t{kMaxViewSide / 8} * (kMaxViewSide / 8);   // of a footprint, with 8x8 tiles

// ------------------------------------------------------------------ pair values
// A pair value holds the item id in bits 0..26 (the plan keeps items below 2^27) and a 4-bit mask
// of the tile's lane groups in bits 27..30.  With 16x16 tiles lane group k is pixel rows
// 4k .. 4k + 3 of the tile.  The emission sets the groups whose rows the footprint can reach (all four
// with other tiles), and the forward's marked copy the groups of which it can reach a pixel.
constexpr int kItemBits = 27;
constexpr uint32_t kItemMask = (1u << kItemBits) - 1u;

// ------------------------------------------------------------------ wave helpers
__device__ __forceinline__ uint32_t lane_id() {
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
// Number of set bits of `mask` in lanes below the calling lane.
__device__ __forceinline__ uint32_t popc_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// ------------------------------------------------------------------ arithmetic
// Correctly rounded float32 square root: the square root of the value in float64, rounded to
// float32.  Rounding twice cannot go wrong here because 53 >= 2 * 24 + 2 (the float64 result,
// even one unit off in its last place, never crosses a float32 rounding boundary); the float32
// square-root instruction alone is only accurate to one unit in the last place.
__device__ __forceinline__ float sqrt_rn_f32(float x) {
  return static_cast<float>(__dsqrt_rn(static_cast<double>(x)));
}

// ------------------------------------------------------------------ sort primitives (scan_sort.hip)
// Stable LSD radix sorts of (key, value) pairs over key bits [0, end_bit) (end_bit <= 32), digit
// width 4..8 bits.  The caller clears the kMaxRadixTotals words at radix_totals() beforehand.  The first
// kRadixHead bytes of the scratch are not the sorts': tile_order_counts() lies there.
constexpr size_t kRadixHead = 4096;
constexpr int kMaxRadixTotals = 8 * 256;    // any sort
constexpr int kMaxDepthTotals = 4 * 256;    // 8-bit digits
constexpr int64_t kBlockSort = 8192;        // elements that one block sorts in LDS
size_t radix_scratch_bytes(int64_t n_max, int digit_bits);
uint32_t* radix_totals(int64_t n_max, int digit_bits, void* scratch);
// The elements i in [0, n) with keys[i] != 0, each with value i; ceil(end_bit / width) passes write (k0, v0) and
// (k1, v1) in turn, so the sorted data ends in the first for an odd number of passes; *count_dev
// receives the number of elements.
vbm_status radix_sort_sparse(const uint32_t* keys, int64_t n, uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1,
                             int end_bit, int digit_bits, uint32_t* count_dev, void* scratch, hipStream_t s);

// Tiles whose lists are composited by four waves each, a band of four pixel rows per wave (16x16 tiles, longest
// lists first).  A launch takes at least as long as its longest list takes one wave, and a batch of few tiles does
// not fill the chip with one wave each; in a batch of many tiles four waves only cost more (the list is staged and
// read four times).
//   Forward: every list in batches of up to kSplitAllTiles tiles, else lists of pairs / 8192 entries or more.
//     us with a wave per list / every list shared (tiles, pairs): 600 / 270 (8,400, 3.4M), 437 / 203 (8,160, 2.4M),
//     499 / 388 (16,320, 4.9M), 668 / 917 (32,640, 9.8M), 533 / 772 (40,000, 7.9M).
//   Backward (its sums over a band cost as much as over a tile): lists of pairs / 2048 entries or more.  us with a wave
//     per list / this rule / pairs / 4096: 773 / 695 / 882 (8,400 tiles, 3.4M pairs), 210 / 141 / 138 (2,400, 0.6M),
//     829 / 751 / 887 (12,544, 4.0M), 115 / 69 / 69 (600, 0.1M).
//     None where that is more than kSplitFew lists and the longest is below pairs / kSplitUneven: most of the pairs are
//     then shared, and the chip was full without.  us with a wave per list / shared (pairs over the longest list, lists
//     shared): 134 / 151 (1187, 1089), 247 / 279 (1247, 1089), 214 / 233 (864, 948), 269 / 280 (1322, 608), but
//     364 / 325 (673, 856), 109 / 74 (677, 890), 167 / 135 (493, 672), 759 / 687 (1806, 107).
constexpr int kMaxSplit = 20480;        // at most
constexpr int kSplitAllTiles = 20480;
constexpr uint32_t kSplitForward = 8192, kSplitBackward = 2048;
constexpr uint32_t kSplitFew = 256, kSplitUneven = 700;
constexpr int kSplitCounter = 6;        // their numbers for the forward and the backward, among the forward's counters
constexpr int kLongestCounter = 8;      // entries of the longest list, among the same

// The tiles' lists after the pair sort.
struct TileLists {
  uint2* ranges;             // [n_tiles]: [start, end) of each tile's list
  int64_t n_tiles;
  uint32_t* order;           // [n_tiles]: tiles in launch order, longest lists first (in steps of 8 entries, stable)
  uint32_t* keys;            // [2][n_tiles]: the order's sort keys
  uint32_t* counters;        // of the forward: the numbers of split tiles go to [6] and [7], the longest list's to [8]
  int32_t* status;           // the caller's
  uint32_t split_fwd, split_bwd;   // shares of split_key
};
// Sorts the pairs in (k[first], v[first]) by tile into (k[0], v[0]) (first as sort_pairs_first says; the count is
// read from *n_dev when non-null, and is at most n_max), and writes the tiles' ranges (cleared beforehand),
// launch order and the status (scratch: radix_scratch_bytes of n_max and of the tiles).  The kTileOrderCounts words at
// tile_order_counts() are cleared beforehand.
constexpr int kTileOrderCounts = 256;
inline uint32_t* tile_order_counts(void* scratch) { return static_cast<uint32_t*>(scratch); }
int sort_pairs_first(int64_t n_max, int64_t n_tiles, int end_bit, int digit_bits);
vbm_status sort_pairs_by_tile(uint32_t* const k[2], uint32_t* const v[2], int first, int64_t capacity, int64_t n_max,
                              const uint32_t* n_dev, int end_bit, int digit_bits, const TileLists& lists,
                              void* scratch, hipStream_t s);

// Several runs of 32-bit words cleared by one launch (used instead of memset nodes so that every step stays
// capturable).
struct ClearList {
  static constexpr int kMax = 6;
  uint32_t* p[kMax];
  int64_t n[kMax];
  int count = 0;
  void add(void* q, int64_t words) {
    p[count] = static_cast<uint32_t*>(q);
    n[count] = words;
    ++count;
  }
};
vbm_status clear_words(const ClearList& c, hipStream_t s);

}  // namespace vbm
