// vbm_dwt3d: transfer function + periodised separable J-level 3D DWT (Sec. 3; Sec. 4.3,
// eq. mul_wavelet_coff).
//
// One kernel per level reads the current n^3 approximation once (at level 1 the scalar field, with
// the transfer function applied once per voxel read) and writes the seven detail octants straight into the
// packed subband layout and LLL into the next level's input.  The three separable filters (x, then y,
// then z) run inside the block, so nothing between them goes through memory:
//   bior4.4  a block owns a column of 64 x 16 voxels (64 x 4 in small levels) and marches along z: a
//            plane's tile with its halo goes to LDS, is filtered along x (LDS to LDS) and along y (LDS
//            to registers), and each thread keeps the running z sums of its (x, y) outputs in registers.
//   Haar     no halo: a thread owns a 2x2x2 cell.
#include <hip/hip_runtime.h>

#include <cstring>
#include <type_traits>

#include "common.h"
#include "filters.h"
#include "tf.h"

namespace vbm {
namespace {

// ------------------------------------------------------------------ transfer function in LDS
// RGBA by linear interpolation between ascending control points, constant beyond the end points
// (Sec. 3, Transfer Function).  Segment table: entry 0 is the constant before the first control point, entry i the
// segment between points i - 1 and i, entry n the constant from the last point on.  A lane's segment index varies, so
// the table is read from LDS (three 16-byte reads) rather than from the kernel arguments.
constexpr int kTfEntries = VBM_TF_MAX_POINTS + 1;

// What the first level reads: RGBA, or a scalar field through the transfer function.  A position in a segment is the
// product with the width's reciprocal, or the quotient where some width has none to work with (tf_form).
enum Input { kRGBA, kTF, kTFDivide };
struct TfSegment {
  float x0, w, inv_w, pad;   // inv_w = 1 / w rounded (kTFDivide: any), 0 where the position is not used (t = 1)
  float base[4];
  float delta[4];
};

// Fills the table (every thread of the block calls it; the caller synchronises).
template <Input kInput>
__device__ __forceinline__ void tf_load(const DevTF& tf, TfSegment* __restrict__ s, int threads) {
  for (int e = threadIdx.x; e <= tf.n; e += threads) {
    const int a = e == 0 ? 0 : e - 1, b = e == 0 || e == tf.n ? a : e;
    TfSegment q;
    q.x0 = tf.x[a];
    q.w = tf.x[b] - tf.x[a];
    q.inv_w = !(q.w > 0.0f) ? 0.0f : kInput == kTFDivide ? 1.0f : __fdiv_rn(1.0f, q.w);
    q.pad = 0.0f;
    for (int c = 0; c < 4; ++c) {
      // t = 1 in an entry without a position: a constant entry keeps its point (delta 0, an infinite one too), a
      // segment of no width takes its end
      q.base[c] = tf.rgba[a][c];
      q.delta[c] = a == b ? 0.0f : tf.rgba[b][c] - tf.rgba[a][c];
    }
    s[e] = q;
  }
}

// The table entries of N values: 0 at or below the first point, n at or above the last, else the
// last segment that begins at or below the value.
template <int N>
__device__ __forceinline__ void tf_find(const DevTF& tf, const float (&f)[N], int (&e)[N]) {
  const int n = tf.n;
#pragma unroll
  for (int k = 0; k < N; ++k) e[k] = 1;
  for (int i = 1; i < n - 1; ++i) {
    const float x = tf.x[i];
#pragma unroll
    for (int k = 0; k < N; ++k) e[k] += x <= f[k] ? 1 : 0;
  }
  const float first = tf.x[0], last = tf.x[n - 1];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    e[k] = f[k] >= last ? n : e[k];
    e[k] = f[k] > first ? e[k] : 0;
  }
}

// The RGBA of a value in table entry e.  The quotient (f - x0) / w is the product with the
// rounded reciprocal, corrected once by its exact remainder.
template <Input kInput>
__device__ __forceinline__ float4 tf_value(const TfSegment* __restrict__ s, int e, float f) {
  const float4* q = reinterpret_cast<const float4*>(s + e);
  const float4 h = q[0], b = q[1], d = q[2];
  const float num = f - h.x;
  float t;
  if (kInput == kTFDivide) {
    t = num / h.y;
  } else {
    t = num * h.z;
    t = fmaf(fmaf(-t, h.y, num), h.z, t);
  }
  t = h.z != 0.0f ? t : 1.0f;
  return make_float4(fmaf(t, d.x, b.x), fmaf(t, d.y, b.y), fmaf(t, d.z, b.z), fmaf(t, d.w, b.w));
}

// Where a level's outputs go: octant o > 0 of channel c at coeffs + c G3 + level_base + (o - 1) h^3,
// octant 0 at lll + c lll_cs.
struct LevelOut {
  float* coeffs;
  float* lll;
  int64_t G3, lll_cs, level_base, h3;
  __device__ __forceinline__ float* at(int c, int o) const {
    return o == 0 ? lll + c * lll_cs : coeffs + c * G3 + level_base + (o - 1) * h3;
  }
};

// Index i of an axis of length n extended periodically; one period on either side covers every
// position that an output of the axis reads, positions beyond (tiles that stick out) are clamped.
__device__ __forceinline__ int wrap(int i, int n) {
  i = i < 0 ? i + n : (i >= n ? i - n : i);
  return min(max(i, 0), n - 1);
}

// Buffer access from a uniform address with a 32-bit byte offset per lane: one address register, and
// an offset of kOut neither loads nor stores.
constexpr uint32_t kOut = 0xFFFFFFFFu;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const float* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, 0x7FFFFFFF, 0x00020000);
}
__device__ __forceinline__ float load_at(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, static_cast<int>(off), 0, 0));
}
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, static_cast<int>(off), 0, 0);
}

// ------------------------------------------------------------------ bior4.4
// CDF 9/7 analysis: output k reads positions 2k - 4 .. 2k + 4 (low-pass) and 2k - 2 .. 2k + 4
// (high-pass), i.e. window entries 0..8 and 2..8 from 2k - 4 on.
struct Taps97 {
  float lo[9];
  float hi[7];
};

constexpr int kKX = 32;              // output pairs of a tile along x (64 voxels, one wave's lanes)
constexpr int kIX = 2 * kKX + 8;     // tile with halo (2 kKX + 7 voxels, one of padding)
constexpr int kXG = 4;               // output pairs per x-filter task (16 inputs, four 16-byte reads)
constexpr int kNT = 2 * kKX * 4 * 2;  // a thread per (x output, channel, half of the tile's rows)
constexpr int kXcds = 8;

// Bounded at level 1 by VALU issue and LDS (per voxel of four channels: a transfer-function value for each of
// the tile's 1.6 voxels per output voxel, 16 multiply-adds per filter and pair), at two blocks per
// CU (105-115 registers a thread, 49 KB of LDS).  Earlier, a kernel per axis with a thread per output pair
// evaluated the transfer function at each of 16 taps, wrapped every tap's index by a division and moved the four
// channels through memory three times: 8.83 ms for 512^3, five levels; this kernel takes 1.09 ms
// (three quarters of it level 1; reading the field and writing the coefficients once is 2.7 GB, 0.52 ms at
// the rate of a large copy).
// kYG: output pairs per thread along y, of which a tile has two threads' worth.
template <Input kInput, int kYG>
__global__ __launch_bounds__(kNT) void k_dwt97(const float* __restrict__ in, int64_t in_cs, int n, int zc, int tiles_x,
                                               int tiles_y, int n_blocks, LevelOut out, Taps97 taps, DevTF tf) {
  constexpr bool kWithTF = kInput != kRGBA;
  constexpr int kKY = 2 * kYG, kIY = 2 * kKY + 7;   // output pairs of the tile, its rows with the halo
  __shared__ __align__(16) float s_in[4][kIY][kIX];
  __shared__ __align__(16) float s_x[4][kIY][2 * kKX];
  __shared__ __align__(16) TfSegment s_tf[kWithTF ? kTfEntries : 1];
  // Dispatches go to the 8 XCDs in turn: each takes a contiguous run of tiles, whose halos then
  // meet in one L2.
  const int per = (n_blocks + kXcds - 1) / kXcds;
  const int blk = (static_cast<int>(blockIdx.x) % kXcds) * per + static_cast<int>(blockIdx.x) / kXcds;
  if (blk >= n_blocks) return;
  const int tid = threadIdx.x;
  const int h = n >> 1;
  const int kx0 = (blk % tiles_x) * kKX, ky0 = (blk / tiles_x % tiles_y) * kKY, kz0 = blk / (tiles_x * tiles_y) * zc;
  const int planes = 2 * min(zc, h - kz0) + 7;
  const int64_t nn = static_cast<int64_t>(n) * n;
  if (kWithTF) tf_load<kInput>(tf, s_tf, kNT);

  // The taps in vector registers, the equal ones (both filters are symmetric) once: a SIMD issues a multiply-add with a
  // scalar operand at half the rate (1.13 against 1.09 ms).
  Taps97 f;
#pragma unroll
  for (int i = 0; i < 5; ++i) __asm__("v_mov_b32 %0, %1" : "=v"(f.lo[i]) : "s"(taps.lo[i]));
#pragma unroll
  for (int i = 0; i < 4; ++i) f.lo[8 - i] = f.lo[i];
#pragma unroll
  for (int i = 0; i < 4; ++i) __asm__("v_mov_b32 %0, %1" : "=v"(f.hi[i]) : "s"(taps.hi[i]));
#pragma unroll
  for (int i = 0; i < 3; ++i) f.hi[6 - i] = f.hi[i];
  // The tile's loads: entry e of the thread is voxel tid + e kNT of the tile, the same one in every
  // channel (32-bit byte offsets within a plane from a uniform plane address).
  constexpr int kTile = kIY * (kIX - 1);
  constexpr int kLoads = (kTile + kNT - 1) / kNT;
  constexpr int kCh = kWithTF ? 1 : 4;
  uint32_t src[kLoads];
  int dst[kLoads];
#pragma unroll
  for (int e = 0; e < kLoads; ++e) {
    const int q = tid + e * kNT;
    const int row = q / (kIX - 1), col = q % (kIX - 1);
    src[e] = q < kTile ? 4u * static_cast<uint32_t>(wrap(2 * ky0 - 4 + row, n) * n + wrap(2 * kx0 - 4 + col, n)) : kOut;
    dst[e] = q < kTile ? row * kIX + col : -1;
  }
  float v[kCh][kLoads];
  auto load_plane = [&](int z) {
#pragma unroll
    for (int c = 0; c < kCh; ++c) {
      const __amdgpu_buffer_rsrc_t pl = rsrc(in + c * in_cs + wrap(z, n) * nn);
#pragma unroll
      for (int e = 0; e < kLoads; ++e) v[c][e] = load_at(pl, src[e]);
    }
  };
  load_plane(2 * kz0 - 4);
  // A wave is the 64 x outputs of one channel and half of the tile's rows.
  const int xc = tid & (2 * kKX - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ch = wave & 3, yg = wave >> 2;
  // Running z sums: plane 2m is the last of output m - 2 and adds to the sums of later outputs, so the
  // sums move down one output in the same multiply-adds (no register moves).
  float L[2 * kYG][4], H[2 * kYG][3];
#pragma unroll
  for (int i = 0; i < 2 * kYG; ++i) {
    L[i][0] = L[i][1] = L[i][2] = L[i][3] = 0.0f;
    H[i][0] = H[i][1] = H[i][2] = 0.0f;
  }
  const int ox = xc >= kKX ? 1 : 0;
  const int kx = kx0 + (xc & (kKX - 1));
  // Output addresses: a uniform row address (octant's y and z bits, row) plus a byte offset per lane (x
  // bit, column: at most 4 (512^3 + 512)); octant 0 is in a buffer of its own.
  float* const band = out.coeffs + ch * out.G3 + out.level_base - out.h3;   // octant o at band + o h^3
  float* const lll = out.lll + ch * out.lll_cs;
  const uint32_t lane_off = kx < h ? 4u * (static_cast<uint32_t>(ox * out.h3) + static_cast<uint32_t>(kx)) : kOut;
  const uint32_t lane_0 = ox ? kOut : lane_off, lane_1 = ox ? lane_off : kOut;
  if (kWithTF) __syncthreads();
  // One plane; kOdd is its parity, known at compile time so that the sums stay in their registers.
  auto plane = [&](int zi, auto odd) __attribute__((always_inline)) {
    constexpr bool kOdd = decltype(odd)::value;
    float* s_flat = &s_in[0][0][0];
    if constexpr (kWithTF) {
      int seg[kLoads];
      tf_find<kLoads>(tf, v[0], seg);
#pragma unroll
      for (int e = 0; e < kLoads; ++e) {
        __builtin_amdgcn_sched_barrier(0);   // one table entry in registers at a time
        const float4 c = tf_value<kInput>(s_tf, seg[e], v[0][e]);
        if (dst[e] >= 0) {
          s_flat[dst[e]] = c.x;
          s_flat[kIY * kIX + dst[e]] = c.y;
          s_flat[2 * kIY * kIX + dst[e]] = c.z;
          s_flat[3 * kIY * kIX + dst[e]] = c.w;
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < kLoads; ++e)
        if (dst[e] >= 0)
#pragma unroll
          for (int k = 0; k < kCh; ++k) s_flat[k * kIY * kIX + dst[e]] = v[k][e];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (zi + 1 < planes) load_plane(2 * kz0 - 3 + zi);   // runs under this plane's filters
    __syncthreads();
    // x: a task filters kXG output pairs of one row
    constexpr int kTasks = 4 * kIY * (kKX / kXG);
#pragma unroll 1
    for (int t = tid; t < kTasks; t += kNT) {
      const int g = t % (kKX / kXG), r = t / (kKX / kXG);
      const float4* a4 = reinterpret_cast<const float4*>(&s_in[0][0][0] + r * kIX + 2 * kXG * g);
      float a[16];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 w = a4[q];
        a[4 * q] = w.x;
        a[4 * q + 1] = w.y;
        a[4 * q + 2] = w.z;
        a[4 * q + 3] = w.w;
      }
      float lo[kXG], hi[kXG];
#pragma unroll
      for (int k = 0; k < kXG; ++k) {
        lo[k] = f.lo[0] * a[2 * k];
        hi[k] = f.hi[0] * a[2 * k + 2];
#pragma unroll
        for (int i = 1; i < 9; ++i) lo[k] = fmaf(f.lo[i], a[2 * k + i], lo[k]);
#pragma unroll
        for (int i = 1; i < 7; ++i) hi[k] = fmaf(f.hi[i], a[2 * k + 2 + i], hi[k]);
      }
      float* d = &s_x[0][0][0] + r * (2 * kKX) + kXG * g;
      *reinterpret_cast<float4*>(d) = make_float4(lo[0], lo[1], lo[2], lo[3]);
      *reinterpret_cast<float4*>(d + kKX) = make_float4(hi[0], hi[1], hi[2], hi[3]);
    }
    __syncthreads();
    // y: entries 0 .. kYG - 1 low-pass, kYG .. 2 kYG - 1 high-pass
    float y[2 * kYG];
    {
      float a[2 * kYG + 7];
#pragma unroll
      for (int i = 0; i < 2 * kYG + 7; ++i) a[i] = s_x[ch][2 * kYG * yg + i][xc];
#pragma unroll
      for (int k = 0; k < kYG; ++k) {
        float lo = f.lo[0] * a[2 * k], hi = f.hi[0] * a[2 * k + 2];
#pragma unroll
        for (int i = 1; i < 9; ++i) lo = fmaf(f.lo[i], a[2 * k + i], lo);
#pragma unroll
        for (int i = 1; i < 7; ++i) hi = fmaf(f.hi[i], a[2 * k + 2 + i], hi);
        y[k] = lo;
        y[kYG + k] = hi;
      }
    }
    // z
    if constexpr (kOdd) {
#pragma unroll
      for (int i = 0; i < 2 * kYG; ++i) {
        L[i][0] = fmaf(f.lo[7], y[i], L[i][0]);
        L[i][1] = fmaf(f.lo[5], y[i], L[i][1]);
        L[i][2] = fmaf(f.lo[3], y[i], L[i][2]);
        L[i][3] = fmaf(f.lo[1], y[i], L[i][3]);
        H[i][0] = fmaf(f.hi[5], y[i], H[i][0]);
        H[i][1] = fmaf(f.hi[3], y[i], H[i][1]);
        H[i][2] = fmaf(f.hi[1], y[i], H[i][2]);
      }
    } else {
      const int kz = kz0 + (zi >> 1) - 4;
      float lo[2 * kYG], hi[2 * kYG];
#pragma unroll
      for (int i = 0; i < 2 * kYG; ++i) {
        lo[i] = fmaf(f.lo[8], y[i], L[i][0]);
        hi[i] = fmaf(f.hi[6], y[i], H[i][0]);
        L[i][0] = fmaf(f.lo[6], y[i], L[i][1]);
        L[i][1] = fmaf(f.lo[4], y[i], L[i][2]);
        L[i][2] = fmaf(f.lo[2], y[i], L[i][3]);
        L[i][3] = f.lo[0] * y[i];
        H[i][0] = fmaf(f.hi[4], y[i], H[i][1]);
        H[i][1] = fmaf(f.hi[2], y[i], H[i][2]);
        H[i][2] = f.hi[0] * y[i];
      }
      if (zi >= 8) {
#pragma unroll
        for (int k = 0; k < kYG; ++k) {
          const int ky = ky0 + kYG * yg + k;
          if (ky < h) {
            const int64_t row = (static_cast<int64_t>(kz) * h + ky) * h;
            store_at(rsrc(lll + row), lane_0, lo[k]);
            store_at(rsrc(band + row), lane_1, lo[k]);
            store_at(rsrc(band + 2 * out.h3 + row), lane_off, lo[kYG + k]);
            store_at(rsrc(band + 4 * out.h3 + row), lane_off, hi[k]);
            store_at(rsrc(band + 6 * out.h3 + row), lane_off, hi[kYG + k]);
          }
        }
      }
    }
  };
  for (int zi = 0; zi < planes; zi += 2) {   // an odd number of planes
    plane(zi, std::false_type());
    if (zi + 1 < planes) plane(zi + 1, std::true_type());
  }
}

// ------------------------------------------------------------------ Haar
struct TapsHaar {
  float lo[2], hi[2];
};

// A pair of neighbouring floats: the rows start on even elements, but the caller's field may start
// anywhere, so only 4-byte alignment is assumed.
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));

// A thread owns the 2x2x2 cell (kx, ky, kz), all four channels, so each value is read and written once and
// neighbouring lanes read neighbouring pairs: bound by memory.  RGBA 200^3, three levels: 0.226 ms
// with a kernel per axis, 0.060 ms now (0.050 ms for 256 MB at the rate of a large copy).
template <Input kInput>
__global__ __launch_bounds__(256) void k_haar(const float* __restrict__ in, int64_t in_cs, int n, LevelOut out,
                                              TapsHaar f, DevTF tf) {
  constexpr bool kWithTF = kInput != kRGBA;
  __shared__ __align__(16) TfSegment s_tf[kWithTF ? kTfEntries : 1];
  if (kWithTF) {
    tf_load<kInput>(tf, s_tf, 256);
    __syncthreads();
  }
  const int h = n >> 1;
  const int64_t total = static_cast<int64_t>(h) * h * h;
  const int64_t nn = static_cast<int64_t>(n) * n;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; t < total;
       t += static_cast<int64_t>(gridDim.x) * 256) {
    const uint32_t row = static_cast<uint32_t>(t / h);
    const int kx = static_cast<int>(t - static_cast<int64_t>(row) * h);
    const int ky = static_cast<int>(row % h), kz = static_cast<int>(row / h);
    const float* src = in + (static_cast<int64_t>(2 * kz) * n + 2 * ky) * n + 2 * kx;
    float2u s[4];   // rows (z, y): 0 (0, 0), 1 (0, 1), 2 (1, 0), 3 (1, 1)
    float rgba[8][4];
    if (kWithTF) {
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = *reinterpret_cast<const float2u*>(src + (r >> 1) * nn + (r & 1) * n);
      const float v[8] = {s[0].x, s[0].y, s[1].x, s[1].y, s[2].x, s[2].y, s[3].x, s[3].y};
      int seg[8];
      tf_find<8>(tf, v, seg);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float4 q = tf_value<kInput>(s_tf, seg[k], v[k]);
        rgba[k][0] = q.x;
        rgba[k][1] = q.y;
        rgba[k][2] = q.z;
        rgba[k][3] = q.w;
      }
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float2u q = *reinterpret_cast<const float2u*>(src + c * in_cs + (r >> 1) * nn + (r & 1) * n);
          rgba[2 * r][c] = q.x;
          rgba[2 * r + 1][c] = q.y;
        }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float x[2][4];   // [x low | high][row]
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[0][r] = fmaf(f.lo[1], rgba[2 * r + 1][c], f.lo[0] * rgba[2 * r][c]);
        x[1][r] = fmaf(f.hi[1], rgba[2 * r + 1][c], f.hi[0] * rgba[2 * r][c]);
      }
#pragma unroll
      for (int o = 0; o < 4; ++o) {   // x and y bits of the octant
        const float* a = x[o & 1];
        const float* w = o & 2 ? f.hi : f.lo;
        const float y0 = fmaf(w[1], a[1], w[0] * a[0]), y1 = fmaf(w[1], a[3], w[0] * a[2]);
        out.at(c, o)[t] = fmaf(f.lo[1], y1, f.lo[0] * y0);
        out.at(c, o | 4)[t] = fmaf(f.hi[1], y1, f.hi[0] * y0);
      }
    }
  }
}

// The quotient where a segment's width is infinite or its reciprocal would not be a normal number with room for the
// remainder, else the product.
Input tf_form(const DevTF& tf) {
  for (int i = 1; i < tf.n; ++i) {
    const float w = tf.x[i] - tf.x[i - 1];
    if (w > 0.0f && !(w >= 0x1p-100f && w <= 0x1p100f)) return kTFDivide;
  }
  return kTF;
}

__global__ __launch_bounds__(256) void k_copy(const float* __restrict__ in, float* __restrict__ out, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * 256)
    out[i] = in[i];
}

// Tile of a bior4.4 level of h output pairs a side.
struct Tile97 {
  int yg, zc;   // output pairs per thread along y, output pairs per block along z
};
Tile97 tile97(int h) {
  // Levels of up to one small tile per CU take as long as a block: planes in turn, each the loads' latency and one
  // wave's instructions.  Few of these and few planes count there.  us a level of RGBA with a kernel per axis / yg 4,
  // zc 2 / yg 1, zc 1 / yg 1, zc 2: 16.1 / 20.2 / 9.7 / 11.4 (side 32), 20.0 / 20.2 / 13.1 / 11.7 (64), 43.4 / 29.8 /
  // 38.8 / 29.2 (96).
  constexpr int64_t kCUs = 256;
  for (int zc = 1; zc <= 2; ++zc)
    if (ceil_div(h, kKX) * ceil_div(h, 2) * ceil_div(h, zc) <= kCUs) return {1, zc};
  // A chunk re-reads seven planes, so it is as long as still leaves about four blocks per CU; at least two outputs.
  Tile97 t{4, 32};
  const int64_t tiles = ceil_div(h, kKX) * ceil_div(h, 2 * t.yg);
  while (t.zc > 2 && tiles * ceil_div(h, t.zc) < 4 * kCUs) t.zc >>= 1;
  return t;
}

}  // namespace
}  // namespace vbm

using namespace vbm;

extern "C" size_t vbm_dwt3d_workspace_size(int32_t G, int32_t J) {
  (void)J;
  if (G <= 0) return 0;
  const size_t plane = static_cast<size_t>(G) * G * G;
  // two buffers of 4 channels for the levels' LLL, used in turn
  return 2 * align_up(4 * plane * sizeof(float), 256);
}

extern "C" vbm_status vbm_dwt3d(const float* vol, int32_t G, int32_t J, int32_t wavelet, const vbm_tf* tf,
                                float* coeffs, void* ws, size_t ws_bytes, void* stream) {
  if (!vol || !coeffs || !ws) {
    set_error("vbm_dwt3d: null pointer");
    return VBM_ERR_INVALID;
  }
  if (G < 2 || G > 1024 || J < 1 || J > 10 || (G % (1 << J)) != 0 || (G >> J) < 2) {
    set_error("vbm_dwt3d: need G %% 2^J == 0, G/2^J >= 2, 1 <= J <= 10, G <= 1024 (G=%d J=%d)", G, J);
    return VBM_ERR_INVALID;
  }
  if (wavelet != VBM_WAVELET_HAAR && wavelet != VBM_WAVELET_BIOR44) {
    set_error("vbm_dwt3d: unknown wavelet %d", wavelet);
    return VBM_ERR_UNSUPPORTED;
  }
  DevTF dtf;
  std::memset(&dtf, 0, sizeof(dtf));
  if (tf) {
    if (tf->n_points < 2 || tf->n_points > VBM_TF_MAX_POINTS) {
      set_error("vbm_dwt3d: transfer function needs 2..%d points", VBM_TF_MAX_POINTS);
      return VBM_ERR_UNSUPPORTED;
    }
    for (int i = 1; i < tf->n_points; ++i)
      if (!(tf->x[i] >= tf->x[i - 1])) {
        set_error("vbm_dwt3d: transfer-function control points must ascend");
        return VBM_ERR_INVALID;
      }
    dtf.n = tf->n_points;
    for (int i = 0; i < tf->n_points; ++i) {
      dtf.x[i] = tf->x[i];
      for (int c = 0; c < 4; ++c) dtf.rgba[i][c] = tf->rgba[i][c];
    }
  }
  if (ws_bytes < vbm_dwt3d_workspace_size(G, J)) {
    set_error("vbm_dwt3d: workspace %zu < %zu bytes", ws_bytes, vbm_dwt3d_workspace_size(G, J));
    return VBM_ERR_WORKSPACE;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const FilterBankD fb = make_filter_bank(wavelet);
  const int64_t G3 = static_cast<int64_t>(G) * G * G;
  float* p = static_cast<float*>(ws);   // this level's LLL, then the next level's input
  float* q = reinterpret_cast<float*>(static_cast<char*>(ws) + align_up(4 * G3 * sizeof(float), 256));
  const float* cur = vol;
  int64_t cur_cs = G3;
  // The first level writes coefficients while other blocks still read the field: one that shares memory with them is
  // read from a copy in the buffer that this level leaves alone.
  const int64_t values = tf ? G3 : 4 * G3;
  const uintptr_t v0 = reinterpret_cast<uintptr_t>(vol), c0 = reinterpret_cast<uintptr_t>(coeffs);
  if (v0 < c0 + 4 * G3 * sizeof(float) && c0 < v0 + values * sizeof(float)) {
    const int64_t blocks = ceil_div(values, 256);
    hipLaunchKernelGGL(k_copy, dim3(static_cast<unsigned>(blocks < 8192 ? blocks : 8192)), dim3(256), 0, s, vol, q,
                       values);
    VBM_LAUNCH_CHECK("dwt_copy");
    cur = q;
  }
  for (int j = 1; j <= J; ++j) {
    const int n = G >> (j - 1);
    const int h = n >> 1;
    LevelOut out;
    out.coeffs = coeffs;
    out.G3 = G3;
    out.h3 = static_cast<int64_t>(h) * h * h;
    out.lll = j == J ? coeffs : p;
    out.lll_cs = j == J ? G3 : out.h3;
    // packed offset of block (j, 1): n_J^3 + sum_{j' > j} 7 n_{j'}^3
    out.level_base = static_cast<int64_t>(G >> J) * (G >> J) * (G >> J);
    for (int jj = J; jj > j; --jj) out.level_base += 7LL * (G >> jj) * (G >> jj) * (G >> jj);
    const Input input = j == 1 && tf ? tf_form(dtf) : kRGBA;
    if (wavelet == VBM_WAVELET_HAAR) {
      TapsHaar f;
      for (int i = 0; i < 2; ++i) {
        f.lo[i] = static_cast<float>(fb.lo_a.taps[i]);
        f.hi[i] = static_cast<float>(fb.hi_a.taps[i]);
      }
      const dim3 grid(static_cast<unsigned>(ceil_div(out.h3, 256) < 65536 ? ceil_div(out.h3, 256) : 65536));
      const auto kernel = input == kRGBA ? k_haar<kRGBA> : input == kTF ? k_haar<kTF> : k_haar<kTFDivide>;
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, cur, cur_cs, n, out, f, dtf);
    } else {
      Taps97 f;
      for (int i = 0; i < 9; ++i) f.lo[i] = static_cast<float>(fb.lo_a.taps[i]);
      for (int i = 0; i < 7; ++i) f.hi[i] = static_cast<float>(fb.hi_a.taps[i]);   // symmetric as rounded, like lo
      const Tile97 t = tile97(h);
      const int tx = static_cast<int>(ceil_div(h, kKX)), ty = static_cast<int>(ceil_div(h, 2 * t.yg));
      const int nb = tx * ty * static_cast<int>(ceil_div(h, t.zc));
      const dim3 grid(static_cast<unsigned>(kXcds * ceil_div(nb, kXcds)));
      auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(kNT), 0, s, cur, cur_cs, n, t.zc, tx, ty, nb, out, f, dtf);
      };
      if (t.yg == 4)
        launch(input == kRGBA ? k_dwt97<kRGBA, 4> : input == kTF ? k_dwt97<kTF, 4> : k_dwt97<kTFDivide, 4>);
      else
        launch(input == kRGBA ? k_dwt97<kRGBA, 1> : input == kTF ? k_dwt97<kTF, 1> : k_dwt97<kTFDivide, 1>);
    }
    VBM_LAUNCH_CHECK("dwt3d");
    cur = p;
    cur_cs = out.h3;
    float* t = p;
    p = q;
    q = t;
  }
  return VBM_OK;
}
