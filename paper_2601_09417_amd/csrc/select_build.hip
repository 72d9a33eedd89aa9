// vbm_build_gaussians: joint-norm global top-K (Supp. A, joint magnitude) and analytical Gaussian
// construction by bank lookup (Sec. 4.3: eq. per_location_weight, eq. wavelet_gaussian_kernel,
// eq. translation_operator).
//
// Selection is exact and deterministic.  Few of the M locations are kept, so one pass over the coefficients writes
// down only candidates: the locations whose float32 key reaches a lower bound that a sample of the keys
// gives (a pass that finds fewer than K candidates is repeated without a bound).  Three radix-select passes over
// the candidates (12, 10 and 10 bits, most significant first) find the K-th largest key t; a last one
// keeps every key > t plus the lowest-index keys == t until K are kept, in ascending index order, and builds
// their Gaussians.
// 512^3, K = 1M: 0.56 ms, where a key written per location and six passes over the keys took 1.93 ms (reading
// the coefficients takes 0.42 ms at the rate of a large copy).
#include <hip/hip_runtime.h>

#include <cmath>

#include "block_scan.h"
#include "common.h"

namespace vbm {
namespace {

constexpr int kT = 256;
constexpr int kPerThread = 16;
constexpr int kRegion = kT * kPerThread;   // locations per region: its candidates lie at the region's own places

// Radix-select digits: bits 31..20, 19..10, 9..0.
constexpr int kBins[3] = {4096, 1024, 1024};
constexpr int kShift[3] = {20, 10, 0};
constexpr int kHistWords = 4096 + 1024 + 1024;
// Blocks of the passes over the candidates.  Their counts meet at the same bins: 256 / 512 / 1024 blocks take 62 / 53
// / 58 us in the three digits and the count (512^3, K = 1M), 97 us with a region at a time per wave and 1024.
constexpr int kHistBlocks = 512;
constexpr int kTallies = 64;               // candidate totals, spread over as many words
constexpr int kGroup = 256;                // regions per partial sum of kept keys
constexpr int kGroupsMax = 1024;           // 1024^3 locations
static_assert(static_cast<int64_t>(kGroupsMax) * kGroup * kRegion >= (int64_t{1} << 30), "groups of the largest grid");

struct SelectState {
  uint32_t bound;      // lower bound of a candidate's key
  uint32_t ticket;     // sample blocks done
  uint32_t prefix[3];  // key bits fixed after each digit
  uint32_t rest[3];    // elements still to take from the bucket matching prefix
};

// Everything of a selection that starts from zero.
struct SelectScratch {
  uint32_t hist[kHistWords];
  uint32_t sample[4096];
  uint32_t tally[kTallies];
  unsigned long long group[kGroupsMax];   // keys above the K-th largest, and equal to it (high half), per group
  SelectState st;
};

#pragma clang fp contract(off)
__device__ __forceinline__ float joint_square(float r, float g, float b, float a) {
  return ((r * r + g * g) + b * b) + a * a;
}
__device__ __forceinline__ uint32_t joint_key(float square) { return __float_as_uint(sqrt_rn_f32(square)); }

__global__ __launch_bounds__(kT) void k_select_init(SelectScratch* __restrict__ sc) {
  uint32_t* w = reinterpret_cast<uint32_t*>(sc);
  for (int i = blockIdx.x * kT + threadIdx.x; i < static_cast<int>(sizeof(SelectScratch) / 4); i += gridDim.x * kT)
    w[i] = 0u;
}

// The digit whose bucket holds the k-th largest element (1-based) of a histogram, and how many of the bucket are
// wanted.  Every thread of the block calls it and gets both.
template <int BINS>
__device__ __forceinline__ void pick_digit(const uint32_t* __restrict__ hist, uint32_t k, uint32_t& digit,
                                           uint32_t& rest) {
  constexpr int PER = BINS / kT;
  __shared__ uint32_t s_digit, s_rest;
  uint32_t h[PER], sum = 0;
  const int top = BINS - 1 - static_cast<int>(threadIdx.x) * PER;   // this thread's bins, from the highest down
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    h[i] = hist[top - i];
    sum += h[i];
  }
  uint32_t all;
  uint32_t above = block_excl_scan(sum, &all);
  if (above < k && k <= above + sum) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (above < k && k <= above + h[i]) {
        s_digit = static_cast<uint32_t>(top - i);
        s_rest = k - above;
      }
      above += h[i];
    }
  }
  __syncthreads();
  digit = s_digit;
  rest = s_rest;
}

// The candidates' lower bound: the keys of 16 consecutive locations (a cache line) in every 2048, counted by their
// top 12 bits; the last block takes the bin where `rank` of the sample's keys are reached.
constexpr int kSampleRun = 16, kSampleStep = 2048;
__global__ __launch_bounds__(kT) void k_select_sample(const float* __restrict__ coeffs, int64_t M, uint32_t rank,
                                                      SelectScratch* __restrict__ sc) {
  __shared__ uint32_t s_hist[4096];
  __shared__ bool s_last;
  for (int i = threadIdx.x; i < 4096; i += kT) s_hist[i] = 0u;
  __syncthreads();
  const int64_t n = M / kSampleStep * kSampleRun;
  constexpr int kAhead = 4;   // samples whose loads are in flight together
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kT;
  for (int64_t t = static_cast<int64_t>(blockIdx.x) * kT + threadIdx.x; t < n; t += kAhead * stride) {
    float sq[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int64_t u = min(t + q * stride, n - 1);
      const int64_t i = u / kSampleRun * kSampleStep + u % kSampleRun;
      sq[q] = joint_square(coeffs[i], coeffs[M + i], coeffs[2 * M + i], coeffs[3 * M + i]);
    }
    // (the bound need not be exact: the plain square root serves)
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
      if (t + q * stride < n) atomicAdd(&s_hist[__float_as_uint(__builtin_amdgcn_sqrtf(sq[q])) >> 20], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 4096; i += kT)
    if (s_hist[i]) atomicAdd(&sc->sample[i], s_hist[i]);
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) s_last = atomicAdd(&sc->st.ticket, 1u) == gridDim.x - 1;
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  for (int i = threadIdx.x; i < 4096; i += kT)
    s_hist[i] = __hip_atomic_load(&sc->sample[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  uint32_t digit, rest;
  pick_digit<4096>(s_hist, rank, digit, rest);
  if (threadIdx.x == 0) sc->st.bound = digit << 20;
}

// Candidates of one region in ascending index order: keys and indices at the region's first places, their number in
// cnt.  A wave takes 1024 consecutive locations; a lane reads four at a time (kVec: 16-byte loads).  The square of the
// joint norm is compared with a bound a little below the key bound's square, so that only the few that
// pass it take the square root.  Bound by reading the coefficients: 0.37 ms for 512^3 (5.9 TB/s).
template <bool kVec>
__device__ __forceinline__ void region_candidates(const float* __restrict__ coeffs, int64_t M, int64_t region,
                                                  uint32_t bound, uint32_t* __restrict__ cand_key,
                                                  uint32_t* __restrict__ cand_idx, uint32_t* __restrict__ cnt,
                                                  uint32_t* __restrict__ tally) {
  __shared__ uint32_t s_wave[kT / 64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t base = region * kRegion, first = base + w * 1024;
  const float tb = __uint_as_float(bound);
  const float sq = tb * tb * 0.999999f;
  const float least = sq > 1e-30f ? sq : (bound >= 0x7F800000u ? sq : 0.0f);   // (inf or NaN: decided by the key)
  float v[4][4];   // squares
  uint32_t mask = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t i = first + r * 256 + lane * 4;
    if (kVec) {
      if (i < M) {   // (M is a multiple of 8)
        const float4 a = *reinterpret_cast<const float4*>(coeffs + i);
        const float4 b = *reinterpret_cast<const float4*>(coeffs + M + i);
        const float4 c = *reinterpret_cast<const float4*>(coeffs + 2 * M + i);
        const float4 d = *reinterpret_cast<const float4*>(coeffs + 3 * M + i);
        v[r][0] = joint_square(a.x, b.x, c.x, d.x);
        v[r][1] = joint_square(a.y, b.y, c.y, d.y);
        v[r][2] = joint_square(a.z, b.z, c.z, d.z);
        v[r][3] = joint_square(a.w, b.w, c.w, d.w);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i + j < M) v[r][j] = joint_square(coeffs[i + j], coeffs[M + i + j], coeffs[2 * M + i + j],
                                              coeffs[3 * M + i + j]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = first + r * 256 + lane * 4 + j;
      if (i < M && !(v[r][j] < least)) mask |= 1u << (4 * r + j);
    }
  uint32_t key[4][4];
  if (__ballot(mask != 0u)) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((mask >> (4 * r + j)) & 1u) {
          key[r][j] = joint_key(v[r][j]);
          if (key[r][j] < bound) mask &= ~(1u << (4 * r + j));
        }
  }
  // places within the wave: per round the candidates of lower lanes, a 16-bit field each
  uint64_t mine = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) mine |= static_cast<uint64_t>(__popc((mask >> (4 * r)) & 15u)) << (16 * r);
  uint64_t incl = 0, total = 0;
  if (__ballot(mask != 0u)) {
    incl = wave_incl_scan(mine);
    total = __shfl(incl, 63, 64);
  }
  uint32_t round_at[4], sum = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    round_at[r] = sum;
    sum += static_cast<uint32_t>(total >> (16 * r)) & 0xFFFFu;
  }
  if (lane == 0) s_wave[w] = sum;
  __syncthreads();
  uint32_t at = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kT / 64; ++i) {
    at += i < w ? s_wave[i] : 0u;
    all += s_wave[i];
  }
  __syncthreads();
  if (mask) {
    const uint64_t excl = incl - mine;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int64_t p = base + at + round_at[r] + (static_cast<uint32_t>(excl >> (16 * r)) & 0xFFFFu);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((mask >> (4 * r + j)) & 1u) {
          cand_key[p] = key[r][j];
          cand_idx[p] = static_cast<uint32_t>(first + r * 256 + lane * 4 + j);
          ++p;
        }
    }
  }
  if (threadIdx.x == 0) {
    cnt[region] = all;
    if (all) atomicAdd(&tally[region % kTallies], all);
  }
}

template <bool kVec>
__global__ __launch_bounds__(kT) void k_candidates(const float* __restrict__ coeffs, int64_t M,
                                                   SelectScratch* __restrict__ sc, uint32_t* __restrict__ cand_key,
                                                   uint32_t* __restrict__ cand_idx, uint32_t* __restrict__ cnt) {
  region_candidates<kVec>(coeffs, M, blockIdx.x, sc->st.bound, cand_key, cand_idx, cnt, sc->tally);
}

// The same without a bound where the bound has left fewer than K candidates (a few blocks that otherwise do nothing).
template <bool kVec>
__global__ __launch_bounds__(kT) void k_candidates_all(const float* __restrict__ coeffs, int64_t M, int64_t K,
                                                       int64_t regions, SelectScratch* __restrict__ sc,
                                                       uint32_t* __restrict__ cand_key,
                                                       uint32_t* __restrict__ cand_idx, uint32_t* __restrict__ cnt) {
  int64_t n = 0;
  for (int i = 0; i < kTallies; ++i) n += sc->tally[i];
  if (n >= K) return;
  for (int64_t r = blockIdx.x; r < regions; r += gridDim.x)
    region_candidates<kVec>(coeffs, M, r, 0u, cand_key, cand_idx, cnt, sc->sample);   // (no one reads that tally)
}

// Calls fn with every candidate key of the wave's regions and done(region) after each: a wave per region, four keys a
// lane at a time.  The regions go to the waves in turn (the coarse levels' are full, most others hold some 30
// candidates), and a wave asks for the counts and first 256 keys of four of them together, so that few blocks, whose
// counts then meet at the same addresses, keep as much in flight as many.
template <class F, class D>
__device__ __forceinline__ void for_candidates(const uint32_t* __restrict__ cand_key, const uint32_t* __restrict__ cnt,
                                               int64_t regions, F&& fn, D&& done) {
  constexpr int kAhead = 4;
  const int lane = threadIdx.x & 63;
  const int64_t waves = static_cast<int64_t>(gridDim.x) * (kT / 64);
  auto use = [&](const uint4& q, uint32_t i, uint32_t n) {
    if (4 * i < n) fn(q.x);
    if (4 * i + 1 < n) fn(q.y);
    if (4 * i + 2 < n) fn(q.z);
    if (4 * i + 3 < n) fn(q.w);
  };
  for (int64_t r0 = static_cast<int64_t>(blockIdx.x) * (kT / 64) + (threadIdx.x >> 6); r0 < regions;
       r0 += kAhead * waves) {
    uint32_t n[kAhead];
    uint4 q[kAhead];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) n[k] = r0 + k * waves < regions ? cnt[r0 + k * waves] : 0u;
    auto keys = [&](int k) {   // (256-byte aligned workspace)
      return reinterpret_cast<const uint4*>(cand_key + (r0 + k * waves) * kRegion);
    };
#pragma unroll
    for (int k = 0; k < kAhead; ++k)
      if (4u * lane < n[k]) q[k] = keys(k)[lane];
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      if (r0 + k * waves >= regions) break;
      use(q[k], lane, n[k]);
      for (uint32_t i = 64 + lane; 4 * (i - lane) < n[k]; i += 64 * kAhead) {
        uint4 p[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          if (4 * (i + 64 * u) < n[k]) p[u] = keys(k)[i + 64 * u];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) use(p[u], i + 64 * u, n[k]);
      }
      done(r0 + k * waves);
    }
  }
}

// Digit D of the candidates whose higher digits are those picked so far, counted.
template <int D>
__global__ __launch_bounds__(kT) void k_select_hist(const uint32_t* __restrict__ cand_key,
                                                    const uint32_t* __restrict__ cnt, int64_t regions, uint32_t K,
                                                    SelectScratch* __restrict__ sc) {
  __shared__ uint32_t s_hist[kBins[D]];
  for (int i = threadIdx.x; i < kBins[D]; i += kT) s_hist[i] = 0u;
  uint32_t prefix = 0;
  if constexpr (D > 0) {   // picks the digit before, as every block does; block 0 notes it for later kernels
    uint32_t digit, rest;
    pick_digit<kBins[D - 1]>(sc->hist + (D == 1 ? 0 : kBins[0]), D == 1 ? K : sc->st.rest[0], digit, rest);
    prefix = (D == 1 ? 0u : sc->st.prefix[0]) | digit << kShift[D - 1];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      sc->st.prefix[D - 1] = prefix;
      sc->st.rest[D - 1] = rest;
    }
  }
  __syncthreads();
  constexpr uint32_t kHigh = D == 0 ? 0u : ~((1u << kShift[D > 0 ? D - 1 : 0]) - 1u);
  for_candidates(
      cand_key, cnt, regions,
      [&](uint32_t k) {
        if ((k & kHigh) == prefix) atomicAdd(&s_hist[(k >> kShift[D]) & (kBins[D] - 1)], 1u);
      },
      [](int64_t) {});
  __syncthreads();
  uint32_t* h = sc->hist + (D == 0 ? 0 : D == 1 ? kBins[0] : kBins[0] + kBins[1]);
  for (int i = threadIdx.x; i < kBins[D]; i += kT)
    if (s_hist[i]) atomicAdd(&h[i], s_hist[i]);
}

__device__ __forceinline__ uint64_t select_flags(uint32_t key, uint32_t thr) {
  return (key > thr ? 1ull : 0ull) | (key == thr ? (1ull << 32) : 0ull);
}

// Keys above the K-th largest, and equal to it (high half), of each region.
__global__ __launch_bounds__(kT) void k_select_count(const uint32_t* __restrict__ cand_key,
                                                     const uint32_t* __restrict__ cnt, int64_t regions,
                                                     SelectScratch* __restrict__ sc, uint64_t* __restrict__ sums) {
  uint32_t digit, rest;
  pick_digit<kBins[2]>(sc->hist + kBins[0] + kBins[1], sc->st.rest[1], digit, rest);
  const uint32_t thr = sc->st.prefix[1] | digit;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc->st.prefix[2] = thr;
    sc->st.rest[2] = rest;
  }
  uint64_t acc = 0;
  for_candidates(
      cand_key, cnt, regions, [&](uint32_t k) { acc += select_flags(k, thr); },
      [&](int64_t r) {
        for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
        if ((threadIdx.x & 63) == 0) sums[r] = acc;
        acc = 0;
      });
}

// The same of each group of regions, a block per group (added by k_select_count's waves as they went, the sums of 256
// regions met at one address: 45 us for both against 18).
__global__ __launch_bounds__(kT) void k_select_groups(const uint64_t* __restrict__ sums, int64_t regions,
                                                      SelectScratch* __restrict__ sc) {
  static_assert(kGroup == kT, "a thread per region");
  const int64_t r = static_cast<int64_t>(blockIdx.x) * kGroup + threadIdx.x;
  uint64_t total;
  block_excl_scan(r < regions ? sums[r] : uint64_t{0}, &total);
  if (threadIdx.x == 0) sc->group[blockIdx.x] = total;
}

struct BuildParams {
  int G, J;
  float h;
  float delta;
  float op_min, op_max;
  int s_mode;
  int unit_weight;
  int64_t M;
};

// Gaussian n of the output from the coefficient at packed index idx.
__device__ __forceinline__ void build_one(const float* __restrict__ coeffs, int64_t idx, int64_t n,
                                          const float* __restrict__ bank, const BuildParams& p,
                                          const vbm_gaussians& out) {
  // decode the packed index: [LLL_J][level J: o=1..7]...[level 1: o=1..7]
  int j = p.J, b = 0;
  int64_t off = idx;
  int64_t nJ = p.G >> p.J;
  int64_t sz = nJ * nJ * nJ;
  int o = 0;
  int64_t side = nJ;
  if (off < sz) {
    o = 0;
  } else {
    off -= sz;
    for (j = p.J; j >= 1; --j) {
      side = p.G >> j;
      const int64_t s3 = side * side * side;
      if (off < 7 * s3) {
        o = 1 + static_cast<int>(off / s3);
        off -= static_cast<int64_t>(o - 1) * s3;
        break;
      }
      off -= 7 * s3;
    }
  }
  b = (o == 0) ? 0 : 1 + 7 * (p.J - j) + (o - 1);
  const int kx = static_cast<int>(off % side);
  const int ky = static_cast<int>((off / side) % side);
  const int kz = static_cast<int>(off / (side * side));
  const float* e = bank + static_cast<int64_t>(b) * VBM_BANK_FLOATS;
  const float w = p.unit_weight ? 1.0f : e[0];
  const float step = static_cast<float>(1 << j);
  out.means[n] = -1.0f + p.h * (e[1] + step * kx + p.delta);
  out.means[out.stride + n] = -1.0f + p.h * (e[2] + step * ky + p.delta);
  out.means[2 * out.stride + n] = -1.0f + p.h * (e[3] + step * kz + p.delta);
  for (int c = 0; c < 3; ++c) out.scales[c * out.stride + n] = p.h * e[4 + c];
  for (int c = 0; c < 4; ++c) out.quats[c * out.stride + n] = e[7 + c];
  const float s = p.s_mode == 0 ? exp2f(-1.5f * static_cast<float>(j)) : 1.0f;
  for (int c = 0; c < 3; ++c) {
    const float amp = s * fabsf(coeffs[c * p.M + idx]) * w;
    out.rgb[c * out.stride + n] = fminf(fmaxf(amp, 0.0f), 1.0f);
  }
  const float amp_a = s * fabsf(coeffs[3 * p.M + idx]) * w;
  out.opacity[n] = fminf(fmaxf(amp_a, p.op_min), p.op_max);
}

__global__ __launch_bounds__(kT) void k_build(const float* __restrict__ coeffs, const int64_t* __restrict__ kept,
                                              int64_t K, const float* __restrict__ bank, BuildParams p,
                                              vbm_gaussians out) {
  const int64_t n = static_cast<int64_t>(blockIdx.x) * kT + threadIdx.x;
  if (n >= K) return;
  const int64_t idx = kept[n];
  if (idx < 0 || idx >= p.M) return;   // a caller-given index outside the grid builds nothing
  build_one(coeffs, idx, n, bank, p, out);
}

// Keeps and builds, in ascending index order; a block per region, which first adds up what the regions before it
// keep (whole groups, then its own group's regions).
__global__ __launch_bounds__(kT) void k_select_build(const float* __restrict__ coeffs,
                                                     const uint32_t* __restrict__ cand_key,
                                                     const uint32_t* __restrict__ cand_idx,
                                                     const uint32_t* __restrict__ cnt,
                                                     const SelectScratch* __restrict__ sc,
                                                     const uint64_t* __restrict__ sums,
                                                     const float* __restrict__ bank, BuildParams p, vbm_gaussians out,
                                                     int64_t* __restrict__ kept_out) {
  const int64_t r = blockIdx.x, group = r / kGroup;
  const uint32_t n = cnt[r];
  if (n == 0 || sums[r] == 0) return;
  const uint32_t thr = sc->st.prefix[2], need = sc->st.rest[2];
  uint64_t before = group * kGroup + threadIdx.x < r ? sums[group * kGroup + threadIdx.x] : 0ull, carry;
  for (int64_t g = threadIdx.x; g < group; g += kT) before += sc->group[g];
  block_excl_scan(before, &carry);
  for (uint32_t t0 = 0; t0 < n; t0 += kT) {
    const uint32_t t = t0 + threadIdx.x;
    const uint64_t f = t < n ? select_flags(cand_key[r * kRegion + t], thr) : 0ull;
    uint64_t tot;
    const uint64_t ex = block_excl_scan(f, &tot) + carry;
    carry += tot;
    const uint32_t gt = static_cast<uint32_t>(ex), eq = static_cast<uint32_t>(ex >> 32);
    if ((f & 1ull) || ((f >> 32) && eq < need)) {
      const int64_t slot = static_cast<int64_t>(gt) + (eq < need ? eq : need);
      const int64_t idx = cand_idx[r * kRegion + t];
      build_one(coeffs, idx, slot, bank, p, out);
      if (kept_out) kept_out[slot] = idx;
    }
  }
}

// Ablation without the transition bank: sigma_iso = mean over the n built Gaussians of the mean of
// their three scales (float64, fixed order: thread-strided sums, then a fixed tree), then every
// Gaussian gets scales sigma_iso and the identity rotation.  One block.
__global__ __launch_bounds__(1024) void k_isotropize(vbm_gaussians out, int64_t n) {
  __shared__ double s_sum[1024];
  const int64_t S = out.stride;
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 1024)
    acc += (static_cast<double>(out.scales[i]) + static_cast<double>(out.scales[S + i]) +
            static_cast<double>(out.scales[2 * S + i])) / 3.0;
  s_sum[threadIdx.x] = acc;
  __syncthreads();
  for (int st = 512; st >= 1; st >>= 1) {
    if (static_cast<int>(threadIdx.x) < st) s_sum[threadIdx.x] += s_sum[threadIdx.x + st];
    __syncthreads();
  }
  const float sigma = static_cast<float>(s_sum[0] / static_cast<double>(n));
  for (int64_t i = threadIdx.x; i < n; i += 1024) {
    out.scales[i] = out.scales[S + i] = out.scales[2 * S + i] = sigma;
    out.quats[i] = 1.0f;
    out.quats[S + i] = out.quats[2 * S + i] = out.quats[3 * S + i] = 0.0f;
  }
}

int grid_cap(int64_t n, int cap) { return static_cast<int>(n < cap ? n : cap); }

struct SelectWs {
  uint32_t* cand_key;
  uint32_t* cand_idx;
  uint32_t* cnt;        // candidates per region
  uint64_t* sums;       // kept keys per region
  SelectScratch* sc;
};
SelectWs carve(Carver& c, int64_t M) {
  const int64_t regions = ceil_div(M, kRegion);
  SelectWs w;
  w.cand_key = c.take<uint32_t>(regions * kRegion);
  w.cand_idx = c.take<uint32_t>(regions * kRegion);
  w.cnt = c.take<uint32_t>(regions);
  w.sums = c.take<uint64_t>(regions);
  w.sc = c.take<SelectScratch>(1);
  return w;
}

// Rank in the sample that gives the candidates' bound, 0 for no bound: K's share of the sample, and more for
// neighbours in a sampled run being alike (eight standard deviations of a sample of whole runs).  Grids of up
// to 64^3 are not sampled (the pass over all of them is as short), nor where most locations are wanted.
uint32_t sample_rank(int64_t M, int64_t K) {
  if (M <= (1 << 18)) return 0;
  const double n = static_cast<double>(M / kSampleStep * kSampleRun);
  const double share = static_cast<double>(K) / static_cast<double>(M) * n;
  const double rank = share * 1.0625 + 8.0 * std::sqrt(kSampleRun * share) + kSampleRun;
  return rank < 0.75 * n ? static_cast<uint32_t>(rank) : 0u;
}

}  // namespace
}  // namespace vbm

using namespace vbm;

extern "C" size_t vbm_build_workspace_size(int32_t G, int32_t J) {
  (void)J;
  if (G <= 0) return 0;
  Carver c(nullptr);
  carve(c, static_cast<int64_t>(G) * G * G);
  return align_up(c.off, 256);
}

extern "C" vbm_status vbm_build_gaussians(const float* coeffs, int32_t G, int32_t J, const float* bank_dev, int64_t K,
                                          const vbm_build_opts* opts, vbm_gaussians out, int64_t* kept_index, void* ws,
                                          size_t ws_bytes, void* stream) {
  if (!coeffs || !bank_dev || !opts || !ws || !out.means || !out.scales || !out.quats || !out.opacity || !out.rgb) {
    set_error("vbm_build_gaussians: null pointer");
    return VBM_ERR_INVALID;
  }
  if (G < 2 || G > 1024 || J < 1 || J > 10 || (G % (1 << J)) != 0 || (G >> J) < 2) {
    set_error("vbm_build_gaussians: bad G=%d J=%d", G, J);
    return VBM_ERR_INVALID;
  }
  const int64_t M = static_cast<int64_t>(G) * G * G;
  if (K < 1 || K > M) {
    set_error("vbm_build_gaussians: K=%lld outside 1..G^3", static_cast<long long>(K));
    return VBM_ERR_INVALID;
  }
  if (out.stride < K) {
    set_error("vbm_build_gaussians: output stride %lld < K", static_cast<long long>(out.stride));
    return VBM_ERR_INVALID;
  }
  if (opts->s_mode != 0 && opts->s_mode != 1) {
    set_error("vbm_build_gaussians: s_mode must be 0 (paper) or 1 (none)");
    return VBM_ERR_INVALID;
  }
  if (!(opts->opacity_min >= 0.0f && opts->opacity_min <= opts->opacity_max && opts->opacity_max <= 1.0f)) {
    set_error("vbm_build_gaussians: need 0 <= opacity_min <= opacity_max <= 1");
    return VBM_ERR_INVALID;
  }
  if ((opts->isotropic != 0 && opts->isotropic != 1) || (opts->unit_weight != 0 && opts->unit_weight != 1)) {
    set_error("vbm_build_gaussians: isotropic and unit_weight must be 0 or 1");
    return VBM_ERR_INVALID;
  }
  if (ws_bytes < vbm_build_workspace_size(G, J)) {
    set_error("vbm_build_gaussians: workspace %zu < %zu", ws_bytes, vbm_build_workspace_size(G, J));
    return VBM_ERR_WORKSPACE;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  Carver c(ws);
  const SelectWs w = carve(c, M);
  const int64_t regions = ceil_div(M, kRegion);
  BuildParams p;
  p.G = G;
  p.J = J;
  p.h = 2.0f / static_cast<float>(G);
  p.delta = opts->delta;
  p.op_min = opts->opacity_min;
  p.op_max = opts->opacity_max;
  p.s_mode = opts->s_mode;
  p.unit_weight = opts->unit_weight;
  p.M = M;
  hipLaunchKernelGGL(k_select_init, dim3(16), dim3(kT), 0, s, w.sc);
  VBM_LAUNCH_CHECK("select_init");
  const uint32_t rank = sample_rank(M, K);
  if (rank) {
    // (few blocks: each adds its counts to the same bins and releases them; 128, 512, 2048 blocks: 29, 69, 196 us)
    hipLaunchKernelGGL(k_select_sample, dim3(128), dim3(kT), 0, s, coeffs, M, rank, w.sc);
    VBM_LAUNCH_CHECK("select_sample");
  }
  // 16-byte loads need every channel plane to start on a 16-byte boundary (M is a multiple of 8)
  const bool vec = (reinterpret_cast<uintptr_t>(coeffs) & 15u) == 0;
  hipLaunchKernelGGL(vec ? k_candidates<true> : k_candidates<false>, dim3(static_cast<unsigned>(regions)), dim3(kT), 0,
                     s, coeffs, M, w.sc, w.cand_key, w.cand_idx, w.cnt);
  VBM_LAUNCH_CHECK("candidates");
  if (rank) {
    hipLaunchKernelGGL(vec ? k_candidates_all<true> : k_candidates_all<false>, dim3(grid_cap(regions, 2048)), dim3(kT),
                       0, s, coeffs, M, K, regions, w.sc, w.cand_key, w.cand_idx, w.cnt);
    VBM_LAUNCH_CHECK("candidates_all");
  }
  const dim3 hist_grid(grid_cap(ceil_div(regions, kT / 64), kHistBlocks));
  const uint32_t K32 = static_cast<uint32_t>(K);
  hipLaunchKernelGGL(k_select_hist<0>, hist_grid, dim3(kT), 0, s, w.cand_key, w.cnt, regions, K32, w.sc);
  VBM_LAUNCH_CHECK("select_hist");
  hipLaunchKernelGGL(k_select_hist<1>, hist_grid, dim3(kT), 0, s, w.cand_key, w.cnt, regions, K32, w.sc);
  VBM_LAUNCH_CHECK("select_hist");
  hipLaunchKernelGGL(k_select_hist<2>, hist_grid, dim3(kT), 0, s, w.cand_key, w.cnt, regions, K32, w.sc);
  VBM_LAUNCH_CHECK("select_hist");
  hipLaunchKernelGGL(k_select_count, hist_grid, dim3(kT), 0, s, w.cand_key, w.cnt, regions, w.sc, w.sums);
  VBM_LAUNCH_CHECK("select_count");
  hipLaunchKernelGGL(k_select_groups, dim3(static_cast<unsigned>(ceil_div(regions, kGroup))), dim3(kT), 0, s, w.sums,
                     regions, w.sc);
  VBM_LAUNCH_CHECK("select_groups");
  hipLaunchKernelGGL(k_select_build, dim3(static_cast<unsigned>(regions)), dim3(kT), 0, s, coeffs, w.cand_key,
                     w.cand_idx, w.cnt, w.sc, w.sums, bank_dev, p, out, kept_index);
  VBM_LAUNCH_CHECK("select_build");
  if (opts->isotropic) {
    hipLaunchKernelGGL(k_isotropize, dim3(1), dim3(1024), 0, s, out, K);
    VBM_LAUNCH_CHECK("isotropize");
  }
  return VBM_OK;
}

extern "C" vbm_status vbm_construct_gaussians(const float* coeffs, int32_t G, int32_t J, const float* bank_dev,
                                              const int64_t* kept_index, int64_t n, const vbm_build_opts* opts,
                                              vbm_gaussians out, void* stream) {
  if (!coeffs || !bank_dev || !opts || (n > 0 && !kept_index) || !out.means || !out.scales || !out.quats ||
      !out.opacity || !out.rgb) {
    set_error("vbm_construct_gaussians: null pointer");
    return VBM_ERR_INVALID;
  }
  if (G < 2 || G > 1024 || J < 1 || J > 10 || (G % (1 << J)) != 0 || (G >> J) < 2) {
    set_error("vbm_construct_gaussians: bad G=%d J=%d", G, J);
    return VBM_ERR_INVALID;
  }
  if (n < 0 || out.stride < n) {
    set_error("vbm_construct_gaussians: need 0 <= n <= out.stride");
    return VBM_ERR_INVALID;
  }
  if ((opts->s_mode != 0 && opts->s_mode != 1) ||
      !(opts->opacity_min >= 0.0f && opts->opacity_min <= opts->opacity_max && opts->opacity_max <= 1.0f) ||
      (opts->isotropic != 0 && opts->isotropic != 1) || (opts->unit_weight != 0 && opts->unit_weight != 1)) {
    set_error("vbm_construct_gaussians: bad opts");
    return VBM_ERR_INVALID;
  }
  if (n == 0) return VBM_OK;
  BuildParams p;
  p.G = G;
  p.J = J;
  p.h = 2.0f / static_cast<float>(G);
  p.delta = opts->delta;
  p.op_min = opts->opacity_min;
  p.op_max = opts->opacity_max;
  p.s_mode = opts->s_mode;
  p.unit_weight = opts->unit_weight;
  p.M = static_cast<int64_t>(G) * G * G;
  hipLaunchKernelGGL(k_build, dim3(ceil_div(n, kT)), dim3(kT), 0, static_cast<hipStream_t>(stream), coeffs,
                     kept_index, n, bank_dev, p, out);
  VBM_LAUNCH_CHECK("construct");
  if (opts->isotropic) {
    hipLaunchKernelGGL(k_isotropize, dim3(1), dim3(1024), 0, static_cast<hipStream_t>(stream), out, n);
    VBM_LAUNCH_CHECK("isotropize");
  }
  return VBM_OK;
}
