// vbm_adaptive_select: adaptive per-subband coefficient selection (Supp. A: global budget
// allocation across subbands, joint multi-channel sparsification, robust MAD-based thresholding,
// top-K selection under sparsity constraints).
//
// Every subband of the packed layout (the LLL block, then the seven detail blocks of each level from the coarsest) is
// cut into chunks of 16384 coefficients that never straddle a subband; the passes after the joint norms take a chunk,
// or a quarter of one on small grids, per block.  The order statistics (the two medians and the K-th largest joint
// norm) come from radix selects on float32 bit patterns (non-negative floats order like their bits) with digits of 12,
// 10 and 10 bits, run for all subbands at once with per-subband histograms.  The pass that writes the joint norms also
// counts their first digit.  The two middle ranks of a median are selected side by side, and the K_band-th largest
// joint norm alongside the median of the joint norms (it does not depend on the threshold: when fewer than K_band
// values pass T, the K-th largest is the smallest value >= T, which the count pass finds).  A histogram is read by
// every block of the pass that follows it: each finds its subband's digit for itself, so that no launch stands between
// two passes.  Every keep/drop decision uses float32 values computed in a fixed order; energies and budgets are
// float64.  Per-subband counts are summed from per-block counts (no same-address atomics across blocks).  Nothing is
// read back to the host.
//
// Eleven launches.  At 256^3 with J = 4 the norms pass takes 64 us (its 320 MB at the rate of a large copy), the five
// histogram passes 15 to 30 us each (64 MB of norms at 13 us, the digit before and, where many keys share the prefix,
// the adds to the subband's bins), counting and writing 16 us each: 223 us a call, against 351 us with 8-bit digits and
// a launch for every step between the passes.
#include <hip/hip_runtime.h>

#include <cmath>

#include "block_scan.h"
#include "common.h"

namespace vbm {
namespace {

constexpr int kT = 256;
constexpr int kChunk = 16384;
constexpr int kPer = kChunk / kT;
constexpr int kMaxBands = 7 * 10 + 1;

struct BandTable {
  int32_t nb;
  int32_t part_shift;              // a chunk is 2^part_shift parts
  int64_t off[kMaxBands];
  int64_t n[kMaxBands];
  int64_t chunk0[kMaxBands + 1];   // first chunk of each subband; chunk0[nb] = number of chunks
};

// Select targets: 0 and 1 the two middle ranks (of v, then of |v - median|), 2 the K_band-th
// largest v (selected alongside the median; active when 1 <= K_band <= N).
constexpr int kTargets = 3;

// Digits 0 to 2 of the first select (of v) and 3 to 5 of the second (of |v - median|), each from the top.  A digit's
// histogram has a set of bins for every target whose higher digits differ (the first digit has one for all).
constexpr int kDigits = 6;
constexpr int digit_shift(int d) { return d % 3 == 0 ? 20 : d % 3 == 1 ? 10 : 0; }
constexpr int digit_bins(int d) { return d % 3 == 0 ? 4096 : 1024; }
constexpr int digit_sets(int d) { return d % 3 == 0 ? 1 : d < 3 ? 3 : 2; }
constexpr int digit_base(int d) { return d == 0 ? 0 : digit_base(d - 1) + digit_sets(d - 1) * digit_bins(d - 1); }
constexpr int kHistWords = digit_base(kDigits);   // per subband

struct Selection {
  uint32_t prefix[kTargets];   // key bits fixed so far, per select target
  uint32_t rank[kTargets];     // ascending 0-based rank still to find inside the prefix's bucket
};

struct BandState {
  Selection sel[kDigits];   // after each digit
  uint32_t use2;            // target 2 active
  uint32_t vmin;            // smallest v >= T (bit pattern; all ones when none)
  double E, quotient;       // reference energy, K_tot S / sum S
  int64_t K_band;           // max(min_band, floor(quotient))
  float med, mad, sigma, T, vK, thr;
  uint32_t C, K;            // #(v >= T), min(K_band, C)
  uint32_t kept, pad;
};

__device__ __forceinline__ int band_of(const BandTable& bt, int64_t chunk) {
  int b = 0;
  while (b + 1 < bt.nb && chunk >= bt.chunk0[b + 1]) ++b;
  return b;
}

// [begin, end) of chunk `chunk` inside subband b.
__device__ __forceinline__ void chunk_range(const BandTable& bt, int b, int64_t chunk, int64_t& begin, int64_t& end) {
  begin = bt.off[b] + (chunk - bt.chunk0[b]) * kChunk;
  end = min(begin + kChunk, bt.off[b] + bt.n[b]);
}

// The same for part `part` (end <= begin: the subband ends before it), and its subband.
__device__ __forceinline__ int part_range(const BandTable& bt, uint32_t part, int64_t& begin, int64_t& end) {
  const int64_t chunk = part >> bt.part_shift;
  const int b = band_of(bt, chunk);
  chunk_range(bt, b, chunk, begin, end);
  const int64_t len = kChunk >> bt.part_shift;
  begin += (part - (static_cast<uint32_t>(chunk) << bt.part_shift)) * len;
  end = min(begin + len, end);
  return b;
}

// Keys begin + q * 256 + thread, q < 16, with indices past `end` clamped to end - 1 (begin < end): the loads are
// unconditional so that all sixteen are in flight at once.
__device__ __forceinline__ void load16(const uint32_t* __restrict__ keys, int64_t begin, int64_t end,
                                       uint32_t (&k)[16]) {
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int64_t i = begin + static_cast<int64_t>(q) * kT + threadIdx.x;
    k[q] = keys[i < end ? i : end - 1];
  }
}

__device__ __forceinline__ double block_sum_f64(double v, double* s_red) {
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  if (lane_id() == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kT / 64; ++w) t += s_red[w];
  __syncthreads();
  return t;
}

__device__ __forceinline__ uint32_t block_min_u32(uint32_t v, uint32_t* s_red) {
  for (int d = 32; d >= 1; d >>= 1) v = min(v, static_cast<uint32_t>(__shfl_xor(v, d, 64)));
  if (lane_id() == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t t = 0xFFFFFFFFu;
  for (int w = 0; w < kT / 64; ++w) t = min(t, s_red[w]);
  __syncthreads();
  return t;
}

__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t* s_red) {
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  if (lane_id() == 0) s_red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t t = 0;
  for (int w = 0; w < kT / 64; ++w) t += s_red[w];
  __syncthreads();
  return t;
}

// Adds the wave's digits to LDS bins.  The lanes that share the first one's digit are added at once: fields with many
// equal values (zeros outside the transfer function's support) would else queue 64 adds at one address.
__device__ __forceinline__ void hist_add(uint32_t* __restrict__ h, uint32_t d, bool valid) {
  const uint64_t m = __ballot(valid);
  if (m == 0) return;
  const int lead = __builtin_ctzll(m);
  const uint32_t d0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(d), lead));
  const bool same = valid && d == d0;
  const uint32_t n = static_cast<uint32_t>(__popcll(__ballot(same)));
  if (valid && (!same || static_cast<int>(lane_id()) == lead)) atomicAdd(&h[d], same ? n : 1u);
}

#pragma clang fp contract(off)
// Joint norm sqrt(((R^2 + G^2) + B^2) + A^2) in float32 (the order of the top-K key) as its bit
// pattern, its first digit's histogram, and the chunk's reference-channel energy in float64 (fixed summation order).
__global__ __launch_bounds__(kT) void k_af_norm(const float* __restrict__ coeffs, int64_t M, BandTable bt, int ref,
                                               uint32_t* __restrict__ keys, double* __restrict__ epart,
                                               uint32_t* __restrict__ ghist) {
  __shared__ double s_red[kT / 64];
  __shared__ uint32_t h[digit_bins(0)];
  const int b = band_of(bt, blockIdx.x);
  int64_t begin, end;
  chunk_range(bt, b, blockIdx.x, begin, end);
  for (int x = threadIdx.x; x < digit_bins(0); x += kT) h[x] = 0;
  __syncthreads();
  double e = 0.0;
  for (int r0 = 0; r0 < kPer; r0 += 4) {
    // four coefficients (sixteen loads) in flight; indices past the chunk are clamped and unused
    float c[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = begin + static_cast<int64_t>(r0 + q) * kT + threadIdx.x;
      const int64_t j = i < end ? i : end - 1;
#pragma unroll
      for (int ch = 0; ch < 4; ++ch) c[q][ch] = coeffs[ch * M + j];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t i = begin + static_cast<int64_t>(r0 + q) * kT + threadIdx.x;
      const float cr = c[q][0], cg = c[q][1], cb = c[q][2], ca = c[q][3];
      const uint32_t k = __float_as_uint(sqrt_rn_f32(((cr * cr + cg * cg) + cb * cb) + ca * ca));
      hist_add(h, k >> digit_shift(0), i < end);
      if (i >= end) continue;
      keys[i] = k;
      const double x = static_cast<double>(ref == 0 ? cr : ref == 1 ? cg : ref == 2 ? cb : ca);
      e += x * x;
    }
  }
  e = block_sum_f64(e, s_red);
  if (threadIdx.x == 0) epart[blockIdx.x] = e;
  uint32_t* g = ghist + static_cast<int64_t>(b) * kHistWords;
  for (int x = threadIdx.x; x < digit_bins(0); x += kT)
    if (h[x]) atomicAdd(&g[x], h[x]);
}

// E per subband and the budgets K_{j,o} = max(min_band, floor(K_tot S / sum S)), S = E^alpha N^beta, in one block.  A
// wave sums a subband's chunks in a fixed order: 256 partial sums (four per lane), added in four groups of 64.
constexpr int kBudgetThreads = 1024;
__global__ __launch_bounds__(kBudgetThreads) void k_af_budget(BandTable bt, const double* __restrict__ epart,
                                                             BandState* __restrict__ st, int64_t K_tot, double alpha,
                                                             double beta, int64_t min_band) {
  __shared__ double s_E[kMaxBands];
  __shared__ double s_S[kMaxBands];
  __shared__ double s_tot;
  for (int b = threadIdx.x >> 6; b < bt.nb; b += kBudgetThreads / 64) {
    double e[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t c = bt.chunk0[b] + lane_id(); c < bt.chunk0[b + 1]; c += 256) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (c + 64 * k < bt.chunk0[b + 1]) e[k] += epart[c + 64 * k];
    }
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      for (int d = 32; d >= 1; d >>= 1) e[k] += __shfl_xor(e[k], d, 64);
      t += e[k];
    }
    if (lane_id() == 0) s_E[b] = t;
  }
  __syncthreads();
  const int b = threadIdx.x;
  if (b < bt.nb) s_S[b] = pow(s_E[b], alpha) * pow(static_cast<double>(bt.n[b]), beta);
  __syncthreads();
  if (b == 0) {
    double t = 0.0;
    for (int k = 0; k < bt.nb; ++k) t += s_S[k];
    s_tot = t;
  }
  __syncthreads();
  if (b < bt.nb) {
    const double q = s_tot == 0.0 ? 0.0 : static_cast<double>(K_tot) * s_S[b] / s_tot;
    const double f = floor(q);
    const int64_t K_band = f > static_cast<double>(min_band) ? static_cast<int64_t>(f) : min_band;
    st[b].E = s_E[b];
    st[b].quotient = q;
    st[b].K_band = K_band;
    st[b].use2 = K_band >= 1 && K_band <= bt.n[b] ? 1u : 0u;
  }
}

// Key of a coefficient for a select: the joint norm (mode 0) or its distance to the subband's
// median (mode 1), both non-negative float32 bit patterns.
__device__ __forceinline__ uint32_t select_key(uint32_t v, int mode, float med) {
  return mode == 0 ? v : __float_as_uint(fabsf(__uint_as_float(v) - med));
}

// Set of bins that holds target t's next digit: targets with the same prefix share the first one's.
__device__ __forceinline__ int target_set(const uint32_t (&p)[kTargets], int t) {
  return t >= 1 && p[t] != p[0] ? (t == 2 && p[2] == p[1] ? 1 : t) : 0;
}

// Finds digit D of subband b's targets from its histogram: the bin that holds each target's rank.  Every thread of the
// block calls it; each thread owns consecutive bins.
template <int D>
__device__ __forceinline__ Selection pick_digit(const BandTable& bt, int b, const BandState& st,
                                                const uint32_t* __restrict__ ghist) {
  constexpr int kOwn = digit_bins(D) / kT;
  constexpr int kActive = D < 3 ? kTargets : 2;
  __shared__ uint32_t s_digit[kTargets], s_rank[kTargets];
  Selection s;
  if (D % 3 == 0) {
    for (int t = 0; t < kTargets; ++t) s.prefix[t] = 0u;
    s.rank[0] = static_cast<uint32_t>((bt.n[b] - 1) / 2);
    s.rank[1] = static_cast<uint32_t>(bt.n[b] / 2);
    s.rank[2] = D < 3 && st.use2 ? static_cast<uint32_t>(bt.n[b] - st.K_band) : 0u;
  } else {
    s = st.sel[D > 0 ? D - 1 : 0];
  }
  const uint32_t* g = ghist + static_cast<int64_t>(b) * kHistWords + digit_base(D);
  uint4 v[kActive][kOwn / 4];
#pragma unroll
  for (int t = 0; t < kActive; ++t) {
    const int set = digit_sets(D) == 1 ? 0 : target_set(s.prefix, t);
#pragma unroll
    for (int k = 0; k < kOwn / 4; ++k)
      v[t][k] = reinterpret_cast<const uint4*>(g + set * digit_bins(D) + threadIdx.x * kOwn)[k];
  }
#pragma unroll
  for (int t = 0; t < kActive; ++t) {
    uint32_t sum = 0, tot;
#pragma unroll
    for (int k = 0; k < kOwn / 4; ++k) sum += v[t][k].x + v[t][k].y + v[t][k].z + v[t][k].w;
    uint32_t below = block_excl_scan(sum, &tot);
    if (below <= s.rank[t] && s.rank[t] < below + sum) {   // this thread's bins hold the rank
      uint32_t digit = threadIdx.x * kOwn;
#pragma unroll
      for (int k = 0; k < kOwn; ++k) {
        const uint4& q = v[t][k / 4];
        const uint32_t c = k % 4 == 0 ? q.x : k % 4 == 1 ? q.y : k % 4 == 2 ? q.z : q.w;
        if (below <= s.rank[t] && s.rank[t] < below + c) {
          s_digit[t] = digit + k;
          s_rank[t] = s.rank[t] - below;
        }
        below += c;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kActive; ++t) {
    if (t == 2 && !st.use2) continue;
    s.prefix[t] |= s_digit[t] << digit_shift(D);
    s.rank[t] = s_rank[t];
  }
  return s;
}

__device__ __forceinline__ float mid_mean(const Selection& s) {
  return (__uint_as_float(s.prefix[0]) + __uint_as_float(s.prefix[1])) * 0.5f;
}

// Finds digit D - 1 and counts digit D over the keys whose higher digits match a target's (target 2 in the first select
// only).  The first block of a subband keeps the digit, and the median once it is known, for the passes that follow.
template <int D>
__global__ __launch_bounds__(kT) void k_af_hist(const uint32_t* __restrict__ keys, BandTable bt,
                                               BandState* __restrict__ st, uint32_t* __restrict__ ghist) {
  constexpr int kSets = digit_sets(D), kBins = digit_bins(D);
  constexpr int kMode = D < 3 ? 0 : 1;
  __shared__ uint32_t h[kSets * kBins];
  int64_t begin, end;
  const int b = part_range(bt, blockIdx.x, begin, end);
  if (begin >= end) return;
  for (int x = threadIdx.x; x < kSets * kBins; x += kT) h[x] = 0;
  const Selection s = pick_digit<D - 1>(bt, b, st[b], ghist);   // synchronises
  const float med = D == 3 ? mid_mean(s) : kMode == 1 ? st[b].med : 0.0f;
  if (threadIdx.x == 0 && begin == bt.off[b]) {
    st[b].sel[D - 1] = s;
    if (D == 3) st[b].med = med;
  }
  constexpr uint32_t hi_mask = D % 3 == 0 ? 0u : 0xFFFFFFFFu << digit_shift(D > 0 ? D - 1 : 0);
  const bool own1 = kSets > 1 && s.prefix[1] != s.prefix[0];   // targets with bins of their own
  const bool own2 = kSets > 2 && st[b].use2 != 0u && s.prefix[2] != s.prefix[0] && s.prefix[2] != s.prefix[1];
  for (int64_t i0 = begin; i0 < end; i0 += 16 * kT) {
    uint32_t kk[16];
    load16(keys, i0, end, kk);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const bool in = i0 + static_cast<int64_t>(q) * kT + threadIdx.x < end;
      const uint32_t k = select_key(kk[q], kMode, med);
      const uint32_t d = (k >> digit_shift(D)) & static_cast<uint32_t>(kBins - 1);
      if (kSets == 1) {
        hist_add(h, d, in);
        continue;
      }
      const uint32_t hk = k & hi_mask;
      int set = hk == s.prefix[0] ? 0 : own1 && hk == s.prefix[1] ? 1 : own2 && hk == s.prefix[2] ? 2 : -1;
      hist_add(h, static_cast<uint32_t>(set) * kBins + d, in && set >= 0);
    }
  }
  __syncthreads();
  uint32_t* g = ghist + static_cast<int64_t>(b) * kHistWords + digit_base(D);
  for (int x = threadIdx.x; x < kSets * kBins; x += kT)
    if (h[x]) atomicAdd(&g[x], h[x]);
}

// MAD, sigma = MAD / 0.6745 and the threshold T = lambda sigma (float32); then, per part, #(v >= T), the smallest such
// v and the number of v at or above the other threshold that k_af_decide may choose: max(T, K_band-th largest v), or
// +inf where nothing is to be kept (K_band = 0, or T not a number).  Keys are non-negative float bit patterns, so their
// unsigned order is the float order.
__global__ __launch_bounds__(kT) void k_af_count(const uint32_t* __restrict__ keys, BandTable bt,
                                                BandState* __restrict__ st, const uint32_t* __restrict__ ghist,
                                                float lambda, uint2* __restrict__ cnt, uint32_t* __restrict__ cmin) {
  __shared__ uint32_t s_red[kT / 64];
  int64_t begin, end;
  const int b = part_range(bt, blockIdx.x, begin, end);
  if (begin >= end) {
    if (threadIdx.x == 0) {
      cnt[blockIdx.x] = make_uint2(0u, 0u);
      cmin[blockIdx.x] = 0xFFFFFFFFu;
    }
    return;
  }
  const Selection s = pick_digit<5>(bt, b, st[b], ghist);
  const float mad = mid_mean(s);
  const float sigma = __fdiv_rn(mad, 0.6745f);
  const float T = lambda * sigma;
  if (threadIdx.x == 0 && begin == bt.off[b]) {
    st[b].mad = mad;
    st[b].sigma = sigma;
    st[b].T = T;
  }
  const float T2 = st[b].K_band < 1 || T != T ? __builtin_inff() : fmaxf(T, __uint_as_float(st[b].sel[2].prefix[2]));
  uint32_t c = 0, c2 = 0, mn = 0xFFFFFFFFu;
  for (int64_t i0 = begin; i0 < end; i0 += 16 * kT) {
    uint32_t kk[16];
    load16(keys, i0, end, kk);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const bool in = i0 + static_cast<int64_t>(q) * kT + threadIdx.x < end;
      const float v = __uint_as_float(kk[q]);
      c += in && v >= T ? 1u : 0u;
      c2 += in && v >= T2 ? 1u : 0u;
      mn = in && v >= T ? min(mn, kk[q]) : mn;
    }
  }
  c = block_sum_u32(c, s_red);
  c2 = block_sum_u32(c2, s_red);
  mn = block_min_u32(mn, s_red);
  if (threadIdx.x == 0) {
    cnt[blockIdx.x] = make_uint2(c, c2);
    cmin[blockIdx.x] = mn;
  }
}

// One block per subband: C = #(v >= T), K = min(K_band, C) and v_(K), the K-th largest joint norm: when K_band <= C it
// is the K_band-th largest, found by target 2 of the first select; otherwise K = C and the C largest values are exactly
// those >= T, so v_(C) is the smallest v >= T and all C are kept.  Keep threshold max(T, v_(K)), or +inf when K = 0.
// offs: kept coefficients of the subband before each part.
__global__ __launch_bounds__(kT) void k_af_decide(BandTable bt, const uint2* __restrict__ cnt,
                                                 const uint32_t* __restrict__ cmin, uint32_t* __restrict__ offs,
                                                 BandState* __restrict__ st) {
  __shared__ uint32_t s_red[kT / 64];
  const int b = blockIdx.x;
  const int64_t p0 = bt.chunk0[b] << bt.part_shift, p1 = bt.chunk0[b + 1] << bt.part_shift;
  uint32_t c = 0, mn = 0xFFFFFFFFu;
  for (int64_t p = p0 + threadIdx.x; p < p1; p += kT) {
    c += cnt[p].x;
    mn = min(mn, cmin[p]);
  }
  c = block_sum_u32(c, s_red);
  mn = block_min_u32(mn, s_red);
  const int64_t C = static_cast<int64_t>(c), K_band = st[b].K_band;
  const int64_t K = K_band < C ? K_band : C;
  const bool all = K >= 1 && K_band > C;
  uint32_t kept = 0;
  for (int64_t q0 = p0; q0 < p1; q0 += kT) {
    const int64_t p = q0 + threadIdx.x;
    const uint2 n2 = p < p1 ? cnt[p] : make_uint2(0u, 0u);
    uint32_t tot;
    const uint32_t before = block_excl_scan(all ? n2.x : n2.y, &tot);
    if (p < p1) offs[p] = kept + before;
    kept += tot;
  }
  if (threadIdx.x == 0) {
    const float vK = K < 1 ? __builtin_inff() : __uint_as_float(all ? mn : st[b].sel[2].prefix[2]);
    st[b].C = c;
    st[b].vmin = mn;
    st[b].K = static_cast<uint32_t>(K);
    st[b].vK = vK;
    st[b].thr = K >= 1 ? fmaxf(st[b].T, vK) : __builtin_inff();
    st[b].kept = kept;
  }
}

// Kept count and the per-subband statistics.
__device__ __forceinline__ void write_stats(const BandTable& bt, const BandState* __restrict__ st,
                                            int64_t* __restrict__ count_dev, double* __restrict__ stats) {
  const int b = threadIdx.x;
  if (b == 0) {
    uint32_t total = 0;
    for (int k = 0; k < bt.nb; ++k) total += st[k].kept;
    count_dev[0] = static_cast<int64_t>(total);
  }
  if (b >= bt.nb || !stats) return;
  const BandState& s = st[b];
  double* o = stats + static_cast<int64_t>(b) * VBM_ADAPTIVE_STATS;
  o[0] = s.E;
  o[1] = static_cast<double>(bt.n[b]);
  o[2] = s.quotient;
  o[3] = static_cast<double>(s.K_band);
  o[4] = s.med;
  o[5] = s.mad;
  o[6] = s.sigma;
  o[7] = s.T;
  o[8] = s.C;
  o[9] = s.K;
  o[10] = s.vK;
  o[11] = static_cast<double>(s.kept);
}

// The kept coefficients' indices in ascending order, a part per block.
__global__ __launch_bounds__(kT) void k_af_write(const uint32_t* __restrict__ keys, BandTable bt,
                                                const BandState* __restrict__ st, const uint32_t* __restrict__ offs,
                                                int64_t capacity, int64_t* __restrict__ kept,
                                                int64_t* __restrict__ count_dev, double* __restrict__ stats) {
  __shared__ uint32_t s_red[kT / 64];
  if (blockIdx.x == gridDim.x - 1) {   // one block more than there are parts
    write_stats(bt, st, count_dev, stats);
    return;
  }
  int64_t begin, end;
  const int b = part_range(bt, blockIdx.x, begin, end);
  const uint32_t part_end = static_cast<uint32_t>(bt.chunk0[b + 1]) << bt.part_shift;
  const uint32_t next = blockIdx.x + 1 < part_end ? offs[blockIdx.x + 1] : st[b].kept;
  if (next == offs[blockIdx.x]) return;   // nothing kept in this part (uniform for the block)
  const uint32_t bands =
      block_sum_u32(static_cast<int>(threadIdx.x) < b ? st[threadIdx.x].kept : 0u, s_red);   // of the subbands before
  // Sub-rounds of 4096 coefficients in which each thread owns 16 consecutive ones, so the block's
  // scan of the per-thread counts numbers the kept ones in ascending index order.  A full sub-round
  // that starts on a 16-byte boundary (subband sizes are cubes of even numbers except for an odd
  // coarsest side) is read as four 16-byte vectors per thread.
  constexpr int kSub = 16;
  const float thr = st[b].thr;
  int64_t pos0 = static_cast<int64_t>(bands + offs[blockIdx.x]);
  for (int64_t base = begin; base < end; base += kSub * kT) {
    uint32_t f = 0;
    const int64_t first = base + static_cast<int64_t>(threadIdx.x) * kSub;
    if (base + kSub * kT <= end && (reinterpret_cast<uintptr_t>(keys + base) & 15u) == 0) {
      const uint4* src = reinterpret_cast<const uint4*>(keys + first);
#pragma unroll
      for (int q = 0; q < kSub / 4; ++q) {
        const uint4 k4 = src[q];
        f |= (__uint_as_float(k4.x) >= thr ? 1u : 0u) << (4 * q);
        f |= (__uint_as_float(k4.y) >= thr ? 1u : 0u) << (4 * q + 1);
        f |= (__uint_as_float(k4.z) >= thr ? 1u : 0u) << (4 * q + 2);
        f |= (__uint_as_float(k4.w) >= thr ? 1u : 0u) << (4 * q + 3);
      }
    } else {
      for (int r = 0; r < kSub; ++r) {
        const int64_t i = first + r;
        if (i < end && __uint_as_float(keys[i]) >= thr) f |= 1u << r;
      }
    }
    uint32_t tot;
    int64_t pos = pos0 + block_excl_scan(static_cast<uint32_t>(__popc(f)), &tot);
    for (int r = 0; r < kSub; ++r) {
      if (!((f >> r) & 1u)) continue;
      if (pos < capacity) kept[pos] = base + static_cast<int64_t>(threadIdx.x) * kSub + r;
      ++pos;
    }
    pos0 += tot;
  }
}

// A block takes a whole chunk where the grid has enough of them for the chip, else a quarter.
// Whole chunks against quarters, a call: 64^3 125 against 92 us, 160^3 (about 270 chunks) 137 against 120, 192^3 (about
// 460) 145 against 149, 256^3 223 against 292: below the line blocks are missing, above it each block's share of the
// histograms' upkeep (finding the digit, clearing and adding up the bins) costs more than the reading.
constexpr int64_t kWholeChunks = 400;

bool make_table(int G, int J, BandTable* bt) {
  if (7 * J + 1 > kMaxBands) return false;
  bt->nb = 7 * J + 1;
  int64_t off = 0, chunk = 0;
  for (int b = 0; b < bt->nb; ++b) {
    const int j = b == 0 ? J : J - (b - 1) / 7;
    const int64_t side = G >> j;
    bt->off[b] = off;
    bt->n[b] = side * side * side;
    bt->chunk0[b] = chunk;
    off += bt->n[b];
    chunk += ceil_div(bt->n[b], kChunk);
  }
  bt->chunk0[bt->nb] = chunk;
  bt->part_shift = chunk >= kWholeChunks ? 0 : 2;
  return off == static_cast<int64_t>(G) * G * G;
}

struct AdaptiveWs {
  uint32_t* keys;
  double* epart;
  uint2* cnt;
  uint32_t* cmin;
  uint32_t* offs;
  BandState* st;
  uint32_t* ghist;
};

AdaptiveWs carve(Carver& c, int64_t M, const BandTable& bt) {
  const int64_t chunks = bt.chunk0[bt.nb], parts = chunks << bt.part_shift;
  AdaptiveWs w;
  w.keys = c.take<uint32_t>(M);
  w.epart = c.take<double>(chunks);
  w.cnt = c.take<uint2>(parts);
  w.cmin = c.take<uint32_t>(parts);
  w.offs = c.take<uint32_t>(parts);
  w.st = c.take<BandState>(kMaxBands);
  w.ghist = c.take<uint32_t>(static_cast<size_t>(bt.nb) * kHistWords);
  return w;
}

bool grid_ok(int G, int J) { return G >= 2 && G <= 1024 && J >= 1 && J <= 10 && (G % (1 << J)) == 0 && (G >> J) >= 2; }

}  // namespace
}  // namespace vbm

using namespace vbm;

extern "C" size_t vbm_adaptive_workspace_size(int32_t G, int32_t J) {
  BandTable bt;
  if (!grid_ok(G, J) || !make_table(G, J, &bt)) return 0;
  Carver c(nullptr);
  carve(c, static_cast<int64_t>(G) * G * G, bt);
  return align_up(c.off, 256);
}

extern "C" vbm_status vbm_adaptive_select(const float* coeffs, int32_t G, int32_t J, const vbm_adaptive_opts* opts,
                                          int64_t capacity, int64_t* kept_index, int64_t* count_dev,
                                          double* band_stats, void* ws, size_t ws_bytes, void* stream) {
  if (!coeffs || !opts || !kept_index || !count_dev || !ws) {
    set_error("vbm_adaptive_select: null pointer");
    return VBM_ERR_INVALID;
  }
  BandTable bt;
  if (!grid_ok(G, J) || !make_table(G, J, &bt)) {
    set_error("vbm_adaptive_select: bad G=%d J=%d", G, J);
    return VBM_ERR_INVALID;
  }
  const int64_t M = static_cast<int64_t>(G) * G * G;
  if (opts->K_tot < 1 || opts->K_tot > M || opts->min_band < 0 || opts->min_band > M ||
      !(opts->lambda >= 0.0f) || !std::isfinite(opts->lambda) || !(opts->alpha >= 0.0) || !(opts->beta >= 0.0) ||
      !std::isfinite(opts->alpha) || !std::isfinite(opts->beta) || opts->ref_channel < 0 || opts->ref_channel > 3) {
    set_error("vbm_adaptive_select: need 1 <= K_tot <= G^3, 0 <= min_band <= G^3, finite lambda, alpha, "
              "beta >= 0 and ref_channel in 0..3");
    return VBM_ERR_INVALID;
  }
  if (capacity < 0) {
    set_error("vbm_adaptive_select: negative capacity");
    return VBM_ERR_INVALID;
  }
  if (ws_bytes < vbm_adaptive_workspace_size(G, J)) {
    set_error("vbm_adaptive_select: workspace %zu < %zu", ws_bytes, vbm_adaptive_workspace_size(G, J));
    return VBM_ERR_WORKSPACE;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  Carver c(ws);
  const AdaptiveWs w = carve(c, M, bt);
  const int64_t chunks = bt.chunk0[bt.nb];
  const dim3 cg(static_cast<unsigned>(chunks)), pg(static_cast<unsigned>(chunks << bt.part_shift)), blk(kT);

  ClearList cl;
  cl.add(w.ghist, static_cast<int64_t>(bt.nb) * kHistWords);
  VBM_TRY(clear_words(cl, s));
  hipLaunchKernelGGL(k_af_norm, cg, blk, 0, s, coeffs, M, bt, opts->ref_channel, w.keys, w.epart, w.ghist);
  VBM_LAUNCH_CHECK("adaptive_norm");
  hipLaunchKernelGGL(k_af_budget, dim3(1), dim3(kBudgetThreads), 0, s, bt, w.epart, w.st, opts->K_tot, opts->alpha,
                     opts->beta, static_cast<int64_t>(opts->min_band));
  VBM_LAUNCH_CHECK("adaptive_budget");
  // two radix selects: median(v) together with the K_band-th largest v, then median(|v - median|)
  hipLaunchKernelGGL(k_af_hist<1>, pg, blk, 0, s, w.keys, bt, w.st, w.ghist);
  hipLaunchKernelGGL(k_af_hist<2>, pg, blk, 0, s, w.keys, bt, w.st, w.ghist);
  hipLaunchKernelGGL(k_af_hist<3>, pg, blk, 0, s, w.keys, bt, w.st, w.ghist);
  hipLaunchKernelGGL(k_af_hist<4>, pg, blk, 0, s, w.keys, bt, w.st, w.ghist);
  hipLaunchKernelGGL(k_af_hist<5>, pg, blk, 0, s, w.keys, bt, w.st, w.ghist);
  VBM_LAUNCH_CHECK("adaptive_hist");
  hipLaunchKernelGGL(k_af_count, pg, blk, 0, s, w.keys, bt, w.st, w.ghist, opts->lambda, w.cnt, w.cmin);
  VBM_LAUNCH_CHECK("adaptive_count");
  hipLaunchKernelGGL(k_af_decide, dim3(static_cast<unsigned>(bt.nb)), blk, 0, s, bt, w.cnt, w.cmin, w.offs, w.st);
  VBM_LAUNCH_CHECK("adaptive_decide");
  hipLaunchKernelGGL(k_af_write, dim3(pg.x + 1), blk, 0, s, w.keys, bt, w.st, w.offs, capacity, kept_index, count_dev,
                     band_stats);
  VBM_LAUNCH_CHECK("adaptive_write");
  return VBM_OK;
}
