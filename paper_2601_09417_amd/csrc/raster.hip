// Front-to-back alpha compositing and its reverse-order backward (Sec. 3, the Gaussian mixture
// rendered by the 3DGS rasteriser cited in Sec. 4.4).
//
// Work decomposition: one wave64 per 256 pixels of a tile (a 16x16 tile is one wave, a 32x32 tile
// four independent waves, an 8x8 tile one wave with one pixel per lane), each lane owning
// PPL = 4 pixels of ONE pixel column (rows 64 / TILE apart), so the horizontal offset to a
// Gaussian's centre is shared by a lane's pixels.  In a batch that does not fill the chip that way the
// lists of 16x16 tiles are shared by four waves, a band of four rows and one pixel per lane each.  The tile's
// depth-sorted list is walked by every wave in lockstep, with each Gaussian's 36-byte record wave-uniform.
// The forward stages the list in LDS: lanes gather an entry's record each with vector loads into a batch
// that the wave then reads entry by entry.  The backward reads each record through the scalar data
// cache into SGPRs, one list step ahead of its use (no LDS, no barriers, no per-lane copies of a uniform
// value), or from LDS batches as the plan chooses.  Either way the per-Gaussian load cost is amortised over
// the wave's pixels; a vector load of a uniform address instead would move 64 lanes' copies through the
// texture address and data units, which the list walk would saturate.
//
// The record holds the exponent in base 2 with the log-opacity folded in:
//   e2(d) = hA dx^2 + hB dx dy + hC dy^2 + log2(o) = log2(o) + power(d) log2(e),
// so alpha = min(0.99, 2^e2) costs one exponential and no multiply by the opacity.  Projection
// keeps only Gaussians with a positive-definite conic, for which power <= 0 at every pixel, so a
// "skip when power > 0" guard could only fire on float32 rounding near the centre and is left out.
// The forward keeps each pixel's transmittance in place; a pixel that stops records its list
// position as n_contrib and parks at a far row, where alpha underflows to zero.
//
// The backward walks the list in reverse from the wave's largest n_contrib, recomputes each
// pixel's transmittance from final_T by division and carries one scalar per pixel for the colour
// behind the current Gaussian (see bwd_step).  The geometric gradient is accumulated as three
// per-lane moments of dL/dpower (sum, first and second moment in dy); the lane's column offset dx
// turns them into the five sums the 2D parameters need.  Nine per-wave sums are then formed by
// cross-row lane swaps and a DPP reduction inside 16-lane rows (one value per lane; in large batches through
// LDS, two entries at a time: see kSumRow), and nine lanes
// issue one float atomic each into the item's 64-byte accumulator row (one cache segment per pair
// instead of nine lines) -- only when some pixel contributed.  The atomics add those raw moments;
// the projection backward turns them into mean/conic/opacity gradients with the item's conic,
// since that map is linear.
#include <hip/hip_runtime.h>

#include "common.h"
#include "composite.h"

namespace vbm {

constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kAlphaMax = 0.99f;
constexpr float kTMin = 1e-4f;

template <int TILE>
struct TileCfg {
  static constexpr int kPix = TILE * TILE;
  static constexpr int kWaves = kPix >= 256 ? kPix / 256 : 1;
  static constexpr int kPPL = kPix / (64 * kWaves);  // pixels per lane
  static constexpr int kThreads = 64 * kWaves;
  static_assert(64 % TILE == 0, "a lane's pixels must share one column");
};

__device__ __forceinline__ int find_view(const DevView* __restrict__ views, int n_views, int tile) {
  int lo = 0, hi = n_views - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (views[mid].tile_offset <= tile) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// One Gaussian's compositing record (wave-uniform values).
struct Rec {
  float mx, my, hA, hB, hC, lo, r, g, b;
};

__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// The record of a (wave-uniform) pair value, fetched through the scalar data cache into SGPRs.
// The item id is clamped to the record arrays (a past-the-end or empty-list step reads a valid
// record that it then ignores).
__device__ __forceinline__ Rec load_rec_s(const float4* __restrict__ crec, const float* __restrict__ cblue,
                                          uint32_t pv, uint32_t imax) {
  const uint32_t it = min(pv & kItemMask, imax);
  const float4 a = crec[2 * it];
  const float4 b = crec[2 * it + 1];
  Rec r;
  r.mx = a.x;
  r.my = a.y;
  r.hA = a.z;
  r.hB = a.w;
  r.hC = b.x;
  r.lo = b.y;
  r.r = b.z;
  r.g = b.w;
  r.b = cblue[it];
  return r;
}

// Waits for every scalar load in flight (they may complete out of order, so only a full wait
// identifies one): the list walks call it where the next record's loads are about to be issued,
// so that the wait covers the record requested one step earlier and not the next one.
__device__ __forceinline__ void wait_scalar_loads() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// True when the predicate holds on some active lane: one scalar test of the predicate's lane mask.
__device__ __forceinline__ bool wave_any(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// Base-2 exponent of the Gaussian at a pixel whose per-lane terms u = hA dx^2 + log2(o) and
// v = hB dx are precomputed; one expression shared by the forward and the backward so that both
// take bit-identical skip / contribute decisions.
__device__ __forceinline__ float exponent2(const Rec& r, float u, float v, float dy) {
  return fmaf(fmaf(r.hC, dy, v), dy, u);
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

// One step of a reduce-scatter inside 16-lane rows: lanes with `hi` clear keep value a, the others
// value b, each adding its DPP partner's copy (the partner always has the opposite `hi`).
template <int CTRL>
__device__ __forceinline__ float rs_pair(float a, float b, bool hi) {
  const float keep = hi ? b : a;
  const float send = hi ? a : b;
  return keep + dpp_move<CTRL>(send);
}
template <int CTRL>
__device__ __forceinline__ float rs_single(float v) {
  return v + dpp_move<CTRL>(v);
}

constexpr int kRowMirror = 0x140;
constexpr int kRowHalfMirror = 0x141;
constexpr int kQuadXor2 = 0x4E;  // quad_perm [2,3,0,1]
constexpr int kQuadXor1 = 0xB1;  // quad_perm [1,0,3,2]

// Wave sums of nine values (every lane active).  Lane l < 16 ends with the sum of value
// rs_index(l): even lanes l hold value 4 b1 + 2 b2 + b3 (b_i = bit i of l), odd lanes value 8.
__device__ __forceinline__ float reduce_scatter9(const float g[9], int lane) {
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
  const float A = rs_pair<kRowMirror>(g[0], g[1], b3);
  const float B = rs_pair<kRowMirror>(g[2], g[3], b3);
  const float C = rs_pair<kRowMirror>(g[4], g[5], b3);
  const float D = rs_pair<kRowMirror>(g[6], g[7], b3);
  float E = rs_single<kRowMirror>(g[8]);
  const float F = rs_pair<kRowHalfMirror>(A, B, b2);
  const float G = rs_pair<kRowHalfMirror>(C, D, b2);
  E = rs_single<kRowHalfMirror>(E);
  const float H = rs_pair<kQuadXor2>(F, G, b1);
  E = rs_single<kQuadXor2>(E);
  const float K = rs_pair<kQuadXor1>(H, E, b0);
  // Cross-row sums for lanes 0..15 only: permlane32_swap hands lanes 0..31 of its second operand
  // the upper half of its first (which keeps its own lower half), permlane16_swap likewise hands
  // row 0 the contents of row 1.
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(K), 0u, false, false);
  const float K2 = __uint_as_float(h[0]) + __uint_as_float(h[1]);
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(K2), 0u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ int rs_index(int lane) {
  return (lane & 1) ? 8 : ((lane >> 1) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 3) & 1);
}

// a + b over the wave's halves: lanes 0..31 get a[l] + a[l + 32], lanes 32..63 b[l - 32] + b[l].
__device__ __forceinline__ float add_halves(float a, float b) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}
// The same over 16-lane row pairs: rows 0 and 2 get a's rows (0 + 1) and (2 + 3), rows 1 and 3 b's.
__device__ __forceinline__ float add_row_pairs(float a, float b) {
  const auto h = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// Wave sums of the nine gradient terms {dx s0, s1, dx^2 s0, dx s1, s2, s0, wr, wg, wb} when lanes
// l, l + 16, l + 32, l + 48 share a pixel column (so dx): the six per-lane sums are first added
// over those lanes (row k of 16 lanes then holds s0, s1, wr, wg column sums in P and s2, s2, wb, wb
// in Q), scaled by dx, dx^2, and the four values P, P dx, P dx^2, Q reduced inside each row.  The
// sums land in the lanes that col_index names.
__device__ __forceinline__ float reduce_cols9(float s0, float s1, float s2, float wr, float wg, float wb, float dx,
                                              float dx2, int lane) {
  const float P = add_row_pairs(add_halves(s0, wr), add_halves(s1, wg));
  const float Z = add_halves(s2, wb);
  const float Q = add_row_pairs(Z, Z);
  const bool b3 = lane & 8, b2 = lane & 4;
  const float V1 = rs_pair<kRowMirror>(P, P * dx, b3);       // lanes 0..7: P, 8..15: P dx
  const float V2 = rs_pair<kRowMirror>(P * dx2, Q, b3);      // lanes 0..7: P dx^2, 8..15: Q
  const float W = rs_pair<kRowHalfMirror>(V1, V2, b2);       // quads: P, P dx^2, P dx, Q
  return rs_single<kQuadXor1>(rs_single<kQuadXor2>(W));
}

// Gradient column (0..8) whose sum reduce_cols9 leaves in the lane, or -1.
__device__ __forceinline__ int col_index(int lane) {
  switch (lane) {
    case 0: return 5;    // s0
    case 4: return 2;    // dx^2 s0
    case 8: return 0;    // dx s0
    case 12: return 4;   // s2
    case 16: return 1;   // s1
    case 24: return 3;   // dx s1
    case 32: return 6;   // wr
    case 44: return 8;   // wb
    case 48: return 7;   // wg
    default: return -1;
  }
}

// Measurement aid: adds the wave's evaluated / contributing (pixel, Gaussian) counts to stats[0..1].
__device__ __forceinline__ void add_stats(unsigned long long* stats, uint32_t n_eval, uint32_t n_used) {
  unsigned long long e = n_eval, u = n_used;
  for (int d = 32; d >= 1; d >>= 1) {
    e += __shfl_xor(e, d, 64);
    u += __shfl_xor(u, d, 64);
  }
  if (lane_id() == 0) {
    atomicAdd(&stats[0], e);
    atomicAdd(&stats[1], u);
  }
}

// A pixel that has terminated (or lies outside the image) gets this row coordinate: its exponent
// then overflows to -inf, alpha underflows to 0 and it never contributes again, so the step needs
// no separate liveness test.
constexpr float kDeadRow = 1e30f;
// log2(1/255) - 0.001: below it 2^e2 < 1/255 with a margin far above the exponential's error.
constexpr float kE2Skip = -7.9953534f;
constexpr float kLiveBound = 1e29f;

// Transmittance behind a Gaussian: T - alpha T in one rounding, written out so that every walk takes the
// same one.
__device__ __forceinline__ float attenuate(float T, float alpha) { return fmaf(-T, alpha, T); }
// And back to the T before a Gaussian whose weight is w, never as one multiply-add with w's product.
__device__ __forceinline__ float restore(float T, float w) {
#pragma clang fp contract(off)
  return T + w;
}

template <int PPL>
__device__ __forceinline__ bool any_live(const float (&fy)[PPL]) {
  float m = fy[0];
#pragma unroll
  for (int k = 1; k < PPL; ++k) m = fminf(m, fy[k]);
  return wave_any(m < kLiveBound);
}

// One list step (0-based list position pos) of the forward for the lane's pixels:
// alpha = min(0.99, 2^e2); a pixel takes the Gaussian when alpha >= 1/255, unless the new
// transmittance would fall below 1e-4, in which case the pixel stops without it and records pos as
// the number of list entries its compositing took into account.  Only the lane groups in `reach`
// (uniform, every group with a pixel that passes the alpha test among them) are looked at.  REACH: they are the groups
// that the footprint can reach; else (32x32 tiles mark every group) a group that it does not reach ends before the
// exponential (200,000 faint Gaussians at 512x512: 1567 us without the test, 1431 us).
template <int PPL, bool REACH, bool STATS>
__device__ __forceinline__ void fwd_step(const Rec& r, uint32_t reach, int pos, float fx, float (&fy)[PPL],
                                         float (&T)[PPL], float (&cr)[PPL], float (&cg)[PPL], float (&cb)[PPL],
                                         int (&nvis)[PPL], uint32_t& n_used) {
  const float dx = r.mx - fx;
  const float u = fmaf(r.hA, dx * dx, r.lo);
  const float vb = r.hB * dx;
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    // a group out of the footprint's reach: nothing to evaluate (a scalar bit test)
    if (!((reach >> k) & 1u)) continue;
    const float dy = r.my - fy[k];
    const float e2 = exponent2(r, u, vb, dy);
    if (!REACH && !wave_any(e2 >= kE2Skip)) continue;
    const float alpha = fminf(kAlphaMax, __builtin_amdgcn_exp2f(e2));
    const bool ok = alpha >= kAlphaMin;
    if (ok) {   // (with selects instead of the lanes masked off: 1.62 against 1.56 ms, 27M pairs at 1080p)
      float w = alpha * T[k];
      T[k] = attenuate(T[k], alpha);
      // A live pixel keeps T >= 1e-4, so only one that takes the Gaussian can fall below: it stops
      // without it (rare, so handled in a uniform branch), its transmittance going back to the value
      // before the Gaussian (T + w, within a unit in the last place of it).
      if (wave_any(T[k] < kTMin)) {
        __asm__ volatile("" ::: "memory");   // keeps this a branch: the compiler would select both ways
        const bool stop = T[k] < kTMin;
        T[k] = stop ? restore(T[k], w) : T[k];
        w = stop ? 0.0f : w;
        fy[k] = stop ? kDeadRow : fy[k];
        nvis[k] = stop ? pos : nvis[k];
      }
      if (STATS) n_used += w > 0.0f ? 1u : 0u;
      cr[k] = fmaf(r.r, w, cr[k]);
      cg[k] = fmaf(r.g, w, cg[k]);
      cb[k] = fmaf(r.b, w, cb[k]);
    }
  }
}

// Records of an LDS batch (the optional staged list walk): B consecutive list entries, one per
// lane, loaded with per-lane vector loads and written to LDS, then read back at a uniform address
// by every list step of the batch.
template <int B>
struct LdsBatch {
  float4 a[2][B], b[2][B];
  float4 c[2][B];   // c.x: blue, c.y: the pair value's bits (a 16-byte slot, so that one address
                    // serves all the reads of an entry)
};

template <int B>
__device__ __forceinline__ void lds_put(LdsBatch<B>& L, int buf, int lane, const float4& ra, const float4& rb,
                                        float bl, uint32_t pv) {
  if (lane < B) {
    L.a[buf][lane] = ra;
    L.b[buf][lane] = rb;
    L.c[buf][lane].x = bl;
    L.c[buf][lane].y = __uint_as_float(pv);
  }
}

// The pair value of entry b, in a scalar register.
template <int B>
__device__ __forceinline__ uint32_t lds_pv(const LdsBatch<B>& L, int buf, int b) {
  return uniform(__float_as_uint(L.c[buf][b].y));
}

template <int B>
__device__ __forceinline__ Rec lds_get(const LdsBatch<B>& L, int buf, int b) {
  const float4 a = L.a[buf][b], c = L.b[buf][b];
  Rec r;
  r.mx = a.x;
  r.my = a.y;
  r.hA = a.z;
  r.hB = a.w;
  r.hC = c.x;
  r.lo = c.y;
  r.r = c.z;
  r.g = c.w;
  r.b = L.c[buf][b].x;
  return r;
}

// Lane t's entry of the batch at list positions pos(t) (per-lane vector loads): its pair value and
// record (the record of a clamped item when the position lies outside [lo, hi], never read).
__device__ __forceinline__ void lds_fetch(const uint32_t* __restrict__ values, const float4* __restrict__ crec,
                                          const float* __restrict__ cblue, uint32_t imax, int pos, bool ok,
                                          uint32_t& pv, float4& ra, float4& rb, float& bl) {
  pv = ok ? values[pos] : 0u;
  const uint32_t it = min(pv & kItemMask, imax);
  ra = crec[2 * it];
  rb = crec[2 * it + 1];
  bl = cblue[it];
}

// A list staged for a wave whose lanes own one pixel each: up to 64 entries, and four of padding.
struct LdsList {
  float4 a[68], b[68];
  float2 c[68];   // blue, the list position's bits
};

// False only when alpha < 1/255 at every pixel centre of a 16x4 band, [x0, x0 + 15] x [y0, y0 + 3]: the largest
// e2 over that rectangle, at the mean if that is inside and else on one of the four edges, where e2 is a 1D quadratic
// with a clamped maximum.  The bound is raised by well over the rounding of this evaluation and of exponent2.
__device__ __forceinline__ bool band_reached(const float4& a, const float4& b, float x0, float y0) {
  const float hA = a.z, hB = a.w, hC = b.x, lo = b.y;
  const float dx0 = x0 - a.x, dx1 = dx0 + 15.0f, dy0 = y0 - a.y, dy1 = dy0 + 3.0f;
  auto e2 = [&](float dx, float dy) { return fmaf(fmaf(hC, dy, hB * dx), dy, fmaf(hA, dx * dx, lo)); };
  const float sx = -0.5f * hB * __builtin_amdgcn_rcpf(hA), sy = -0.5f * hB * __builtin_amdgcn_rcpf(hC);
  const float m = fmaxf(fmaxf(e2(dx0, __builtin_amdgcn_fmed3f(sy * dx0, dy0, dy1)),
                              e2(dx1, __builtin_amdgcn_fmed3f(sy * dx1, dy0, dy1))),
                        fmaxf(e2(__builtin_amdgcn_fmed3f(sx * dy0, dx0, dx1), dy0),
                              e2(__builtin_amdgcn_fmed3f(sx * dy1, dx0, dx1), dy1)));
  const float ax = fmaxf(fabsf(dx0), fabsf(dx1)), ay = fmaxf(fabsf(dy0), fabsf(dy1));
  const float terms = fmaf(fabsf(hA) * ax, ax, fmaf(fabsf(hB) * ax, ay, fabsf(hC) * ay * ay));
  const bool inside = dx0 <= 0.0f && dx1 >= 0.0f && dy0 <= 0.0f && dy1 >= 0.0f;
  return inside || !(m + fmaf(4e-6f, terms, 0.01f) < kE2Skip);
}

// The list walk of a wave with one pixel per lane (8x8 tiles, or one band of a 16x16 tile that four waves share):
// the list goes through LDS in batches of 64 entries, with bands only those that can reach the band
// (the pair value's mark of the band's rows, then band_reached, a lane per entry), closed up;
// four entries are evaluated at a time, independently of each other up to the
// transmittance, and the stop test is made once for the four (they are taken again one by one when a
// pixel stops).  The arithmetic per entry is fwd_step's.  The next batch's records are requested while this one is
// walked and its pair values one batch earlier, so that a lone wave waits for neither.
template <bool STATS, bool kBand>
__device__ __forceinline__ void fwd_walk_pixels(LdsList& L, const uint32_t* __restrict__ pair_item, int start, int end,
                                                uint32_t group, float band_x0, float band_y0,
                                                const float4* __restrict__ crec, const float* __restrict__ cblue,
                                                uint32_t* __restrict__ planes, int lane, float fx, float& fy,
                                                float& T, float& cr, float& cg, float& cb, int& nvis,
                                                uint32_t& n_used) {
  float4 ra, rb;
  float bl = 0.0f;
  auto fetch = [&](uint32_t pv, bool ok) {
    if (ok) {
      const uint32_t it = pv & kItemMask;
      ra = crec[2 * it];
      rb = crec[2 * it + 1];
      bl = cblue[it];
    }
  };
  uint32_t pv = start + lane < end ? pair_item[start + lane] : 0u;
  uint32_t pv_next = start + 64 + lane < end ? pair_item[start + 64 + lane] : 0u;
  fetch(pv, (pv & group) != 0u);
  for (int base = start; base < end; base += 64) {
    bool ok = (pv & group) != 0u;   // (0 past the end of the list)
    if (kBand) ok = ok && band_reached(ra, rb, band_x0, band_y0);
    const uint64_t m = __ballot(ok);
    const int n = __popcll(m);
    if (kBand && lane < 2) planes[(base - start) / 64 * 8 + lane] = static_cast<uint32_t>(m >> (32 * lane));
    if (ok) {
      const int at = static_cast<int>(popc_below(m));
      L.a[at] = ra;
      L.b[at] = rb;
      L.c[at] = make_float2(bl, __int_as_float(base - start + lane));
    }
    if (lane < 4) {   // padding entries: alpha 0
      L.a[n + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      L.b[n + lane] = make_float4(0.0f, -__builtin_inff(), 0.0f, 0.0f);
      L.c[n + lane] = make_float2(0.0f, 0.0f);
    }
    pv = pv_next;
    fetch(pv, (pv & group) != 0u);
    pv_next = base + 128 + lane < end ? pair_item[base + 128 + lane] : 0u;
    for (int i = 0; i < n; i += 4) {
      float alpha[4], w[4], red[4], green[4], blue[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 ra4 = L.a[i + k], rb4 = L.b[i + k];
        const Rec r{ra4.x, ra4.y, ra4.z, ra4.w, rb4.x, rb4.y, rb4.z, rb4.w, L.c[i + k].x};
        red[k] = r.r;
        green[k] = r.g;
        blue[k] = r.b;
        const float dx = r.mx - fx;
        const float e2 = exponent2(r, fmaf(r.hA, dx * dx, r.lo), r.hB * dx, r.my - fy);
        const float al = fminf(kAlphaMax, __builtin_amdgcn_exp2f(e2));
        alpha[k] = al >= kAlphaMin ? al : 0.0f;
      }
      const float T0 = T;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        w[k] = alpha[k] * T;
        T = attenuate(T, alpha[k]);
      }
      if (wave_any(T < kTMin)) {
        __asm__ volatile("" ::: "memory");   // keeps this a branch
        // the pixels that stop here, again one entry after the other (one that has stopped before may have a T one unit
        // in the last place below the threshold)
        if (T < kTMin && fy < kLiveBound) {
          T = T0;
          bool go = true;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float a = go ? alpha[k] : 0.0f;
            w[k] = a * T;
            T = attenuate(T, a);
            const bool stop = go && T < kTMin;
            T = stop ? restore(T, w[k]) : T;
            w[k] = stop ? 0.0f : w[k];
            nvis = stop ? __float_as_int(L.c[i + k].y) : nvis;
            go = go && !stop;
          }
          fy = kDeadRow;
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (STATS) n_used += w[k] > 0.0f ? 1u : 0u;
        cr = fmaf(red[k], w[k], cr);
        cg = fmaf(green[k], w[k], cg);
        cb = fmaf(blue[k], w[k], cb);
      }
    }
    if (!wave_any(fy < kLiveBound)) {
      if (kBand)   // the entries that no pixel of the band lived to see
        for (int q = (base - start) / 64 + 1 + (lane >> 1); start + 64 * q < end; q += 32)
          planes[8 * q + (lane & 1)] = 0u;
      break;
    }
  }
}

// Marks of a split tile, whose bands are walked by different waves: bit l of the 64-bit plane of band k and batch q
// tells whether entry 64 q + l of the list can reach band k.  The planes lie in the idle tile-key buffer at
// the list's own places, eight words per batch (a split list has 16 entries or more, so they fit).
__device__ __forceinline__ uint32_t* mark_plane(uint32_t* planes, int start, int band) {
  return planes + start + 2 * band;
}

// Work of one compositing wave: a tile, and with 16x16 tiles either all of it or one of its four bands
// (band >= 0).  The first n_split tiles of the launch order, which have the longest lists, are taken by four waves
// each, so that the longest list is no longer what the launch waits for (split_key in
// scan_sort.hip says which).  tile < 0: nothing to do.
struct WaveWork {
  int tile, band;
};
template <int TILE>
__device__ __forceinline__ WaveWork wave_work(const uint32_t* __restrict__ tile_order, int n_tiles,
                                              const uint32_t* __restrict__ n_split) {
  const int b = static_cast<int>(blockIdx.x);
  if (TILE != 16) return {static_cast<int>(tile_order[b]), -1};
  const int ns = static_cast<int>(*n_split);
  if (b < 4 * ns) return {static_cast<int>(tile_order[b >> 2]), b & 3};
  if (b - 3 * ns >= n_tiles) return {-1, -1};
  return {static_cast<int>(tile_order[b - 3 * ns]), -1};
}

// Entries per LDS batch of the forward's walk with four pixels per lane: with 64 the walk took 0.99
// against 0.90 ms (16M pairs, 1080p), and through the scalar cache 1.13 ms.  A test of each band by the wave (an
// exponent and a ballot per step and band) instead of the staging lane's took 1.72 against 1.63 ms (27M pairs);
// marks that tell whether a pixel passed the alpha test, collected in scalar registers, 1.82 ms for 2% of the backward.
constexpr int kFwdBatch = 32;

template <int TILE, bool STATS>
__global__ __launch_bounds__(TileCfg<TILE>::kThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_composite_fwd(
    const DevView* __restrict__ views, int n_views, int n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ tile_order, const uint32_t* __restrict__ n_split,
    const uint32_t* __restrict__ pair_item, uint32_t* __restrict__ pair_marked, uint32_t* __restrict__ planes,
    const float* __restrict__ coef, const float* __restrict__ blue, int64_t n_items, float* __restrict__ image,
    float* __restrict__ final_T, int32_t* __restrict__ n_contrib, unsigned long long* __restrict__ stats) {
  using C = TileCfg<TILE>;
  constexpr int PPL = C::kPPL;
  // one list buffer per wave; a wave's LDS operations complete in issue order, so no barrier separates its
  // writes from its reads
  union Lists {
    LdsBatch<kFwdBatch> batch;
    LdsList list;
  };
  __shared__ __align__(16) char lds[C::kWaves][sizeof(Lists)];
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int wave = static_cast<int>(threadIdx.x) >> 6;
  const WaveWork work = wave_work<TILE>(tile_order, n_tiles, n_split);
  if (work.tile < 0) return;
  const int tile = work.tile;
  const DevView& v = views[find_view(views, n_views, tile)];
  const int local = tile - v.tile_offset;
  const int tx = local % v.tiles_x, ty = local / v.tiles_x;
  const uint2 rg = ranges[tile];
  // the range is the same for every lane: keep it (and the list walk's counters) in scalar registers
  const int start = static_cast<int>(uniform(rg.x)), end = static_cast<int>(uniform(rg.y));
  const float4* __restrict__ crec = reinterpret_cast<const float4*>(coef);
  uint32_t n_eval = 0, n_used = 0;
  const int64_t HW = static_cast<int64_t>(v.width) * v.height;
  float* img = image + 3 * static_cast<int64_t>(v.pixel_offset);
  auto store = [&](int px, int py, float T, float cr, float cg, float cb, int nvis) {
    const int64_t pix = static_cast<int64_t>(py) * v.width + px;
    img[pix] = cr + T * v.bg[0];
    img[HW + pix] = cg + T * v.bg[1];
    img[2 * HW + pix] = cb + T * v.bg[2];
    final_T[v.pixel_offset + pix] = T;
    n_contrib[v.pixel_offset + pix] = nvis;
  };
  const int q0 = wave * (C::kPix / C::kWaves) + lane;
  const int px = tx * TILE + q0 % TILE;
  const float fx = static_cast<float>(px) + 0.5f;
  if (PPL == 1 || work.band >= 0) {
    const int band = PPL == 1 ? 0 : work.band;
    const int py = ty * TILE + (q0 + 64 * band) / TILE;
    const bool inside = px < v.width && py < v.height;
    float fy = inside ? static_cast<float>(py) + 0.5f : kDeadRow, T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
    int nvis = end - start;
    fwd_walk_pixels<STATS, PPL != 1>(*reinterpret_cast<LdsList*>(lds[wave]), pair_item, start, end,
                                     1u << (kItemBits + band), static_cast<float>(tx * TILE) + 0.5f,
                                     static_cast<float>(ty * TILE + 4 * band) + 0.5f, crec, blue,
                                     mark_plane(planes, start, band), lane, fx, fy, T, cr, cg, cb, nvis, n_used);
    if (STATS) {
      // every list entry up to and with the one that stopped the pixel
      n_eval = !inside ? 0u : static_cast<uint32_t>(nvis + (fy < kLiveBound ? 0 : 1));
      add_stats(stats, n_eval, n_used);
    }
    if (inside) store(px, py, T, cr, cg, cb, nvis);
    return;
  }
  if constexpr (PPL > 1) {
    float fy[PPL], T[PPL], cr[PPL], cg[PPL], cb[PPL];
    int nvis[PPL], py[PPL];
    bool inside[PPL];
#pragma unroll
    for (int k = 0; k < PPL; ++k) {
      py[k] = ty * TILE + (q0 + k * 64) / TILE;
      inside[k] = px < v.width && py[k] < v.height;
      fy[k] = inside[k] ? static_cast<float>(py[k]) + 0.5f : kDeadRow;
      T[k] = 1.0f;
      cr[k] = cg[k] = cb[k] = 0.0f;
      nvis[k] = end - start;
    }
    // Double-buffered batches: the next batch's entries are loaded into registers (one per lane)
    // while the current one is walked, then written to the other LDS buffer.  With 16x16 tiles two lanes fetch an
    // entry and test two of its four bands each (32 tests of some 35 operations serve a batch, where a test by the wave
    // costs every step an exponent and a ballot per band), and the pair value goes to pair_marked with
    // the bands they found in bits kItemBits..: the backward visits only those.  One lane with four tests per
    // entry: 1.56 against 1.52 ms (27M pairs at 1080p).
    constexpr bool kMark = TILE == 16;
    const uint32_t imax = n_items > 0 ? static_cast<uint32_t>(n_items - 1) : 0u;
    LdsBatch<kFwdBatch>& L = *reinterpret_cast<LdsBatch<kFwdBatch>*>(lds[wave]);
    uint32_t pv;
    float4 ra, rb;
    float bl;
    const int entry = kMark ? lane & (kFwdBatch - 1) : lane;
    const int band0 = 2 * (lane / kFwdBatch);
    auto stage = [&](int buf, int base) {
      if (kMark) {
        uint32_t reach = 0;
#pragma unroll
        for (int k = 0; k < 2; ++k)
          reach |= (band_reached(ra, rb, static_cast<float>(tx * TILE) + 0.5f,
                                 static_cast<float>(ty * TILE + 4 * (band0 + k)) + 0.5f) ? 1u : 0u) << k;
        reach <<= kItemBits + band0;
        const auto halves = __builtin_amdgcn_permlane32_swap(reach, reach, false, false);
        pv &= kItemMask | halves[0] | halves[1];
        if (lane < kFwdBatch && base + lane < end) pair_marked[base + lane] = pv;
      }
      lds_put<kFwdBatch>(L, buf, lane, ra, rb, bl, pv);
    };
    lds_fetch(pair_item, crec, blue, imax, start + entry, entry < kFwdBatch && start + entry < end, pv, ra, rb, bl);
    stage(0, start);
    int buf = 0;
    for (int base = start; base < end; base += kFwdBatch) {
      if (!any_live(fy)) break;
      const int nb = base + kFwdBatch;
      lds_fetch(pair_item, crec, blue, imax, nb + entry, entry < kFwdBatch && nb + entry < end, pv, ra, rb, bl);
      // batch length and first list position, kept scalar so that the step loop runs on the SALU
      const int n = static_cast<int>(uniform(static_cast<uint32_t>(min(kFwdBatch, end - base))));
      const int pos0 = static_cast<int>(uniform(static_cast<uint32_t>(base - start)));
      for (int b = 0; b < n; ++b) {
        const Rec r = lds_get<kFwdBatch>(L, buf, b);
        const uint32_t reach = lds_pv<kFwdBatch>(L, buf, b) >> kItemBits;
        fwd_step<PPL, kMark, STATS>(r, reach, pos0 + b, fx, fy, T, cr, cg, cb, nvis, n_used);
      }
      buf ^= 1;
      stage(buf, nb);
    }
    if (STATS)   // every list entry up to and with the one that stopped the pixel
#pragma unroll
      for (int k = 0; k < PPL; ++k)
        n_eval += !inside[k] ? 0u : static_cast<uint32_t>(nvis[k] + (fy[k] < kLiveBound ? 0 : 1));
    if (STATS) add_stats(stats, n_eval, n_used);
#pragma unroll
    for (int k = 0; k < PPL; ++k)
      if (inside[k]) store(px, py[k], T[k], cr[k], cg[k], cb[k], nvis[k]);
  }
}

// Per-wave gradient state of one list step of the backward (see bwd_step).
template <int PPL>
struct BwdPix {
  float fy[PPL], T[PPL], dr[PPL], dg[PPL], db[PPL], S[PPL];
  int nc[PPL];
};

// One list step (list position j, 0-based) of the backward for the lane's pixels.  A pixel takes
// part when j < n_contrib and the forward's alpha test holds; its transmittance before the
// Gaussian is T / (1 - alpha), dL/dalpha = T_before * sum_c dL/dC_c (c_c - acc_c) with acc the
// normalised colour behind the Gaussian (the background at first), which then becomes
// alpha c + (1 - alpha) acc.  Only the projection S = sum_c dL/dC_c acc_c enters, so that scalar is
// what the pixel carries: dL/dalpha = T_before (D_c - S) with D_c = sum_c dL/dC_c c_c, and S moves
// to S + alpha (D_c - S).  dL/dpower = alpha dL/dalpha unless alpha was clamped.
// Leaves the lane's sums over its pixels: s0 = sum dp, s1 = sum dp dy, s2 = sum dp dy^2 (dp = dL/dpower), and the
// colour weights alpha T_before dL/dC.  False (for the whole wave) when no group is marked or, without marks, no pixel
// takes part.
// RARE: a clamped alpha, of which there are few, is handled in uniform branches instead of by a minimum and a select
// for every pixel: fewer instructions, but a lone wave waits for every branch (see kLdsSumShare).
struct BwdSums {
  float s0, s1, s2, wr, wg, wb;
};
// FIRST (one pixel per lane): an entry that no pixel takes ends before its update, not after it.
template <int PPL, bool MARKED, bool FIRST, bool RARE, bool STATS>
__device__ __forceinline__ bool bwd_step(const Rec& r, uint32_t groups, int j, float dx, float dx2, BwdPix<PPL>& P,
                                         BwdSums& sums, uint32_t& n_eval, uint32_t& n_used) {
  if (STATS)
#pragma unroll
    for (int k = 0; k < PPL; ++k) n_eval += j < P.nc[k] ? 1u : 0u;
  // MARKED: groups holds the lane groups that the forward left marked, a superset of those
  // with a contributing pixel; each is handled wholly inside its own uniform branch.
  if (!MARKED) groups = (1u << PPL) - 1u;
  if (groups == 0) return false;
  const float u = fmaf(r.hA, dx2, r.lo);
  const float vb = r.hB * dx;
  float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, wr = 0.0f, wg = 0.0f, wb = 0.0f;
  bool anyc = false;
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    if (!((groups >> k) & 1u)) continue;
    const float dy = r.my - P.fy[k];
    const float G2 = __builtin_amdgcn_exp2f(exponent2(r, u, vb, dy));
    float alpha = RARE ? G2 : fminf(kAlphaMax, G2);
    const bool c = j < P.nc[k] && !(alpha < kAlphaMin);
    if (STATS) n_used += c ? 1u : 0u;
    if (FIRST && !wave_any(c)) return false;
    anyc |= c;
    if (c) {
      const bool clamped = RARE && wave_any(!(G2 <= kAlphaMax));
      if (clamped) {
        __asm__ volatile("");   // keeps this a branch
        alpha = fminf(kAlphaMax, G2);
      }
      const float Tk = P.T[k] * __builtin_amdgcn_rcpf(1.0f - alpha);
      P.T[k] = Tk;
      const float D = fmaf(P.dr[k], r.r, fmaf(P.dg[k], r.g, P.db[k] * r.b)) - P.S[k];
      P.S[k] = fmaf(alpha, D, P.S[k]);
      const float w = alpha * Tk;
      wr = fmaf(w, P.dr[k], wr);
      wg = fmaf(w, P.dg[k], wg);
      wb = fmaf(w, P.db[k], wb);
      float dp = w * D;     // alpha dL/dalpha, unless alpha was clamped
      if (!RARE || clamped) {
        if (RARE) __asm__ volatile("");
        dp = G2 <= kAlphaMax ? dp : 0.0f;
      }
      const float t = dp * dy;
      s0 += dp;
      s1 += t;
      s2 = fmaf(t, dy, s2);
    }
  }
  sums = BwdSums{s0, s1, s2, wr, wg, wb};
  // (with marks the superset is tight enough that the test does not pay for itself)
  return MARKED || FIRST || wave_any(anyc);
}

// The nine wave sums of two list entries at a time, through LDS (tiles at most 16 wide).  Every lane leaves its six
// sums of an entry in six rows of 64; lane 4 (6 e + v) + q then takes the four words 16 r + 4 q .. + 3 of row v of
// entry e, r = 0..3: four pixel columns.  It adds a column's pixels, weighs the columns with 1, dx and dx^2, and the
// quad adds its four lanes' sums, of which lane q issues the q-th.
// Why not in registers: a SIMD issues two vector instructions in four cycles, but only one of the two may be a lane
// swap, a DPP or a select or read a scalar register (measured: 2.2 G wave instructions/s per CU of those, 1.2 of
// swaps, against 4.0 of plain adds and fused multiply-adds), and 16 of the 24 that reduce_cols9 takes are of that kind
// (the swaps twice as slow). Here about 7 of 26 per entry are.  27M pairs at 1080p: 4.03 -> 3.76 ms, with the branches
// of RARE 3.62 ms.
constexpr int kSumRow = 80;                 // words between rows: a quarter wave's 16-byte reads touch every bank once
constexpr int kSumWords = 12 * kSumRow;     // per wave
__device__ __forceinline__ int sum_column(int lane) {   // the gradient column (0..8) that the lane issues, or -1
  const int v = (lane >> 2) % 6, q = lane & 3;
  if (lane >= 48) return -1;
  if (v == 0) return q == 0 ? 5 : q == 1 ? 0 : q == 2 ? 2 : -1;   // s0, dx s0, dx^2 s0
  if (v == 1) return q == 0 ? 1 : q == 1 ? 3 : -1;                // s1, dx s1
  return q != 0 ? -1 : v == 2 ? 4 : v + 3;                        // s2, wr, wg, wb
}

// One entry's sums to slot e (0 or 1).
__device__ __forceinline__ void sums_put(float* __restrict__ red, int e, int lane, const BwdSums& s) {
  float* p = red + e * (6 * kSumRow) + lane;
  p[0] = s.s0;
  p[kSumRow] = s.s1;
  p[2 * kSumRow] = s.s2;
  p[3 * kSumRow] = s.wr;
  p[4 * kSumRow] = s.wg;
  p[5 * kSumRow] = s.wb;
}

// The wave sum of column sum_column(lane) of the lane's entry, 4 lanes of slots 0 and 1 each; mx: the entry's mean x,
// fx0: the lane's first column.
__device__ __forceinline__ float sums_total(const float* __restrict__ red, int lane, float mx, float fx0) {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const float4* p = reinterpret_cast<const float4*>(red + min(lane >> 2, 11) * kSumRow + 4 * (lane & 3));
  const float4 r0 = p[0], r1 = p[4], r2 = p[8], r3 = p[12];
  const float c0 = (r0.x + r1.x) + (r2.x + r3.x), c1 = (r0.y + r1.y) + (r2.y + r3.y);
  const float c2 = (r0.z + r1.z) + (r2.z + r3.z), c3 = (r0.w + r1.w) + (r2.w + r3.w);
  const float d0 = mx - fx0, d1 = mx - (fx0 + 1.0f), d2 = mx - (fx0 + 2.0f), d3 = mx - (fx0 + 3.0f);
  float a = (c0 + c1) + (c2 + c3);
  float b = fmaf(c0, d0, c1 * d1) + fmaf(c2, d2, c3 * d3);
  float c = fmaf(c0, d0 * d0, c1 * (d1 * d1)) + fmaf(c2, d2 * d2, c3 * (d3 * d3));
  a = rs_single<kQuadXor1>(rs_single<kQuadXor2>(a));
  b = rs_single<kQuadXor1>(rs_single<kQuadXor2>(b));
  c = rs_single<kQuadXor1>(rs_single<kQuadXor2>(c));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return (lane & 2) ? c : (lane & 1) ? b : a;
}

// A split tile in the backward: its four bands are walked by the four waves of a block, in batches of 64 list
// entries whose records the block stages once.  Each wave takes the entries marked for its band and leaves their
// nine sums in LDS; the block then adds the bands' sums in a fixed order, so that an item's row gets one addition
// per tile and value, as from one wave (fewer atomics, and no more spread between two runs).
struct BandLists {
  float4 a[64], b[64];
  float2 c[64];              // blue, the item's bits
  float4 sum[64 * 9];        // entry, value: a lane of the vector per band
  int maxn[4];
};

template <bool STATS>
__device__ __forceinline__ void bwd_walk_bands(BandLists& L, const uint32_t* __restrict__ pair_values, int start,
                                               const float4* __restrict__ crec, const float* __restrict__ cblue,
                                               int wave, int lane, float fx, BwdPix<1>& P, int out_k, bool out_lane,
                                               float* __restrict__ grad2d, uint32_t& n_used) {
  const int tid = wave * 64 + lane;
  int maxn = P.nc[0];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) maxn = max(maxn, __shfl_xor(maxn, d, 64));
  if (lane == 0) L.maxn[wave] = maxn;
  for (int i = tid; i < 64 * 9; i += 256) L.sum[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  __syncthreads();
  const int band_n = __builtin_amdgcn_readfirstlane(maxn);
  maxn = __builtin_amdgcn_readfirstlane(max(max(L.maxn[0], L.maxn[1]), max(L.maxn[2], L.maxn[3])));
  // entry e of the batch that ends at position hi is position hi - e; the wave's first 16 lanes fetch a quarter of the
  // batch
  float4 ra, rb;
  float bl = 0.0f;
  uint32_t item = 0;
  auto value = [&](int pos) { return pos >= 0 ? pair_values[start + pos] : 0u; };
  auto fetch = [&](int hi) {
    const int pos = hi - 16 * wave - lane;
    if (lane < 16 && pos >= 0) {
      item = pair_values[start + pos] & kItemMask;
      ra = crec[2 * item];
      rb = crec[2 * item + 1];
      bl = cblue[item];
    }
  };
  fetch(maxn - 1);
  uint32_t pv = value(maxn - 1 - lane);
  for (int hi = maxn - 1; hi >= 0; hi -= 64) {
    if (lane < 16) {
      const int e = 16 * wave + lane;
      L.a[e] = ra;
      L.b[e] = rb;
      L.c[e] = make_float2(bl, __uint_as_float(item));
    }
    // the band's entries, without those behind the last one that any of its pixels took into account
    uint64_t m = __ballot((pv >> (kItemBits + wave)) & 1u && hi - lane < band_n);
    fetch(hi - 64);
    pv = value(hi - 64 - lane);
    __syncthreads();
    while (m) {
      const int e = __builtin_ctzll(m);
      m &= m - 1;
      const float4 a = L.a[e], b = L.b[e];
      const Rec r{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, L.c[e].x};
      uint32_t unused = 0;
      const float dx = r.mx - fx, dx2 = dx * dx;
      BwdSums s;
      if (!bwd_step<1, false, false, false, STATS>(r, 1u, hi - e, dx, dx2, P, s, unused, n_used)) continue;
      const float sum = reduce_cols9(s.s0, s.s1, s.s2, s.wr, s.wg, s.wb, dx, dx2, lane);
      if (out_lane && sum != 0.0f) reinterpret_cast<float*>(&L.sum[9 * e + out_k])[wave] = sum;
    }
    __syncthreads();
    for (int i = tid; i < 64 * 9; i += 256) {
      const float4 v = L.sum[i];
      const float s = (v.x + v.y) + (v.z + v.w);
      if (s != 0.0f) {
        const int e = i / 9;
        unsafeAtomicAdd(&grad2d[16 * static_cast<size_t>(__float_as_uint(L.c[e].y)) + (i - 9 * e)], s);
      }
      L.sum[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    __syncthreads();   // the sums and items are read: the next batch may be staged
  }
}

// Threads of a backward block: with 16x16 tiles four waves, which share a split tile or take a tile each.
template <int TILE>
constexpr int kBwdThreads = TILE == 16 ? 256 : TileCfg<TILE>::kThreads;

// Batches whose pairs are kLdsSumShare longest lists or more keep every SIMD supplied with waves, and the instructions
// that a SIMD can issue set the backward's time: sums through LDS and branches around the rare cases save some.
// With fewer, the time is that of the longest lists, whose waves wait for each LDS round trip and branch.  us with
// sums in registers / this form (pairs over the longest list):
// 710 / 871 (1,800), 736 / 851 (2,400), 888 / 815 (3,700), 1248 / 1115 (4,700), 1559 / 1435 (7,400), 4028 / 3617
// (11,000), 1291 / 1151 (12,500); with 8x8 tiles 96 / 105 (2,200), 249 / 207 (6,000), 2177 / 2035 (50,000).
constexpr uint32_t kLdsSumShare = 3000;
template <int TILE, bool STATS, int LDSB>
constexpr bool kBwdSums = TILE <= 16 && !STATS && LDSB == 0;   // the kernel has both forms

// LDS of a backward block: a split tile's lists, or per wave the staged lists or the sums of two entries.
template <int TILE, bool STATS, int LDSB>
constexpr size_t bwd_wave_bytes() {
  return kBwdSums<TILE, STATS, LDSB> ? sizeof(float) * kSumWords
         : LDSB > 0 ? sizeof(LdsBatch<LDSB == 0 ? 1 : LDSB>) : 16;
}
template <int TILE, bool STATS, int LDSB>
constexpr size_t bwd_lds_bytes() {
  const size_t waves = bwd_wave_bytes<TILE, STATS, LDSB>() * (kBwdThreads<TILE> / 64);
  return TILE == 16 && sizeof(BandLists) > waves ? sizeof(BandLists) : waves;
}

// A tile's list for the backward wave that walks it.
struct BwdTile {
  const uint32_t* __restrict__ values;   // pair values, from the list's first
  const float4* __restrict__ crec;
  const float* __restrict__ blue;
  uint32_t imax;
  int lane;
  float fx;
  float col0;      // the first of the lane's four columns in the sums through LDS
  float* __restrict__ grad2d;
};
template <int TILE, int LDSB, bool SUMS, bool STATS, class F>
__device__ __forceinline__ void bwd_walk_tile(const BwdTile& t, unsigned char* __restrict__ lds, F&& load_pixel,
                                              uint32_t& n_eval, uint32_t& n_used) {
  using C = TileCfg<TILE>;
  constexpr int PPL = C::kPPL;
  constexpr bool kCols = 16 % TILE == 0;   // lanes l, l + 16, l + 32, l + 48 share a pixel column
  static_assert(!SUMS || (kCols && LDSB == 0), "sums through LDS: columns in rows of 16, no staged lists");
  // 16x16 tiles walk the forward's marked copy.  An 8x8 tile has one group, which the projection has found within
  // reach; where its pixels in reach have stopped, the entry ends at the first test of bwd_step (two views of 256x256
  // with opacities of 0.5 and more: 101.7 us with every entry summed, 84.9 us; the same test in shared 16x16 lists:
  // 133 -> 144 us).
  constexpr bool kMarked = TILE == 16;
  const int lane = t.lane;
  BwdPix<PPL> P;
  int maxn = 0;
#pragma unroll
  for (int k = 0; k < PPL; ++k) {
    load_pixel(k, P.fy[k], P.T[k], P.nc[k], P.dr[k], P.dg[k], P.db[k], P.S[k]);
    maxn = max(maxn, P.nc[k]);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) maxn = max(maxn, __shfl_xor(maxn, d, 64));
  maxn = __builtin_amdgcn_readfirstlane(maxn);
  const float fx = t.fx;
  const uint32_t imax = t.imax;
  const uint32_t* __restrict__ values = t.values;
  const float4* __restrict__ crec = t.crec;
  const float* __restrict__ blue = t.blue;
  float* __restrict__ grad2d = t.grad2d;
  const int out_k = kCols ? col_index(lane) : rs_index(lane & 15);
  const bool out_lane = kCols ? out_k >= 0 : lane < 16 && ((lane & 1) == 0 || lane == 1);
  float* red = reinterpret_cast<float*>(lds);   // with SUMS
  const int sum_k = sum_column(lane);
  int slot = 0;   // entries in red
  float mx0 = 0.0f;
  uint32_t item0 = 0;
  auto flush = [&](int n, float mx1, uint32_t item1) __attribute__((always_inline)) {
    const bool second = lane >= 24;
    const float sum = sums_total(red, lane, second ? mx1 : mx0, t.col0);
    if (sum_k >= 0 && lane < 24 * n && sum != 0.0f)
      unsafeAtomicAdd(&grad2d[16 * static_cast<size_t>(second ? item1 : item0) + sum_k], sum);
  };
  auto step = [&](const Rec& r, uint32_t pv, int j) __attribute__((always_inline)) {
    const float dx = r.mx - fx, dx2 = dx * dx;
    BwdSums s;
    if (!bwd_step<PPL, kMarked, TILE == 8, SUMS, STATS>(r, pv >> kItemBits, j, dx, dx2, P, s, n_eval, n_used)) return;
    const uint32_t item = pv & kItemMask;
    if constexpr (SUMS) {
      sums_put(red, slot, lane, s);
      if (slot == 0) {
        mx0 = r.mx;
        item0 = item;
        slot = 1;
        return;
      }
      flush(2, r.mx, item);
      slot = 0;
    } else {
      float sum;
      if constexpr (kCols) {
        sum = reduce_cols9(s.s0, s.s1, s.s2, s.wr, s.wg, s.wb, dx, dx2, lane);
      } else {
        const float g[9] = {dx * s.s0, s.s1, dx2 * s.s0, dx * s.s1, s.s2, s.s0, s.wr, s.wg, s.wb};
        sum = reduce_scatter9(g, lane);
      }
      if (out_lane && sum != 0.0f) unsafeAtomicAdd(&grad2d[16 * static_cast<size_t>(item) + out_k], sum);
    }
  };
  if constexpr (LDSB > 0) {
    static_assert(C::kWaves == 1, "LDS batches are wave-private");
    // LDS batches walked in reverse: the batch ending at list position hi holds
    // positions hi, hi - 1, ... in lanes 0, 1, ...
    LdsBatch<LDSB>& L = *reinterpret_cast<LdsBatch<LDSB>*>(lds);
    uint32_t pv;
    float4 ra, rb;
    float bl;
    int hi = maxn - 1;
    lds_fetch(values, crec, blue, imax, hi - lane, lane < LDSB && hi - lane >= 0, pv, ra, rb, bl);
    lds_put<LDSB>(L, 0, lane, ra, rb, bl, pv);
    int buf = 0;
    for (; hi >= 0; hi -= LDSB) {
      const int nh = hi - LDSB;
      lds_fetch(values, crec, blue, imax, nh - lane, lane < LDSB && nh - lane >= 0, pv, ra, rb, bl);
      const int n = min(LDSB, hi + 1);
      for (int b = 0; b < n; ++b) {
        const Rec r = lds_get<LDSB>(L, buf, b);
        step(r, lds_pv<LDSB>(L, buf, b), hi - b);
      }
      buf ^= 1;
      lds_put<LDSB>(L, buf, lane, ra, rb, bl, pv);
    }
  } else {
  // Records through the scalar cache one step ahead of their use, pair values through the scalar
  // cache one step before the record they address, walking positions maxn - 1 .. 0 (positions
  // below 0 are clamped to 0 and their loads never used).
  const int top = max(maxn - 1, 0);
  uint32_t u0 = values[top];
  Rec R0 = load_rec_s(crec, blue, u0, imax), R1, R2;
  uint32_t u1 = values[max(top - 1, 0)], u2;
  for (int j = maxn - 1; j >= 0; j -= 3) {
    wait_scalar_loads();
    R1 = load_rec_s(crec, blue, u1, imax);
    u2 = values[max(j - 2, 0)];
    step(R0, u0, j);
    if (j == 0) break;
    wait_scalar_loads();
    R2 = load_rec_s(crec, blue, u2, imax);
    u0 = values[max(j - 3, 0)];
    step(R1, u1, j - 1);
    if (j == 1) break;
    wait_scalar_loads();
    R0 = load_rec_s(crec, blue, u0, imax);
    u1 = values[max(j - 4, 0)];
    step(R2, u2, j - 2);
  }
  }
  if (SUMS && slot) flush(1, mx0, item0);
}

template <int TILE, bool STATS, int LDSB>
__global__ __launch_bounds__(kBwdThreads<TILE>) void k_composite_bwd(
    const DevView* __restrict__ views, int n_views, int n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ tile_order, const uint32_t* __restrict__ n_split,
    const uint32_t* __restrict__ n_pairs, const uint32_t* __restrict__ longest,
    const uint32_t* __restrict__ pair_item, const uint32_t* __restrict__ pair_marked, const float* __restrict__ coef,
    const float* __restrict__ blue, const float* __restrict__ final_T, const int32_t* __restrict__ n_contrib,
    const float* __restrict__ dL_dimg, float* __restrict__ grad2d, int64_t n_items,
    unsigned long long* __restrict__ stats) {
  using C = TileCfg<TILE>;
  constexpr int PPL = C::kPPL;
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int block_wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int wave = TILE == 16 ? 0 : block_wave;   // of the tile's
  // 16x16 tiles: the first n_split[1] tiles take a block each, the others a wave each
  const int ns = TILE == 16 ? static_cast<int>(n_split[1]) : 0;
  const int b = static_cast<int>(blockIdx.x);
  const bool split = TILE == 16 && b < ns;
  const int place = TILE != 16 || split ? b : ns + 4 * (b - ns) + block_wave;
  if (place >= n_tiles) return;
  const int tile = static_cast<int>(tile_order[place]);
  const DevView& v = views[find_view(views, n_views, tile)];
  const int local = tile - v.tile_offset;
  const int tx = local % v.tiles_x, ty = local / v.tiles_x;
  const int64_t HW = static_cast<int64_t>(v.width) * v.height;
  const int q0 = wave * (C::kPix / C::kWaves) + lane;
  const int px = tx * TILE + q0 % TILE;
  const float fx = static_cast<float>(px) + 0.5f;
  auto load_pixel = [&](int py, float& fy, float& T, int& nc, float& dr, float& dg, float& db, float& S) {
    fy = static_cast<float>(py) + 0.5f;
    T = 1.0f;
    nc = 0;
    dr = dg = db = 0.0f;
    if (px < v.width && py < v.height) {
      const int64_t pix = static_cast<int64_t>(py) * v.width + px;
      T = final_T[v.pixel_offset + pix];
      nc = n_contrib[v.pixel_offset + pix];
      const float* g = dL_dimg + 3 * static_cast<int64_t>(v.pixel_offset);
      dr = g[pix];
      dg = g[HW + pix];
      db = g[2 * HW + pix];
    }
    S = fmaf(dr, v.bg[0], fmaf(dg, v.bg[1], db * v.bg[2]));
  };
  const int start = static_cast<int>(uniform(ranges[tile].x));
  // Lanes l, l + 16, l + 32, l + 48 share a pixel column when the tile is at most 16 wide.
  constexpr bool kCols = 16 % TILE == 0;
  const float4* __restrict__ crec = reinterpret_cast<const float4*>(coef);
  __shared__ __align__(16) unsigned char lds[bwd_lds_bytes<TILE, STATS, LDSB>()];
  if constexpr (TILE == 16) {
    if (split) {   // uniform for the block
      BandLists& bands = *reinterpret_cast<BandLists*>(lds);
      BwdPix<1> P;
      load_pixel(ty * TILE + (lane + 64 * block_wave) / TILE, P.fy[0], P.T[0], P.nc[0], P.dr[0], P.dg[0], P.db[0],
                 P.S[0]);
      uint32_t n_used = 0;
      const int out_k = col_index(lane);
      bwd_walk_bands<STATS>(bands, pair_marked, start, crec, blue, block_wave, lane, fx, P, out_k, out_k >= 0, grad2d,
                            n_used);
      if (STATS) add_stats(stats, static_cast<uint32_t>(P.nc[0]), n_used);
      return;
    }
  }
  const uint32_t* __restrict__ pair_values = TILE == 16 ? pair_marked : pair_item;
  const uint32_t imax = n_items > 0 ? static_cast<uint32_t>(n_items - 1) : 0u;
  const uint32_t* __restrict__ values = pair_values + start;
  uint32_t n_eval = 0, n_used = 0;
  auto load = [&](int k, float& fy, float& T, int& nc, float& dr, float& dg, float& db, float& S)
                  __attribute__((always_inline)) {
    load_pixel(ty * TILE + (q0 + k * 64) / TILE, fy, T, nc, dr, dg, db, S);
  };
  unsigned char* wave_lds = lds + (TILE == 16 ? block_wave : 0) * bwd_wave_bytes<TILE, STATS, LDSB>();
  const BwdTile tile_data{values, crec, blue, imax, lane, fx,
                          static_cast<float>(tx * TILE + (4 * (lane & 3)) % TILE) + 0.5f, grad2d};
  if constexpr (kBwdSums<TILE, STATS, LDSB>) {
    if (*n_pairs / kLdsSumShare >= *longest) {
      bwd_walk_tile<TILE, LDSB, true, STATS>(tile_data, wave_lds, load, n_eval, n_used);
      return;
    }
  }
  bwd_walk_tile<TILE, LDSB, false, STATS>(tile_data, wave_lds, load, n_eval, n_used);
  if (STATS) add_stats(stats, n_eval, n_used);
}

// Before the backward: clears the gradient rows (the first fill_blocks blocks, 16-byte stores), and writes the
// marked copy of the tiles that the forward has split, a block each, from their mark planes.
__global__ __launch_bounds__(256) void k_prepare_bwd(uint4* __restrict__ grad, int64_t n4, int fill_blocks,
                                                     const uint32_t* __restrict__ n_split,
                                                     const uint32_t* __restrict__ tile_order,
                                                     const uint2* __restrict__ ranges,
                                                     const uint32_t* __restrict__ pair_item,
                                                     const uint32_t* __restrict__ planes,
                                                     uint32_t* __restrict__ pair_marked) {
  const int b = static_cast<int>(blockIdx.x);
  if (b < fill_blocks) {
    for (int64_t i = static_cast<int64_t>(b) * 256 + threadIdx.x; i < n4; i += static_cast<int64_t>(fill_blocks) * 256)
      grad[i] = make_uint4(0u, 0u, 0u, 0u);
    return;
  }
  if (b - fill_blocks >= static_cast<int>(*n_split)) return;
  const uint2 r = ranges[tile_order[b - fill_blocks]];
  for (uint32_t j = threadIdx.x; j < r.y - r.x; j += 256) {
    const uint32_t* q = planes + r.x + 8u * (j >> 6) + ((j >> 5) & 1u);
    uint32_t marks = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) marks |= ((q[2 * k] >> (j & 31u)) & 1u) << k;
    pair_marked[r.x + j] = (pair_item[r.x + j] & kItemMask) | (marks << kItemBits);
  }
}

vbm_status launch_prepare_bwd(int tile, const CompositeArgs& a, float* grad2d, hipStream_t s) {
  const int64_t n4 = 4 * a.n_items;   // 16-float rows
  const int64_t want = ceil_div(n4, 256);
  const int fill_blocks = static_cast<int>(want < 8192 ? want : 8192);
  const int tiles = tile == 16 ? static_cast<int>(a.n_tiles < kMaxSplit ? a.n_tiles : kMaxSplit) : 0;
  if (fill_blocks + tiles == 0) return VBM_OK;
  hipLaunchKernelGGL(k_prepare_bwd, dim3(static_cast<unsigned>(fill_blocks + tiles)), dim3(256), 0, s,
                     reinterpret_cast<uint4*>(grad2d), n4, fill_blocks, a.n_split, a.tile_order, a.ranges,
                     a.pair_item, a.planes, a.pair_marked);
  VBM_LAUNCH_CHECK("prepare_bwd");
  return VBM_OK;
}

template <int TILE>
static unsigned wave_grid(const CompositeArgs& a) {
  // with 16x16 tiles room for three more waves per tile that can be split (those left over do nothing)
  return static_cast<unsigned>(a.n_tiles + (TILE == 16 ? 3 * (a.n_tiles < kMaxSplit ? a.n_tiles : kMaxSplit) : 0));
}

template <int TILE>
static vbm_status launch_fwd_t(const CompositeArgs& a, float* image, float* final_T, int32_t* n_contrib,
                               hipStream_t s) {
  const dim3 grid(wave_grid<TILE>(a)), block(TileCfg<TILE>::kThreads);
  if (a.stats)
    hipLaunchKernelGGL((k_composite_fwd<TILE, true>), grid, block, 0, s, a.views, a.n_views,
                       static_cast<int>(a.n_tiles), a.ranges, a.tile_order, a.n_split, a.pair_item, a.pair_marked,
                       a.planes, a.coef, a.blue, a.n_items, image, final_T, n_contrib, a.stats);
  else
    hipLaunchKernelGGL((k_composite_fwd<TILE, false>), grid, block, 0, s, a.views, a.n_views,
                       static_cast<int>(a.n_tiles), a.ranges, a.tile_order, a.n_split, a.pair_item, a.pair_marked,
                       a.planes, a.coef, a.blue, a.n_items, image, final_T, n_contrib, a.stats);
  VBM_LAUNCH_CHECK("composite_fwd");
  return VBM_OK;
}

template <int TILE, int LDSB>
static vbm_status launch_bwd_t(const CompositeArgs& a, const float* final_T, const int32_t* n_contrib,
                               const float* dL_dimg, float* grad2d, hipStream_t s) {
  // with 16x16 tiles a block per split tile and a wave for each of the others (blocks left over do nothing)
  const int64_t split = a.n_tiles < kMaxSplit ? a.n_tiles : kMaxSplit;
  const dim3 grid(static_cast<unsigned>(TILE == 16 ? split + ceil_div(a.n_tiles, 4) : a.n_tiles));
  const dim3 block(kBwdThreads<TILE>);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, s, a.views, a.n_views, static_cast<int>(a.n_tiles), a.ranges,
                       a.tile_order, a.n_split, a.n_pairs, a.longest, a.pair_item, a.pair_marked, a.coef, a.blue,
                       final_T, n_contrib, dL_dimg, grad2d, a.n_items, a.stats);
  };
  launch(a.stats ? k_composite_bwd<TILE, true, LDSB> : k_composite_bwd<TILE, false, LDSB>);
  VBM_LAUNCH_CHECK("composite_bwd");
  return VBM_OK;
}

vbm_status launch_composite_fwd(int tile, const CompositeArgs& a, float* image, float* final_T, int32_t* n_contrib,
                                hipStream_t s) {
  if (tile == 8) return launch_fwd_t<8>(a, image, final_T, n_contrib, s);
  if (tile == 16) return launch_fwd_t<16>(a, image, final_T, n_contrib, s);
  if (tile == 32) return launch_fwd_t<32>(a, image, final_T, n_contrib, s);
  set_error("unsupported tile size %d", tile);
  return VBM_ERR_UNSUPPORTED;
}

vbm_status launch_composite_bwd(int tile, int lds_batch, const CompositeArgs& a, const float* final_T,
                                const int32_t* n_contrib, const float* dL_dimg, float* grad2d, hipStream_t s) {
#define VBM_BWD(T, B) return launch_bwd_t<T, B>(a, final_T, n_contrib, dL_dimg, grad2d, s)
  if (tile == 8 && lds_batch == 0) VBM_BWD(8, 0);
  if (tile == 8 && lds_batch == 32) VBM_BWD(8, 32);
  if (tile == 8 && lds_batch == 64) VBM_BWD(8, 64);
  if (tile == 16 && lds_batch == 0) VBM_BWD(16, 0);
  if (tile == 16 && lds_batch == 32) VBM_BWD(16, 32);
  if (tile == 16 && lds_batch == 64) VBM_BWD(16, 64);
  if (tile == 32 && lds_batch == 0) VBM_BWD(32, 0);
#undef VBM_BWD
  set_error("unsupported tile size %d with LDS batch %d", tile, lds_batch);
  return VBM_ERR_UNSUPPORTED;
}

}  // namespace vbm
