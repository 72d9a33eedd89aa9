// vbm_adam_init / vbm_adam_step (Adam on the raw parameters, Sec. 5 Implementation Details) and vbm_dvr_render
// (ray-marched supervision images, Sec. 4.4).
#include <hip/hip_runtime.h>

#include <cmath>

#include "common.h"
#include "tf.h"

namespace vbm {
namespace {

constexpr int kRows = 14;   // parameters of a Gaussian

struct AdamParams {
  float lr[5];
  float beta1, beta2, eps;
  float bc1, bc2;  // 1 - beta^t when the step count is a host value
};

// Advances the device step counter; k_adam then reads it (keeps a captured graph replayable).
__global__ void k_step_inc(int32_t* step) {
  if (threadIdx.x == 0) step[0] += 1;
}

// One thread per Gaussian; rows 0-2 means, 3-5 log scales, 6-9 quats, 10 logit opacity, 11-13 rgb.
__global__ __launch_bounds__(256) void k_adam(int64_t n, int64_t stride, float* __restrict__ raw,
                                              float* __restrict__ m, float* __restrict__ v, vbm_gaussians_c g,
                                              vbm_gaussians act, AdamParams p, const int32_t* __restrict__ step_dev) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  if (step_dev) {
    const float t = static_cast<float>(step_dev[0]);
    p.bc1 = 1.0f - powf(p.beta1, t);
    p.bc2 = 1.0f - powf(p.beta2, t);
  }
  const int64_t GS = g.stride, AS = act.stride;
  // every load before the first store: a small set's time is that of one round trip instead of one per row
  float x[kRows], gr[kRows], mm[kRows], vv[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int64_t o = r * stride + i;
    x[r] = raw[o];
    gr[r] = r < 3 ? g.means[r * GS + i]
            : r < 6 ? g.scales[(r - 3) * GS + i]
            : r < 10 ? g.quats[(r - 6) * GS + i]
            : r == 10 ? g.opacity[i] : g.rgb[(r - 11) * GS + i];
    mm[r] = m[o];
    vv[r] = v[o];
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const int grp = r < 3 ? 0 : (r < 6 ? 1 : (r < 10 ? 2 : (r == 10 ? 3 : 4)));
    const int64_t o = r * stride + i;
    if (grp == 1) {
      gr[r] = gr[r] * expf(x[r]);
    } else if (grp == 3) {
      const float sg = 1.0f / (1.0f + expf(-x[r]));
      gr[r] = gr[r] * sg * (1.0f - sg);
    }
    mm[r] = p.beta1 * mm[r] + (1.0f - p.beta1) * gr[r];
    vv[r] = p.beta2 * vv[r] + (1.0f - p.beta2) * gr[r] * gr[r];
    m[o] = mm[r];
    v[o] = vv[r];
    const float mhat = mm[r] / p.bc1;
    const float vhat = vv[r] / p.bc2;
    x[r] -= p.lr[grp] * mhat / (sqrtf(vhat) + p.eps);
    raw[o] = x[r];
    if (grp == 0) act.means[r * AS + i] = x[r];
    else if (grp == 1) act.scales[(r - 3) * AS + i] = expf(x[r]);
    else if (grp == 2) act.quats[(r - 6) * AS + i] = x[r];
    else if (grp == 3) act.opacity[i] = 1.0f / (1.0f + expf(-x[r]));
    else act.rgb[(r - 11) * AS + i] = x[r];
  }
}

// One thread per Gaussian: raw rows from the activated ones (log of the scales, logit of the
// opacity, the other rows copied) and zeroed moments.
__global__ __launch_bounds__(256) void k_adam_init(int64_t n, int64_t stride, vbm_gaussians_c act,
                                                   float* __restrict__ raw, float* __restrict__ m,
                                                   float* __restrict__ v) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t AS = act.stride;
#pragma unroll
  for (int r = 0; r < 14; ++r) {
    float x;
    if (r < 3) x = act.means[r * AS + i];
    else if (r < 6) x = logf(act.scales[(r - 3) * AS + i]);
    else if (r < 10) x = act.quats[(r - 6) * AS + i];
    else if (r == 10) {
      const float o = act.opacity[i];
      x = logf(o / (1.0f - o));
    } else x = act.rgb[(r - 11) * AS + i];
    const int64_t o = r * stride + i;
    raw[o] = x;
    m[o] = 0.0f;
    v[o] = 0.0f;
  }
}

// ------------------------------------------------------------------ supervision images
// Transfer function in float64 at a float64 scalar (the control points are float32 values), as a table in LDS:
// entry 0 is the constant up to the first point, entry i the segment between points i - 1 and i, entry n the
// constant from the last point on.
struct DvrSegment {
  double x0, inv_w;        // position in the segment is (f - x0) inv_w; inv_w = 0: the whole entry is base
  double base[4], delta[4];
};

__device__ __forceinline__ void dvr_table(const DevTF& tf, DvrSegment* __restrict__ s, int threads) {
  for (int e = threadIdx.x; e <= tf.n; e += threads) {
    const int a = e == 0 ? 0 : e - 1, b = e == 0 || e == tf.n ? a : e;
    const double x0 = tf.x[a], w = static_cast<double>(tf.x[b]) - x0;
    const bool jump = a != b && !(w > 0.0);   // a segment of no width takes its end
    DvrSegment q;
    q.x0 = x0;
    q.inv_w = w > 0.0 ? 1.0 / w : 0.0;
    for (int k = 0; k < 4; ++k) {
      const double c0 = tf.rgba[a][k], c1 = tf.rgba[b][k];
      q.base[k] = jump ? c1 : c0;
      q.delta[k] = c1 - c0;
    }
    s[e] = q;
  }
}

__device__ __forceinline__ void dvr_transfer(const DevTF& tf, const DvrSegment* __restrict__ s, double f,
                                             double (&c)[4]) {
  const int n = tf.n;
  int e = 1;
  for (int i = 1; i < n - 1; ++i) e += static_cast<double>(tf.x[i]) <= f ? 1 : 0;
  e = f >= static_cast<double>(tf.x[n - 1]) ? n : e;
  e = f > static_cast<double>(tf.x[0]) ? e : 0;
  const DvrSegment& q = s[e];
  // (f may be infinite or not a number in the constant entries, where the maximum is 0; a compare and a select took
  // 51.7 against 44.6 us for 100x80 pixels of 64^3)
  const double t = fmax((f - q.x0) * q.inv_w, 0.0);
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = fma(t, q.delta[k], q.base[k]);
}

// Square root of x in [0, 1]: the hardware's reciprocal square root, one Newton step for both y = sqrt(x) and
// h = 1 / (2 sqrt(x)), and a last correction of y by its exact residual.
__device__ __forceinline__ double unit_sqrt(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  double y = x * r, h = 0.5 * r;
  const double e = fma(-h, y, 0.5);
  y = fma(y, e, y);
  h = fma(h, e, h);
  y = fma(fma(-y, y, x), h, y);
  return x > 0.0 ? y : (x == 0.0 ? 0.0 : __builtin_nan(""));
}

// Pairs of neighbouring voxels, from any 4-byte boundary.
typedef float float2u __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kDvrViews = 8;   // views per launch
struct DvrViews {
  vbm_view view[kDvrViews];
  int64_t first[kDvrViews];    // first value of the view's image
};

// One thread per pixel, 8x8 pixels per wave (whose rays sample neighbouring voxels), blockIdx.y a view.  The
// supervision images are made once per scene, off the
// fine-tuning loop, and every image the renderer is fitted to comes from here; so the ray, the
// sample positions, the trilinear weights, the transfer function and the compositing run in
// float64 (on CDNA the float64 vector rate equals the unpacked float32 rate), and only the volume
// and the control points are float32 values.  Over the thousand-odd samples of a 512^3 ray,
// float32 positions and products would drift by more than 1e-5 of the image.
// Bound by VALU issue: the position along an axis is one multiply-add from the entry point's (in voxels), the
// transfer function has no division, and the next sample's eight voxels (four pair loads) are requested before
// this one is composited.  A 1080p view of a 512^3 volume: 0.86 -> 0.43 ms (with a transfer function whose rays end
// late 1.46 -> 0.77 ms), against a kernel with two f64 divisions and a library square root per sample and 64 pixels of
// one row per wave. kSmall: the volume's byte offsets fit 32 bits.  kHalf: half-voxel steps, whose opacity correction
// is a square root.
template <bool kSmall, bool kHalf>
__global__ __launch_bounds__(256) void k_dvr(const float* __restrict__ vol, int G, DevTF tf, DvrViews views,
                                             double step_vox, float* __restrict__ images) {
  __shared__ DvrSegment s_tf[VBM_TF_MAX_POINTS + 1];
  dvr_table(tf, s_tf, 256);
  __syncthreads();
  const vbm_view& view = views.view[blockIdx.y];
  const int blocks_x = (view.width + 15) >> 4;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int px = (static_cast<int>(blockIdx.x) % blocks_x) * 16 + (wave & 1) * 8 + (lane & 7);
  const int py = (static_cast<int>(blockIdx.x) / blocks_x) * 16 + (wave >> 1) * 8 + (lane >> 3);
  if (px >= view.width || py >= view.height) return;
  double V[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) V[i] = view.viewmat[i];
  // eye = -R^T t, direction = R^T d_cam (normalised)
  const double e[3] = {-(V[0] * V[3] + V[4] * V[7] + V[8] * V[11]), -(V[1] * V[3] + V[5] * V[7] + V[9] * V[11]),
                       -(V[2] * V[3] + V[6] * V[7] + V[10] * V[11])};
  const double u = (static_cast<double>(px) + 0.5 - static_cast<double>(view.cx)) / static_cast<double>(view.fx);
  const double w = (static_cast<double>(py) + 0.5 - static_cast<double>(view.cy)) / static_cast<double>(view.fy);
  double d[3] = {V[0] * u + V[4] * w + V[8], V[1] * u + V[5] * w + V[9], V[2] * u + V[6] * w + V[10]};
  const double nrm = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  double tn = -INFINITY, tf_ = INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    d[a] /= nrm;
    const double inv = 1.0 / d[a];
    const double t1 = (-1.0 - e[a]) * inv, t2 = (1.0 - e[a]) * inv;
    tn = fmax(tn, fmin(t1, t2));
    tf_ = fmin(tf_, fmax(t1, t2));
  }
  tn = fmax(tn, 0.0);
  double T = 1.0, cr = 0.0, cg = 0.0, cb = 0.0;
  if (tf_ > tn) {
    const double half = 0.5 * static_cast<double>(G);   // voxels per unit
    const double h = 2.0 / static_cast<double>(G);
    const int64_t nsteps = static_cast<int64_t>(floor((tf_ - tn) / (step_vox * h))) + 1;
    const int64_t G2 = static_cast<int64_t>(G) * G;
    double q0[3], dq[3];   // voxel coordinates of sample k: q0 + k dq
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      q0[a] = fma(fma(tn, d[a], e[a]) + 1.0, half, -0.5);
      dq[a] = step_vox * d[a];
    }
    const double last = static_cast<double>(G - 1);
    float2u c[4];   // the voxel pairs (z, y) of the sample ahead: (0, 0), (0, 1), (1, 0), (1, 1)
    double f[3];
    auto request = [&](int64_t k) {
      int i0[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double q = fmin(fmax(fma(static_cast<double>(k), dq[a], q0[a]), 0.0), last);
        i0[a] = min(static_cast<int>(q), G - 2);
        f[a] = q - static_cast<double>(i0[a]);
      }
      if (kSmall) {
        const uint32_t at = 4u * (static_cast<uint32_t>(i0[2] * G + i0[1]) * static_cast<uint32_t>(G) +
                                  static_cast<uint32_t>(i0[0]));
        const char* b = reinterpret_cast<const char*>(vol);
        c[0] = *reinterpret_cast<const float2u*>(b + at);
        c[1] = *reinterpret_cast<const float2u*>(b + 4 * static_cast<int64_t>(G) + at);
        c[2] = *reinterpret_cast<const float2u*>(b + 4 * G2 + at);
        c[3] = *reinterpret_cast<const float2u*>(b + 4 * (G2 + G) + at);
      } else {
        const float* b = vol + i0[2] * G2 + static_cast<int64_t>(i0[1]) * G + i0[0];
        c[0] = *reinterpret_cast<const float2u*>(b);
        c[1] = *reinterpret_cast<const float2u*>(b + G);
        c[2] = *reinterpret_cast<const float2u*>(b + G2);
        c[3] = *reinterpret_cast<const float2u*>(b + G2 + G);
      }
    };
    request(0);
    for (int64_t k = 0; k < nsteps && T >= 1e-4; ++k) {
      double lo[4], di[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lo[r] = c[r].x;
        di[r] = static_cast<double>(c[r].y) - lo[r];
      }
      const double fx = f[0], fy = f[1], fz = f[2];
      request(k + 1);   // (past the end: clamped into the volume, and not used)
      const double c00 = fma(fx, di[0], lo[0]), c01 = fma(fx, di[1], lo[1]);
      const double c10 = fma(fx, di[2], lo[2]), c11 = fma(fx, di[3], lo[3]);
      const double c0 = fma(fy, c01 - c00, c00), c1 = fma(fy, c11 - c10, c10);
      double rgba[4];
      dvr_transfer(tf, s_tf, fma(fz, c1 - c0, c0), rgba);
      const double keep = kHalf ? unit_sqrt(1.0 - rgba[3]) : pow(1.0 - rgba[3], step_vox);
      const double a = 1.0 - keep;
      const double wgt = T * a;
      cr = fma(wgt, rgba[0], cr);
      cg = fma(wgt, rgba[1], cg);
      cb = fma(wgt, rgba[2], cb);
      T *= 1.0 - a;
    }
  }
  const int64_t HW = static_cast<int64_t>(view.width) * view.height;
  float* image = images + views.first[blockIdx.y] + static_cast<int64_t>(py) * view.width + px;
  image[0] = static_cast<float>(cr + T * view.bg[0]);
  image[HW] = static_cast<float>(cg + T * view.bg[1]);
  image[2 * HW] = static_cast<float>(cb + T * view.bg[2]);
}

}  // namespace
}  // namespace vbm

using namespace vbm;

extern "C" vbm_status vbm_adam_step(int64_t n, int64_t stride, float* raw, float* m, float* v, vbm_gaussians_c g,
                                    vbm_gaussians act, const vbm_adam_opts* o, int32_t* step_dev, void* stream) {
  if (!raw || !m || !v || !o || !g.means || !g.scales || !g.quats || !g.opacity || !g.rgb || !act.means ||
      !act.scales || !act.quats || !act.opacity || !act.rgb) {
    set_error("vbm_adam_step: null argument");
    return VBM_ERR_INVALID;
  }
  if (n < 0 || stride < n || g.stride < n || act.stride < n || (!step_dev && o->step < 1) ||
      !(o->beta1 >= 0.0f && o->beta1 < 1.0f) || !(o->beta2 >= 0.0f && o->beta2 < 1.0f) || !(o->eps >= 0.0f)) {
    set_error("vbm_adam_step: bad sizes or hyper-parameters");
    return VBM_ERR_INVALID;
  }
  if (n == 0) return VBM_OK;
  AdamParams p;
  for (int k = 0; k < 5; ++k) p.lr[k] = o->lr[k];
  p.beta1 = o->beta1;
  p.beta2 = o->beta2;
  p.eps = o->eps;
  p.bc1 = p.bc2 = 1.0f;
  if (!step_dev) {
    p.bc1 = static_cast<float>(1.0 - std::pow(static_cast<double>(o->beta1), o->step));
    p.bc2 = static_cast<float>(1.0 - std::pow(static_cast<double>(o->beta2), o->step));
  } else {
    hipLaunchKernelGGL(k_step_inc, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), step_dev);
    VBM_LAUNCH_CHECK("adam_step_inc");
  }
  hipLaunchKernelGGL(k_adam, dim3(ceil_div(n, 256)), dim3(256), 0, static_cast<hipStream_t>(stream), n, stride, raw, m,
                     v, g, act, p, static_cast<const int32_t*>(step_dev));
  VBM_LAUNCH_CHECK("adam");
  return VBM_OK;
}

extern "C" vbm_status vbm_adam_init(int64_t n, int64_t stride, vbm_gaussians_c act, float* raw, float* m, float* v,
                                    void* stream) {
  if (!raw || !m || !v || !act.means || !act.scales || !act.quats || !act.opacity || !act.rgb) {
    set_error("vbm_adam_init: null argument");
    return VBM_ERR_INVALID;
  }
  if (n < 0 || stride < n || act.stride < n) {
    set_error("vbm_adam_init: bad sizes (n %lld, stride %lld, parameter stride %lld)", static_cast<long long>(n),
              static_cast<long long>(stride), static_cast<long long>(act.stride));
    return VBM_ERR_INVALID;
  }
  if (n == 0) return VBM_OK;
  hipLaunchKernelGGL(k_adam_init, dim3(ceil_div(n, 256)), dim3(256), 0, static_cast<hipStream_t>(stream), n, stride,
                     act, raw, m, v);
  VBM_LAUNCH_CHECK("adam_init");
  return VBM_OK;
}

extern "C" vbm_status vbm_dvr_render(const float* vol, int32_t G, const vbm_tf* tf, const vbm_view* views,
                                     int32_t n_views, float step_vox, float* image, void* stream) {
  if (!vol || !tf || !views || !image) {
    set_error("vbm_dvr_render: null argument");
    return VBM_ERR_INVALID;
  }
  if (G < 2 || G > 2048 || n_views < 1 || !(step_vox > 0.0f) || !tf_valid(*tf)) {
    set_error("vbm_dvr_render: bad grid, view count, step or transfer function");
    return VBM_ERR_INVALID;
  }
  const DevTF dtf = make_dev_tf(*tf);
  int64_t off = 0;
  for (int v = 0; v < n_views; ++v) {
    if (views[v].width < 1 || views[v].height < 1 || !(views[v].fx > 0.0f) || !(views[v].fy > 0.0f)) {
      set_error("vbm_dvr_render: view %d is invalid", v);
      return VBM_ERR_INVALID;
    }
  }
  for (int v0 = 0; v0 < n_views; v0 += kDvrViews) {
    DvrViews chunk;
    int64_t blocks = 0;
    const int n = n_views - v0 < kDvrViews ? n_views - v0 : kDvrViews;
    for (int v = 0; v < n; ++v) {
      const vbm_view& w = views[v0 + v];
      chunk.view[v] = w;
      chunk.first[v] = off;
      off += 3 * static_cast<int64_t>(w.width) * w.height;
      const int64_t b = ceil_div(w.width, 16) * ceil_div(w.height, 16);
      blocks = b > blocks ? b : blocks;
    }
    const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(n));
    // 32-bit byte offsets reach a 1024^3 volume
    const bool small = G <= 1024, half = step_vox == 0.5f;
    const auto kernel = small ? (half ? k_dvr<true, true> : k_dvr<true, false>)
                              : (half ? k_dvr<false, true> : k_dvr<false, false>);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, static_cast<hipStream_t>(stream), vol, G, dtf, chunk,
                       static_cast<double>(step_vox), image);
    VBM_LAUNCH_CHECK("dvr");
  }
  return VBM_OK;
}
