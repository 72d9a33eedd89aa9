// Piecewise-linear transfer function in the form the kernels take it (Sec. 3, Transfer Function):
// RGBA by linear interpolation between ascending control points, constant beyond the end points.
#pragma once

#include <hip/hip_runtime.h>

#include <cstring>

#include "common.h"

namespace vbm {

struct DevTF {
  float x[VBM_TF_MAX_POINTS];
  float rgba[VBM_TF_MAX_POINTS][4];
  int n;
};

inline DevTF make_dev_tf(const vbm_tf& tf) {
  DevTF d;
  std::memset(&d, 0, sizeof(d));
  d.n = tf.n_points;
  for (int i = 0; i < tf.n_points; ++i) {
    d.x[i] = tf.x[i];
    for (int c = 0; c < 4; ++c) d.rgba[i][c] = tf.rgba[i][c];
  }
  return d;
}

inline bool tf_valid(const vbm_tf& tf) {
  if (tf.n_points < 2 || tf.n_points > VBM_TF_MAX_POINTS) return false;
  for (int i = 1; i < tf.n_points; ++i)
    if (!(tf.x[i] >= tf.x[i - 1])) return false;
  return true;
}

}  // namespace vbm
