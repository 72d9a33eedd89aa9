// Compositing launches (raster.hip), called by the renderer's host side.
#pragma once

#include "common.h"

namespace vbm {

struct CompositeArgs {
  const DevView* views;
  int n_views;
  int64_t n_tiles;
  const uint2* ranges;          // each tile's list
  const uint32_t* tile_order;   // longest lists first
  const uint32_t* n_split;      // device: the first n_split[0] tiles of the order are shared by four waves in the
                                // forward, the first n_split[1] <= n_split[0] in the backward (16x16 tiles)
  const uint32_t* n_pairs;      // device: pairs of the batch
  const uint32_t* longest;      // device: entries of its longest list
  const uint32_t* pair_item;    // sorted pair values
  uint32_t* pair_marked;        // the forward's marked copy
  uint32_t* planes;             // the marks of split tiles, a bit per entry and band (see mark_plane)
  const float* coef;            // compositing records
  const float* blue;
  int64_t n_items;
  unsigned long long* stats;    // measurement counters of the pass, or null
};

vbm_status launch_composite_fwd(int tile, const CompositeArgs& a, float* image, float* final_T, int32_t* n_contrib,
                                hipStream_t s);
// Clears the gradient rows and completes the marked copy for the tiles that the forward has split.
vbm_status launch_prepare_bwd(int tile, const CompositeArgs& a, float* grad2d, hipStream_t s);
vbm_status launch_composite_bwd(int tile, int lds_batch, const CompositeArgs& a, const float* final_T,
                                const int32_t* n_contrib, const float* dL_dimg, float* grad2d, hipStream_t s);

}  // namespace vbm
