// The direct CONV kernel whose operands are fetched by wavefronts of their own
// (conv_tile.hip), and the time model that chooses between its tile shapes and
// k_conv's.
#pragma once

#include <hip/hip_runtime.h>

#include "conv_args.h"

namespace sa {

// Rows of the model: the shapes of k_conv_tile, then k_conv's two.
constexpr int kTileSplit = 0;    // k_conv_tile, 64 x 64: the shape of split-K launches
constexpr int kTileShapes = 7;
constexpr int kConv128x128 = 7;  // k_conv, 128 pixels x 128 filters
constexpr int kConv128x64 = 8;   // k_conv, 128 pixels x 64 filters

// Time in microseconds that the model expects of one launch for every group of
// a (its pixels, groups, columns and input; split over ksplit chunks of
// columns) with shape `row` on cus CUs.
float tile_time(const ConvArgs &a, int row, int ksplit, int64_t cus);
// The fastest shape by that model.
int tile_pick(const ConvArgs &a);
// Pixels and filters of a tile of shape `row`, its fetching wavefronts (0:
// k_conv) and the slices that its LDS holds.
void tile_shape(int row, int *pixels, int *filters, int *fetchers, int *slices);
// Does every slice of 64 columns lie in one tap?
bool tile_one_tap(const ConvArgs &a);
// Launches every group of a with k_conv_tile shape `row` < kTileShapes (with
// a.ksplit > 1: kTileSplit, binary32 partial sums).
int tile_run(const ConvArgs &a, int row, hipStream_t stream);

}  // namespace sa
