// mrt_tile.h -- constants of the tile march shared by its kernel
// (tile_kernel, mrt_kernels.hip) and the host library (mrt_api.hip).
#pragma once

namespace mrt {

// The tile march holds `rows` (8, 12 or 16) rows of 64 columns in a block and
// stores those cells less `overlap` on every side.
constexpr int kTileMaxSteps = 6;
constexpr int tile_width(int overlap) { return 64 - 2 * overlap; }
constexpr int tile_height(int rows, int overlap) { return rows - 2 * overlap; }

}  // namespace mrt
