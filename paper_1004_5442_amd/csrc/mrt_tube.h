// mrt_tube.h -- constants of the tube march shared by its kernel
// (tube_kernel, mrt_kernels.hip) and the host library (mrt_api.hip).
#pragma once

namespace mrt {

// The number of time steps per pass by which the library names the tube
// march (the least it takes; a launch takes up to kTubeMaxSteps).
constexpr int kTubeSteps = 4;
constexpr int kTubeMaxSteps = 24;

// Columns a block of `waves` 64-column waves stores after `steps` steps: its
// lanes less the recomputed overlap of one column per step on either side.
constexpr int tube_width(int waves, int steps) { return 64 * waves - 2 * steps; }

}  // namespace mrt
