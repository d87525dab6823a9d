// mrt_pipe.h -- constants of the level pipeline shared by its kernel
// (pipe_kernel, mrt_kernels.hip) and the host library (mrt_api.hip).
#pragma once

namespace mrt {

// Time steps per pass (the levels of the pipeline).  With `waves` waves per
// level a block covers 64 * waves columns and stores those less the
// recomputed overlap of one column per level on either side.
constexpr int kPipeSteps = 4;
constexpr int pipe_width(int waves) { return 64 * waves - 2 * kPipeSteps; }

}  // namespace mrt
