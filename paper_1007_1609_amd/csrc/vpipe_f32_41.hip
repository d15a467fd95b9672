// The pipelined recursion's FP32 kernels for lanes of 4 columns.
#include "vpipe.hpp"

namespace cbdg {

int launch_pipe_f32_41(const PipeArgs &A, hipStream_t st) { return launch_pipe_w<float, 4, 1>(A, st); }

}  // namespace cbdg
