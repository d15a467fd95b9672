// The pipelined recursion's FP32 kernels for lanes of 2 columns.
#include "vpipe.hpp"

namespace cbdg {

int launch_pipe_f32_21(const PipeArgs &A, hipStream_t st) { return launch_pipe_w<float, 2, 1>(A, st); }

}  // namespace cbdg
