// The pipelined recursion's FP32 kernels for lanes of 4 columns, two wavefronts per row.
#include "vpipe.hpp"

namespace cbdg {

int launch_pipe_f32_42(const PipeArgs &A, hipStream_t st) { return launch_pipe_w<float, 4, 2>(A, st); }

}  // namespace cbdg
