// The pipelined recursion's FP64 kernels for lanes of 4 columns, two wavefronts per row.
#include "vpipe.hpp"

namespace cbdg {

int launch_pipe_f64_42(const PipeArgs &A, hipStream_t st) { return launch_pipe_w<double, 4, 2>(A, st); }

}  // namespace cbdg
