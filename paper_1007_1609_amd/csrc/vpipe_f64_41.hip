// The pipelined recursion's FP64 kernels for lanes of 4 columns.
#include "vpipe.hpp"

namespace cbdg {

int launch_pipe_f64_41(const PipeArgs &A, hipStream_t st) { return launch_pipe_w<double, 4, 1>(A, st); }

}  // namespace cbdg
