// The pipelined recursion's FP64 kernels for lanes of 1 column.
#include "vpipe.hpp"

namespace cbdg {

int launch_pipe_f64_11(const PipeArgs &A, hipStream_t st) { return launch_pipe_w<double, 1, 1>(A, st); }

}  // namespace cbdg
