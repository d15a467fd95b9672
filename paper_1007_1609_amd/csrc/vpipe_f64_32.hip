// The pipelined recursion's FP64 kernels for lanes of 3 columns, two wavefronts per row.
#include "vpipe.hpp"

namespace cbdg {

int launch_pipe_f64_32(const PipeArgs &A, hipStream_t st) { return launch_pipe_w<double, 3, 2>(A, st); }

}  // namespace cbdg
