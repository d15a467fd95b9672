// The general row pipeline's kernels: complex, uniform operators, FP64.
#include "gpipe.hpp"

namespace cbdg {

int launch_gpipe_f64_cu(const GPipeArgs &G, int grid, hipStream_t st)
{
    switch (G.P.W) {
    case 1: return launch_gpipe_w<double, true, false, 1>(G, grid, st);
    case 2: return launch_gpipe_w<double, true, false, 2>(G, grid, st);
    default: return fail(CBDG_EUNSUPPORTED, "row pipeline: no width for Lx = %d", G.P.Lx);
    }
}

}  // namespace cbdg
