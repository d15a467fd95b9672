// The general row pipeline's kernels: real, per-bond operators, FP32.
#include "gpipe.hpp"

namespace cbdg {

int launch_gpipe_f32_rg(const GPipeArgs &G, int grid, hipStream_t st)
{
    switch (G.P.W) {
    case 1: return launch_gpipe_w<float, false, true, 1>(G, grid, st);
    case 2: return launch_gpipe_w<float, false, true, 2>(G, grid, st);
    case 3: return launch_gpipe_w<float, false, true, 3>(G, grid, st);
    default: return fail(CBDG_EUNSUPPORTED, "row pipeline: no width for Lx = %d", G.P.Lx);
    }
}

}  // namespace cbdg
