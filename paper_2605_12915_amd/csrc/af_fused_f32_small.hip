// FP32 step of small grids: 8x8 tiles of 256 threads, the packed tile (21 KB of LDS).  A
// grid whose 31x10 tiles leave most CUs idle is bound by the chain of one tile's phases:
// smaller tiles shorten it (fewer wavefronts per phase) and spread over more CUs.  us per
// step with 31x10 and 8x8 tiles: 64^2 10.8 and 7.2, 128^2 11.2 and 7.7, 192^2 (576 tiles) 11.8 and
// 10.6; at 256^2 (1024 tiles) 12.6 and 13.8.  Compiled without merging LDS reads in pairs
// (64^2: 8.0 merged, 7.2 not; the 31x10 kernel is the faster with merged ones, 256^2 12.6 and
// 13.4).  The arithmetic of a node does not depend on the tile: results are bitwise those
// of the 31x10 kernel.
// Grids of at most one 4x4 tile per CU take that tile, two wavefronts to each: 32^2 8.1 and
// 7.4 us, 64^2 7.9 and 7.5; at 72^2 (324 tiles) 8.3 and 8.0, at 96^2 8.2 and 8.4.
#include <hip/hip_runtime.h>

#include "af_batch.h"
#include "af_fused.h"

namespace af {

hipError_t launch_step_fused_f32_small(const StepArgs& a) {
    const PolPert<float> pol = pert_pol_f32(a.bg, a.gamma);
    if (tiny_grid(a.nx, a.ny)) return launch_fused<float, PolPert<float>, 4, 4, 128, true, 1, 0, true, false>(a, pol);
    return launch_fused<float, PolPert<float>, 8, 8, 256, true, 4, 0, true, true>(a, pol);
}

hipError_t prepare_fused_f32_small(int nx, int ny) {
    if (tiny_grid(nx, ny)) return prepare_fused<float, PolPert<float>, 4, 4, 128, true, 1, 0, true, false>();
    return prepare_fused<float, PolPert<float>, 8, 8, 256, true, 4, 0, true, true>();
}

}  // namespace af
