// FP32 precision form of the fused step: float perturbations about a background
// state (PolPert) with the Kahan-compensated average update.  Compiled with
// -ffp-contract=on, like the batched kernel (af_batch.hip): only products and sums
// inside one source expression are fused, so both kernels round every node's
// arithmetic identically and a batched grid reproduces its single-grid result bit
// for bit.
#include <hip/hip_runtime.h>

#include "af_batch.h"
#include "af_fused.h"

namespace af {

// 31x10 cells, 512 threads, registers capped for 4 waves per SIMD (two 77 KB workgroups
// share a CU and overlap each other's barriers), point-update targets in rows of 32
// lanes with the run-time family, as in the FP64 kernel.  Measured at 4096^2 against
// the earlier 24x13 tile with tight rows and the family as a template constant
// (2.061 ms): the run-time family alone 1.994 ms, the 31x10 rows with the constant
// family 1.953 ms, both 1.905 ms; all four give identical bits.  Then the phase-2
// family fence (no more scratch traffic from spills) 1.826 ms and the FP64 row layout
// of the staged arrays (bank conflicts cut eightfold) 1.742 ms, identical bits.
// (at 4096^2 now 1.46 ms: the folded increments, the interpolation of u + du and the
// field-by-field order of the points; bound by vector issue, 1.06e9 instructions a launch, 64% of
// the busy cycles at two cycles to an instruction, and by the LDS.)
constexpr int kFTX = 31, kFTY = 10, kFNT = 512, kFMinW = 4, kFRW = 32;

// A grid of at most one such tile per CU (of 256) has no second workgroup to share a CU with:
// 1024 threads then take the tile in half the rounds, with the same wavefronts per SIMD.  us
// per step with 512 and 1024 threads: 192^2 11.9 and 11.4, 224^2 12.2 and 11.9, 256^2 12.6 and 12.2;
// at 288^2 (290 tiles) 18.3 and 20.9.
constexpr int kFNTWide = 1024;

PolPert<float> pert_pol_f32(const double bg[4], double g) {
    const double r0 = bg[0], u0 = bg[1], v0 = bg[2], p0 = bg[3];
    const double E0 = p0 / (g - 1.0) + 0.5 * r0 * (u0 * u0 + v0 * v0);
    PolPert<float> pol;
    pol.gamma = (float)g;
    pol.gm1inv = (float)(1.0 / (g - 1.0));
    pol.r0 = (float)r0; pol.u0 = (float)u0; pol.v0 = (float)v0; pol.p0 = (float)p0;
    pol.m0x = (float)(r0 * u0); pol.m0y = (float)(r0 * v0); pol.H0 = (float)(E0 + p0);
    return pol;
}

hipError_t launch_step_fused_f32(const StepArgs& a) {
    if (small_grid(true, a.nx, a.ny)) return launch_step_fused_f32_small(a);
    const PolPert<float> pol = pert_pol_f32(a.bg, a.gamma);
    if (one_tile_per_cu_f32(a.nx, a.ny))
        return launch_fused<float, PolPert<float>, kFTX, kFTY, kFNTWide, true, kFMinW, kFRW, true>(a, pol);
    return launch_fused<float, PolPert<float>, kFTX, kFTY, kFNT, true, kFMinW, kFRW, true>(a, pol);
}

hipError_t prepare_fused_f32(int nx, int ny) {
    if (small_grid(true, nx, ny)) return prepare_fused_f32_small(nx, ny);
    if (one_tile_per_cu_f32(nx, ny))
        return prepare_fused<float, PolPert<float>, kFTX, kFTY, kFNTWide, true, kFMinW, kFRW, true>();
    return prepare_fused<float, PolPert<float>, kFTX, kFTY, kFNT, true, kFMinW, kFRW, true>();
}

}  // namespace af
