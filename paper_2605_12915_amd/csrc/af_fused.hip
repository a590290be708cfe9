// Fused, LDS-tiled RB-TAI step (one launch per step), FP64 and FP32, gfx950.
//
// One workgroup owns a TX x TY tile of cells and produces their new averages and
// the new point values of the nodes they own (V_ij, Ev_ij, Eh_ij).  Every
// intermediate of Sec. 6.1 stays on chip:
//   phase 0  stage the primitive node values of cells [-2, T+3)^2 in LDS,
//   phase 1  recovered centres W^C of cells [-2, T+2)^2 (eq. center-node),
//   phase 2  acoustic increments of V, Ev, Eh, C at node-cells [-1, T+2)^2 for
//            tau = dt/2 and dt (App. D, eq. compact-monomial-block),
//   phase 3  transported point update (Sec. 6.1 steps 3-4) of the targets of
//            node-cells [0, T] (the extra row/column feeds the tile's far edges),
//            and per target the time-Simpson flux (F(W^0) + 4F(W^1/2) + F(W^1))/6,
//   phase 4  spatial Simpson edge fluxes and the average update (eq. af-average-update).
// Halo sizes follow from the foot guard |displacement| < 1 cell: a foot of a target
// in node-cells [0, T] lies in cells [-1, T], whose nodes are node-cells [-1, T+1].
// Workgroups are numbered so that spatially adjacent tiles share an XCD (and its L2).
// The kernel template (af_fused.h) serves the FP64 path (absolute variables, this
// file) and the FP32 path (perturbations about a background state, PolPert;
// Kahan-compensated average update whose compensation planes persist across steps;
// af_fused_f32.hip).
#include <hip/hip_runtime.h>

#include "af_fused.h"

namespace af {

// 15x10 cells, 512 threads, the packed tile (79 KB of LDS) and at most 128 registers: two
// workgroups share a CU, four waves per SIMD.  With one workgroup per CU (31x10 cells, 512
// threads, 256 registers, two waves per SIMD) the step was bound by latency: the vector
// units were busy 51% of the cycles, the rest went to barriers, LDS and global round
// trips of one workgroup that nothing overlapped.  Two independent workgroups overlap
// each other's phases and four waves hide the LDS latency (vector units 72% busy),
// which outweighs the larger halo (18x13 node-cells for 150 cells, 1.56 per cell, against
// 1.43).  Phase 2 gives each wavefront one pair of node families (234 node-cells x 2
// pairs in 2 x 256 lanes), phase 3 one target to a lane: 16x11 V, 16x10 Ev and 15(+1)x11
// Eh targets are exactly 512.  This file is compiled without merging LDS reads in pairs:
// a ds_read2_b64 takes 8.2 cycles of the LDS, two ds_read_b64 4.7 (measured at 16 waves per
// CU).  2048^2 step on one GPU: 31x10 0.79 ms; 31x10 with 1024 threads 0.76, unpaired reads 0.73;
// 15x9 unpacked at two workgroups per CU 0.72, unpaired reads 0.68; 15x10 packed 0.73, unpaired 0.62.
constexpr int kTX = 15, kTY = 10, kNT = 512, kRW = 16, kMinW = 4;
// Grids whose 8x8 tiles do not outnumber the CUs: one such tile per CU, whose phases are
// single rounds of one wave per SIMD, is the shorter chain (us per step with 15x10
// and 8x8 tiles: 64^2 9.8 and 7.9, 96^2 10.0 and 8.2, 128^2 (256 tiles) 10.4 and 8.6; beyond, at
// 192^2, 14.9 and 16.0).
constexpr int kSX = 8, kSY = 8, kSNT = 256;
// And grids of at most one 4x4 tile per CU spread over four times the CUs, two wavefronts to a
// tile (unpacked: packing buys nothing at 22 KB of LDS).  us per step with 8x8 and 4x4 tiles:
// 32^2 7.8 and 7.0, 64^2 (256 tiles) 7.9 and 7.2; at 72^2 (324 tiles) 8.1 and 9.2.  With two
// lanes to a target, one for each duration, 64^2 took 8.0.
constexpr int kTinyX = 4, kTinyY = 4, kTinyNT = 128;

// Grids whose 15x10 tiles just exceed the 512 that run at once, so that a few tiles make a
// second round, while 31x10 tiles fit the CUs in one (wide_grid): 256 registers, one workgroup
// to a CU.  us per step with 15x10 and 31x10 tiles: 31x1701 20.9 and 16.1, 61x1100 20.6 and 15.6; in two
// rounds of wide tiles the narrow ones are the faster (62x2000 26.5 and 28.4) but for 31 columns,
// which take three of them to a wide one (31x4096 32.5 and 29.0, 31x30000 191 and 160; 31x2570,
// 257 wide tiles, 26.9 and 28.2).
constexpr int kWX = 31, kWY = 10, kWNT = 512, kWRW = 32;

hipError_t launch_step_fused_f64(const StepArgs& a) {
    PolAbs<double> pol{a.gamma, 1.0 / (a.gamma - 1.0)};
    if (wide_grid(a.nx, a.ny))
        return launch_fused<double, PolAbs<double>, kWX, kWY, kWNT, false, 1, kWRW, true, false>(a, pol);
    if (tiny_grid(a.nx, a.ny))
        return launch_fused<double, PolAbs<double>, kTinyX, kTinyY, kTinyNT, false, 1, 0, true, false>(a, pol);
    if (small_grid(false, a.nx, a.ny))
        return launch_fused<double, PolAbs<double>, kSX, kSY, kSNT, false, 1, 0, true, true>(a, pol);
    return launch_fused<double, PolAbs<double>, kTX, kTY, kNT, false, kMinW, kRW, true, true>(a, pol);
}

hipError_t prepare_fused_f64(int nx, int ny) {
    if (wide_grid(nx, ny)) return prepare_fused<double, PolAbs<double>, kWX, kWY, kWNT, false, 1, kWRW, true, false>();
    if (tiny_grid(nx, ny))
        return prepare_fused<double, PolAbs<double>, kTinyX, kTinyY, kTinyNT, false, 1, 0, true, false>();
    if (small_grid(false, nx, ny)) return prepare_fused<double, PolAbs<double>, kSX, kSY, kSNT, false, 1, 0, true, true>();
    return prepare_fused<double, PolAbs<double>, kTX, kTY, kNT, false, kMinW, kRW, true, true>();
}

}  // namespace af
