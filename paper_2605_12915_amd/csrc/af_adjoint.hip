// Reverse-mode derivative of one FP64 RB-TAI step (transposed Sec. 6.1 dataflow).
//
// cot_n = (d step / d state_n)^T cot_np1 at fixed dt, in three kernels.  The reverse
// of a gather stencil is a scatter: every block accumulates its scattered
// contributions in an LDS window over its cells plus the reach of the stencil (LDS
// FP64 atomics).  The point kernel then adds its window to global memory (one global
// atomic per entry instead of one per contribution); the increments kernel evaluates
// the pairs that reach its block from outside too and stores the block's own cells:
//   k_adj_fwd      forward intermediates recomputed from state_n (recovered centres
//                  W^C, node increments of both durations); zeroes the accumulation
//                  planes.
//   k_adj_points   average update and space-time Simpson fluxes (transposed), then
//                  for every target and duration the transposed point update (TAI:
//                  density closure, Q2 evaluation of W and of the increments at the
//                  foot, values and foot position, the two Picard stages; RB: Q2 of W
//                  at the foot, the target's own increments).  Scatters into cot_n
//                  (point planes), lambda_C and lambda_D.
//   k_adj_incr     transposed node increments (Horner in r, freezing c_K, Z_K, the
//                  folded blocks and the lines shared by a pair of families,
//                  transposed), then the transposed centre recovery (prim(U_c),
//                  inverse Simpson, U(W) at the eight boundary nodes); adds to the point
//                  planes of cot_n and writes its average planes.
// The floor() that locates a foot is piecewise constant: its derivative is zero
// (the usual convention; the step is continuous across faces because R_h and I_h are).
#include <hip/hip_runtime.h>

#include <mutex>

#include "af_adjoint.h"
#include "af_internal.h"

namespace af {

// Scatter target of the point kernel: an LDS window of 40 planes over node-cells
// [ri0, ri0 + R) x [rj0, rj0 + R) (unwrapped indices; the flush wraps them), the planes of a
// row side by side.  Planes: 0..11 point values (family * 4 + (rho, u, v, p)), 12..15 recovered
// centres, 16..39 increments (tau * 12 + family * 3 + (u, v, p)).
template <int R>
struct PointWin {
    static constexpr int kPlane = R, kRX = 40 * R, SIZE = R * kRX;
    double* a;
    int ri0, rj0;
    // offset of node-cell (i, j); addb adds to plane pl at that offset plus a small constant
    // one (so that every add of one cell's nodes shares a base)
    __device__ __forceinline__ int base(int i, int j) const { return (j - rj0) * kRX + (i - ri0); }
    __device__ __forceinline__ void addb(int pl, int b, int off, double v) const { atomicAdd(a + b + (pl * kPlane + off), v); }
};

struct PlaneList { double* p[40]; };

// Cotangent planes read by cell with a periodic wrap of at most one grid length.
struct CotAcc {
    StatePtrs<double> s;
    int nx, ny;
    __device__ __forceinline__ double get(int k, int i, int j) const {
        i = (i < 0) ? i + nx : (i >= nx ? i - nx : i);
        j = (j < 0) ? j + ny : (j >= ny ? j - ny : j);
        return s.p[k][(size_t)j * nx + i];
    }
};

// The forward state of a block, staged in LDS like its scatter window.
template <int R>
struct StageWin {
    static constexpr int kPlane = R, kRX = 40 * R;
    const double* a;
    int ri0, rj0;
    __device__ __forceinline__ int base(int i, int j) const { return (j - rj0) * kRX + (i - ri0); }
    __device__ __forceinline__ double at(int pl, int b, int off) const { return a[b + (pl * kPlane + off)]; }
};

// Add a window to its global planes (periodic wrap), one atomic per nonzero entry: each
// thread takes whole node-cells of the window, wraps its global index once and walks the
// planes (so the plane pointer is the same across the wavefront).
template <int R>
__device__ __forceinline__ void flush_window(const PointWin<R>& w, const PlaneList& G, int nx, int ny) {
    for (int e = threadIdx.x; e < R * R; e += blockDim.x) {
        int i = w.ri0 + e % R, j = w.rj0 + e / R;
        i = (i % nx + nx) % nx;
        j = (j % ny + ny) % ny;
        const size_t k = (size_t)j * nx + i;
        const double* c = w.a + (e / R) * PointWin<R>::kRX + e % R;
#pragma unroll 8
        for (int pl = 0; pl < 40; ++pl) {
            const double v = c[pl * R];
            if (v != 0.0) atomicAdd(G.p[pl] + k, v);
        }
    }
}

// Periodic index.
__device__ __forceinline__ int wrap_any(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

// Forward intermediates of a TX x TY tile, recomputed from state_n for the reverse
// sweep: the tile's primitive node values (node-cells [-1, T+1)) and recovered centres
// (cells [-1, T)) staged in LDS, then the increments of both durations at the tile's
// own node-cells (every wedge of a node-cell in [0, T) lies in cells [-1, T); with `sum`
// u + du and v + dv in place of du and dv, as the point kernel takes them).  Writes
// W^C of the tile's cells and the 24 increment planes, and zeroes the tile's cells of the
// planes the point kernel accumulates into.
template <int TX, int TY>
struct IntTile {
    static constexpr int PX = TX + 2, PY = TY + 2, CX = TX + 1, CY = TY + 1;
    double P[12][PY][PX];
    double C[4][CY][CX];
};

template <int TX, int TY>
struct IntAcc {
    const IntTile<TX, TY>* t;
    __device__ __forceinline__ Prim<double> node(int fam, int x, int y) const {
        if (fam == F_C) return {t->C[0][y + 1][x + 1], t->C[1][y + 1][x + 1], t->C[2][y + 1][x + 1], t->C[3][y + 1][x + 1]};
        const int b = 4 * fam;
        return {t->P[b][y + 1][x + 1], t->P[b + 1][y + 1][x + 1], t->P[b + 2][y + 1][x + 1], t->P[b + 3][y + 1][x + 1]};
    }
};

// XCD-aware workgroup numbering (as in the step kernels): workgroup b runs on XCD
// b mod 8; each XCD takes a contiguous run of the row-major block list, so that the
// overlapping halos and accumulation windows of neighbouring blocks meet in one L2.
__device__ __forceinline__ int xcd_tile(int b, int ntiles) {
    const int xcd = b & 7;
    int base = 0;
    for (int x = 0; x < xcd; ++x) base += (ntiles - x + 7) >> 3;
    return base + (b >> 3);
}

constexpr int kFBX = 32, kFBY = 8, kFNT = kFBX * kFBY;
using FwdTile = IntTile<kFBX, kFBY>;

// two workgroups per CU (256 registers per lane)
__global__ void __launch_bounds__(kFNT, 2) k_adj_fwd(StatePtrs<double> prim, double* C, double* D, PlaneList Z,
                                                     int nzero, bool sum, int nx, int ny, int tiles_x, int ntiles,
                                                     double gamma, double lam0, double lam1, unsigned* status) {
    __shared__ FwdTile L;
    const int tile = xcd_tile(blockIdx.x, ntiles), tid = threadIdx.x;
    const int i0 = (tile % tiles_x) * kFBX, j0 = (tile / tiles_x) * kFBY;
    const size_t N = (size_t)nx * ny;
    const int ox = tid % kFBX, oy = tid / kFBX;
    const bool own = i0 + ox < nx && j0 + oy < ny;
    const size_t g = own ? (size_t)(j0 + oy) * nx + (i0 + ox) : 0;
    unsigned st = 0;
    // stage primitives: all loads of a thread's rounds are issued before its stores
    {
        constexpr int NP = FwdTile::PX * FwdTile::PY, R = (NP + kFNT - 1) / kFNT;
        double v[R][12];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = r * kFNT + tid;
            if (e < NP) {
                const size_t k = (size_t)wrap_any(j0 - 1 + e / FwdTile::PX, ny) * nx + wrap_any(i0 - 1 + e % FwdTile::PX, nx);
#pragma unroll
                for (int q = 0; q < 12; ++q) v[r][q] = prim.p[4 + q][k];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = r * kFNT + tid;
            if (e < NP)
#pragma unroll
                for (int q = 0; q < 12; ++q) L.P[q][e / FwdTile::PX][e % FwdTile::PX] = v[r][q];
        }
    }
    if (own) {
        for (int q = 0; q < nzero; ++q) Z.p[q][g] = 0.0;
    }
    __syncthreads();
    // recovered centres of cells [-1, T)
    {
        const IntAcc<kFBX, kFBY> A{&L};
        for (int e = tid; e < FwdTile::CX * FwdTile::CY; e += kFNT) {
            const int x = e % FwdTile::CX - 1, y = e / FwdTile::CX - 1;
            const size_t k = (size_t)wrap_any(j0 + y, ny) * nx + wrap_any(i0 + x, nx);
            const double Ub[4] = {prim.p[0][k], prim.p[1][k], prim.p[2][k], prim.p[3][k]};
            const Prim<double> w = recover_centre(Ub, A.node(F_V, x, y), A.node(F_V, x + 1, y), A.node(F_V, x, y + 1),
                                                  A.node(F_V, x + 1, y + 1), A.node(F_EH, x, y), A.node(F_EH, x, y + 1),
                                                  A.node(F_EV, x, y), A.node(F_EV, x + 1, y), gamma);
            L.C[0][y + 1][x + 1] = w.r;
            L.C[1][y + 1][x + 1] = w.u;
            L.C[2][y + 1][x + 1] = w.v;
            L.C[3][y + 1][x + 1] = w.p;
            if (x >= 0 && y >= 0 && i0 + x < nx && j0 + y < ny) {
                const size_t c = (size_t)(j0 + y) * nx + (i0 + x);
                C[c] = w.r;
                C[N + c] = w.u;
                C[2 * N + c] = w.v;
                C[3 * N + c] = w.p;
                if (!(w.r > 0.0) || !(w.p > 0.0)) st |= SB_NONPHYS;
            }
        }
    }
    __syncthreads();
    // increments of the tile's own node-cells
    if (own) {
        const IntAcc<kFBX, kFBY> A{&L};
        const PolAbs<double> pol{gamma, 1.0 / (gamma - 1.0)};
        cell_increments(A, ox, oy, pol, lam0, lam1, st, [&](int pl, double v) {
            const int fam = (pl % 12) / 3, q = pl % 3;
            if (q < 2 && sum) v += q == 0 ? A.node(fam, ox, oy).u : A.node(fam, ox, oy).v;
            D[(size_t)pl * N + g] = v;
        });
    }
    if (st) atomicOr(status, st);
}

// Reverse of the point update, fluxes and average update for a BX x BY block of
// cells, one thread per (cell, target family).  Feet stay within one cell (guarded),
// so every read of the forward state and every contribution lies in node-cells
// [-1, B + 2) of the block: the block stages the forward state of that window in LDS
// (each thread loads all 40 planes of one node-cell at once) and accumulates into an
// LDS window of the same shape.
// 8x8 blocks: the staged state and the window take 79 KB, so two blocks share a CU and
// one's staging overlaps the other's work (2% faster than 16x8 at one block per CU,
// despite the larger window overlap, 1.89x against 1.63x).
// The planes of a window row lie side by side: 40 x 11 doubles from row to row, 24 modulo the
// 32 that the banks hold, so that the four rows of 8 lanes that a half-wavefront reads or
// adds to at a common offset start in four distinct quarters of the banks (512^2: 1.9e6 conflict
// cycles for 3.7e6 LDS instructions, 8.2e6 with rows apart by plane; feet of different offsets,
// the staging and the flush make the rest).
// Bound by the LDS additions and by two wavefronts per SIMD hiding little of the FP64 chains:
// both durations' feet in one cell share an addition per node and plane, and the velocities'
// part of the increment planes is left to the increments' kernel (SCHEME 0; 512^2: 104.7 -> 94.0
// us, 1000^2 461 -> 438).  That keeps both durations' weights (FootAdj) through the second
// one's evaluation: 54 registers spilled for SCHEME 0 (60 bytes of scratch a lane; writes to memory
// 0.047 -> 0.058 GB a launch at 512^2) and 28 for SCHEME 1, none and 2 without; the gain above is
// net of it.
template <int BX, int BY>
struct PointBlock {
    static_assert(BX == BY, "square blocks");
    static constexpr int NT = 3 * BX * BY, R = BX + 3, WIN = R * R;
    static constexpr size_t LDS = sizeof(double) * 2 * 40 * WIN;   // staged state + accumulators
    static_assert(WIN <= NT, "one staging round");
    static_assert((BX * BY) % 64 == 0, "each wavefront holds one target family");
};

// (registers bounded for MINB blocks per CU at 2 waves per SIMD: the workgroup alone
// would let the compiler take accumulation registers too, and the RB instantiation did,
// at one wave per SIMD)
template <int SCHEME, int BX, int BY, int MINB>
__global__ void __launch_bounds__(3 * BX * BY, MINB)
    k_adj_points(StatePtrs<double> prim, const double* C, const double* Dfwd, StatePtrs<double> cot1, PlaneList G,
                 int nx, int ny, int tiles_x, int ntiles, double gamma, double lam0, double lam1) {
    using B = PointBlock<BX, BY>;
    extern __shared__ __align__(16) unsigned char smem[];
    double* stage = reinterpret_cast<double*>(smem);   // [R][40][R]
    const int tile = xcd_tile(blockIdx.x, ntiles);
    const int i0 = (tile % tiles_x) * BX, j0 = (tile / tiles_x) * BY;
    const PointWin<B::R> O{stage + 40 * B::WIN, i0 - 1, j0 - 1};
    for (int e = threadIdx.x; e < 40 * B::WIN; e += B::NT) O.a[e] = 0.0;
    if (threadIdx.x < B::WIN) {
        const int e = threadIdx.x;
        const int i = wrap_any(i0 - 1 + e % B::R, nx), j = wrap_any(j0 - 1 + e / B::R, ny);
        const size_t N = (size_t)nx * ny, k = (size_t)j * nx + i;
        double v[40];
#pragma unroll
        for (int pl = 0; pl < 12; ++pl) v[pl] = prim.p[4 + pl][k];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[12 + q] = C[q * N + k];
#pragma unroll
        for (int q = 0; q < 24; ++q) v[16 + q] = Dfwd[q * N + k];
#pragma unroll
        for (int pl = 0; pl < 40; ++pl) stage[(e / B::R) * (40 * B::R) + pl * B::R + e % B::R] = v[pl];
    }
    __syncthreads();
    const StageWin<B::R> S{stage, i0 - 1, j0 - 1};
    const int cell = (int)threadIdx.x % (BX * BY), fam = (int)threadIdx.x / (BX * BY);   // wave-uniform
    const int i = i0 + cell % BX, j = j0 + cell / BX;
    if (i < nx && j < ny) {
        const CotAcc C1{cot1, nx, ny};
        unsigned fix;
        if (fam == F_V) fix = point_adj_target<F_V, SCHEME, 0>(S, C1, O, i, j, gamma, lam0, lam1);
        else if (fam == F_EV) fix = point_adj_target<F_EV, SCHEME, 0>(S, C1, O, i, j, gamma, lam0, lam1);
        else fix = point_adj_target<F_EH, SCHEME, 0>(S, C1, O, i, j, gamma, lam0, lam1);
        // targets whose feet lie in different cells (rare): their shares of those cells
        if (__any(fix != 0u)) {
            if (fam == F_V) point_adj_target<F_V, SCHEME, 1>(S, C1, O, i, j, gamma, lam0, lam1, fix);
            else if (fam == F_EV) point_adj_target<F_EV, SCHEME, 1>(S, C1, O, i, j, gamma, lam0, lam1, fix);
            else point_adj_target<F_EH, SCHEME, 1>(S, C1, O, i, j, gamma, lam0, lam1, fix);
        }
    }
    __syncthreads();
    flush_window(O, G, nx, ny);
}

template <int SCHEME, int BX, int BY, int MINB>
void launch_points(const StepArgs& a, StatePtrs<double> prim, const double* C, const double* Dfwd,
                   StatePtrs<double> cot1, const PlaneList& L, double lam0, double lam1) {
    using B = PointBlock<BX, BY>;
    const int tx = (a.nx + BX - 1) / BX, nt = tx * ((a.ny + BY - 1) / BY);
    hipLaunchKernelGGL((k_adj_points<SCHEME, BX, BY, MINB>), dim3(nt), dim3(B::NT), B::LDS, a.stream, prim, C, Dfwd,
                       cot1, L, a.nx, a.ny, tx, nt, a.gamma, lam0, lam1);
}

template <int BX, int BY, int MINB>
hipError_t prepare_points() {
    using B = PointBlock<BX, BY>;
    hipError_t e = hipFuncSetAttribute((const void*)k_adj_points<0, BX, BY, MINB>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)B::LDS);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void*)k_adj_points<1, BX, BY, MINB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)B::LDS);
}

// Transposed node increments and centre recovery for a 16 x 8 block of node-cells, whose
// share of cot_n the block completes by itself: it takes the pairs of families of the
// node-cells [-1, B + 1), whose stencils reach node-cells [-2, B + 2) and are all that reach
// [0, B), and the centre recovery of cells [-1, B).  The forward nodes of that window are
// staged in LDS, the contributions accumulated in an LDS window of the same shape, and the
// block's own node-cells added to global memory by plain loads and stores.  Rows hold all
// planes side by side ([y][plane][x], an odd multiple of 16 doubles), so that two rows of 16
// items fall on different banks, as the centres' and the last phase's nearly are; the pairs, the
// bulk of the accesses, are walked in rows of 18, whose second row meets the first on the
// banks in every half-wavefront (512^2: 3.5e6 conflict cycles for 1.7e6 LDS instructions).  The
// pairs are evaluated 1.41 times per node-cell; adding each block's overlapping window to
// global memory by atomics instead took 30 k of the block's 52 k cycles (512^2: 68 us against
// 61; 1000^2 272 and 236).
constexpr int kIBX = 16, kIBY = 8, kINT = 256;

struct IncrWin {
    static constexpr int RX = kIBX + 4, RY = kIBY + 4, kPlane = RX + 1, kRX = 16 * kPlane, SIZE = RY * kRX;
    double* a;
    __device__ __forceinline__ int base(int x, int y) const { return (y + 2) * kRX + (x + 2); }
    // planes 0..11 point values, 12..15 centres; the averages' (16..19) take the centres'
    // place once those are consumed
    __device__ __forceinline__ void addb(int pl, int b, int off, double v) const {
        atomicAdd(a + b + ((pl >= 16 ? pl - 4 : pl) * kPlane + off), v);
    }
    __device__ __forceinline__ void node(int fam, int x, int y, const double g[4]) const {
        const int b = base(x, y), pl = fam == F_C ? 12 : 4 * fam;
#pragma unroll
        for (int q = 0; q < 4; ++q) addb(pl + q, b, 0, g[q]);
    }
};

struct IncrNodes {
    const double* a;
    __device__ __forceinline__ Prim<double> node(int fam, int x, int y) const {
        const double* c = a + (y + 2) * IncrWin::kRX + (x + 2) + (fam == F_C ? 12 : 4 * fam) * IncrWin::kPlane;
        return {c[0], c[IncrWin::kPlane], c[2 * IncrWin::kPlane], c[3 * IncrWin::kPlane]};
    }
};

// dst: cot_n (0..11 point values, to which the point kernel has added; 12..15 averages); avg:
// the averages' cotangent of cot_np1 (the averages enter the new averages with unit weight)
constexpr size_t kIncrLds = 2 * IncrWin::SIZE * sizeof(double);

struct IncrOut { double* dst[16]; const double* avg[4]; };

__global__ void __launch_bounds__(kINT, 2) k_adj_incr(StatePtrs<double> prim, const double* C, const double* lD,
                                                      const double* lC, IncrOut G, bool sum, int nx, int ny, int tiles_x,
                                                      int ntiles, double gamma, double lam0, double lam1) {
    extern __shared__ __align__(16) unsigned char smem[];
    double* stage = reinterpret_cast<double*>(smem);
    double* win = stage + IncrWin::SIZE;
    const int tile = xcd_tile(blockIdx.x, ntiles), tid = threadIdx.x;
    const int i0 = (tile % tiles_x) * kIBX, j0 = (tile / tiles_x) * kIBY;
    const size_t N = (size_t)nx * ny;
    const IncrWin O{win};
    const IncrNodes A{stage};
    // items of one round each: staged node-cells [-2, B + 2), pairs [-1, B + 1), centres [-1, B)
    constexpr int PW = kIBX + 2, PH = kIBY + 2, CW = kIBX + 1, CH = kIBY + 1;
    static_assert(IncrWin::RX * IncrWin::RY <= kINT && PW * PH <= kINT && CW * CH <= kINT, "one round each");
    const int px = tid % PW - 1, py = tid / PW - 1, cx = tid % CW - 1, cy = tid / CW - 1;
    const bool pair = tid < PW * PH, centre = tid < CW * CH;
    double l[4][2][3], lW[4];
    if (tid < IncrWin::RX * IncrWin::RY) {
        const int wx = tid % IncrWin::RX, wy = tid / IncrWin::RX;
        const size_t k = (size_t)wrap_any(j0 - 2 + wy, ny) * nx + wrap_any(i0 - 2 + wx, nx);
        double v[16];
#pragma unroll
        for (int pl = 0; pl < 12; ++pl) v[pl] = prim.p[4 + pl][k];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[12 + q] = C[q * N + k];
        if (pair) {
            const double* d = lD + (size_t)wrap_any(j0 + py, ny) * nx + wrap_any(i0 + px, nx);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int f = 0; f < 4; ++f)
#pragma unroll
                    for (int q = 0; q < 3; ++q) l[f][t][q] = d[(size_t)(t * 12 + f * 3 + q) * N];
        }
        if (centre) {
            const double* d = lC + (size_t)wrap_any(j0 + cy, ny) * nx + wrap_any(i0 + cx, nx);
#pragma unroll
            for (int q = 0; q < 4; ++q) lW[q] = d[q * N];
        }
#pragma unroll
        for (int pl = 0; pl < 16; ++pl) stage[wy * IncrWin::kRX + pl * IncrWin::kPlane + wx] = v[pl];
    }
    for (int e = tid; e < IncrWin::SIZE; e += kINT) win[e] = 0.0;
    __syncthreads();
    if (pair) {
        incr_adj<5>(A, O, px, py, l[F_V], l[F_EV], sum, gamma, lam0, lam1);
        incr_adj<3>(A, O, px, py, l[F_EH], l[F_C], sum, gamma, lam0, lam1);
    }
    __syncthreads();
    // each centre entry is read (and cleared: the averages' contributions take its place) by
    // one thread, which scatters into the point planes besides
    if (centre) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double* c = win + O.base(cx, cy) + (12 + k) * IncrWin::kPlane;
            lW[k] += *c;
            *c = 0.0;
        }
        centre_adj(A, O, cx, cy, lW, gamma);
    }
    __syncthreads();
    // the block's own node-cells, half the planes to a thread: planes 8 h .. 8 h + 7
    const int x = tid % kIBX, y = tid / kIBX % kIBY, h = tid / (kIBX * kIBY);   // h: wave-uniform
    if (i0 + x < nx && j0 + y < ny) {
        const size_t g = (size_t)(j0 + y) * nx + (i0 + x);
        const double* w = win + O.base(x, y);
        double v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = h == 0 ? G.dst[q][g] : (q < 4 ? G.dst[8 + q][g] : G.avg[q - 4][g]);
#pragma unroll
        for (int q = 0; q < 8; ++q) (h == 0 ? G.dst[q] : G.dst[8 + q])[g] = v[q] + w[(8 * h + q) * IncrWin::kPlane];
    }
}

hipError_t launch_adjoint_f64(const StepArgs& a, const void* const cot1_[16], void* const cot0_[16]) {
    const size_t N = (size_t)a.nx * a.ny;
    double* C = (double*)a.scratch;
    double* Dfwd = C + 4 * N;
    double* lC = Dfwd + 24 * N;
    double* lD = lC + 4 * N;
    StatePtrs<double> prim, cot1, cot0;
    for (int k = 0; k < 16; ++k) {
        prim.p[k] = (double*)a.in[k];
        cot1.p[k] = (double*)cot1_[k];
        cot0.p[k] = (double*)cot0_[k];
    }
    PlaneList L;
    int np = 0;
    for (int k = 4; k < 16; ++k) L.p[np++] = cot0.p[k];
    for (int k = 0; k < 4; ++k) L.p[np++] = lC + k * N;
    for (int k = 0; k < 24; ++k) L.p[np++] = lD + k * N;
    // L lists the window planes in PointWin order: point values, centres, increments
    IncrOut out;
    for (int k = 0; k < 12; ++k) out.dst[k] = cot0.p[4 + k];
    for (int k = 0; k < 4; ++k) { out.dst[12 + k] = cot0.p[k]; out.avg[k] = cot1.p[k]; }
    const double lam1 = a.dt / a.h, lam0 = 0.5 * lam1;
    {
        const int tx = (a.nx + kFBX - 1) / kFBX, nt = tx * ((a.ny + kFBY - 1) / kFBY);
        hipLaunchKernelGGL(k_adj_fwd, dim3(nt), dim3(kFNT), 0, a.stream, prim, C, Dfwd, L, np, a.scheme == 0,
                           a.nx, a.ny, tx, nt, a.gamma, lam0, lam1, a.status);
    }
    if (a.ev_begin) (void)hipEventRecord(a.ev_begin, a.stream);
    // point kernel: 8x8-cell blocks, two per CU (16x8 blocks at one per CU, whose
    // half-wavefronts read rows of 16 consecutive words, measured 3% slower)
    if (a.scheme == 0) launch_points<0, 8, 8, 2>(a, prim, C, Dfwd, cot1, L, lam0, lam1);
    else launch_points<1, 8, 8, 2>(a, prim, C, Dfwd, cot1, L, lam0, lam1);
    {
        const int tx = (a.nx + kIBX - 1) / kIBX, nt = tx * ((a.ny + kIBY - 1) / kIBY);
        hipLaunchKernelGGL(k_adj_incr, dim3(nt), dim3(kINT), kIncrLds, a.stream, prim, C, lD, lC, out, a.scheme == 0,
                           a.nx, a.ny, tx, nt, a.gamma, lam0, lam1);
    }
    if (a.ev_end) (void)hipEventRecord(a.ev_end, a.stream);
    return hipGetLastError();
}

hipError_t prepare_adjoint_f64() {
    const hipError_t e = hipFuncSetAttribute((const void*)k_adj_incr, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)kIncrLds);
    return e != hipSuccess ? e : prepare_points<8, 8, 2>();
}

size_t scratch_bytes_adjoint_f64(int nx, int ny) { return (size_t)nx * ny * (4 + 24 + 4 + 24) * sizeof(double); }

// ---- allocation-free form of the adjoint step ------------------------------------
// The scratch of launch_adjoint_f64 (56 planes: forward intermediates and reverse
// accumulators) and the status word, in a file-scope device array sized for grids of
// up to kNoallocMaxCells cells.  Every device that loads the library holds its own copy
// for the life of the process.  Only its device address (hipGetSymbolAddress, taken
// once per device with that device current) is ever handed to kernels; the array's name
// in host code is a host-side stand-in.  k_adj_fwd zeroes every accumulation plane for
// the grid's cells itself; the status word is cleared by a fill kernel on each call.
constexpr size_t kNoallocStatusWords = 32;   // 256 bytes: the planes stay 256-byte aligned
static __device__ __align__(256) double scratch[kNoallocStatusWords + kNoallocMaxCells * 56];

static_assert(sizeof(scratch) == kNoallocBytes, "scratch size as declared in af_internal.h");

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mutex;
void* g_noalloc_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_ptr(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_noalloc_mutex);
    if (!g_noalloc_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        // the point kernel's LDS exceeds the default limit: allowed once per device here
        e = prepare_adjoint_f64();
        if (e != hipSuccess) return e;
        g_noalloc_ptr[dev] = p;
    }
    *out = g_noalloc_ptr[dev];
    return hipSuccess;
}

hipError_t launch_adjoint_noalloc(StepArgs a, const void* const cot1[16], void* const cot0[16]) {
    void* p = nullptr;
    hipError_t e = noalloc_scratch_ptr(&p);
    if (e != hipSuccess) return e;
    a.status = (unsigned*)p;
    a.scratch = (double*)p + kNoallocStatusWords;
    e = launch_zero(p, kNoallocStatusWords * sizeof(double), a.stream);
    if (e != hipSuccess) return e;
    return launch_adjoint_f64(a, cot1, cot0);
}

}  // namespace af
