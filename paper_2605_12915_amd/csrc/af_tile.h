// Layout of the fused step's LDS tile and the work items of its phases: host and
// device code, so that a host build can walk every item of every phase through the
// node-level arithmetic with bounds-checked arrays (tests/tile_bounds.cpp).
#pragma once
#include <hip/hip_runtime.h>

#include "af_kernels.h"

namespace af {

// P, C and D share one row stride (PX), and phases 1 and 2 walk their items in rows of
// that stride (the items past a region's width idle), so the lanes of a wave read
// consecutive LDS words of every plane instead of colliding on banks where the rows of
// the item grid and of the array wrap at different widths (FP64 2% faster; FP32 4.6%,
// its bank-conflict cycles had outnumbered its active LDS cycles).
template <class T, int TX, int TY>
struct FusedTile {
    using S = T;
    static constexpr int X = TX, Y = TY;
    static constexpr int PX = TX + 5, PY = TY + 5;   // primitives: cells [-2, T+3)
    static constexpr int CX = TX + 4, CY = TY + 4;   // centres:    cells [-2, T+2)
    static constexpr int DX = TX + 3, DY = TY + 3;   // increments: node-cells [-1, T+2)
    static constexpr int VX = TX + 1, VY = TY + 1;   // flux nodes: node-cells [0, T]
    static constexpr int SC = PX, SD = PX;           // row strides of C, D
    T P[12][PY][PX];
    T C[4][CY][SC];
    union {
        T D[2][12][DY][SD];                          // [tau][fam*3 + var]
        struct {
            T FV[8][VY][VX];                         // V nodes: F~ (0..3), G~ (4..7)
            T FE[4][TY][VX];                         // Ev nodes: F~
            T GE[4][VY][TX];                         // Eh nodes: G~
        } F;
    };

    // element (y, x) of primitive plane k, centre plane k, increment plane q of duration t
    AF_HD T& p(int k, int y, int x) { return P[k][y][x]; }
    AF_HD T& c(int k, int y, int x) { return C[k][y][x]; }
    AF_HD T& d(int t, int q, int y, int x) { return D[t][q][y][x]; }
    AF_HD const T& p(int k, int y, int x) const { return P[k][y][x]; }
    AF_HD const T& c(int k, int y, int x) const { return C[k][y][x]; }
    AF_HD const T& d(int t, int q, int y, int x) const { return D[t][q][y][x]; }
    // whether the tile holds row y of increment plane q
    static AF_HD constexpr bool has_d(int, int) { return true; }
    // items of phases 0, 1 and 2 (those past a region's width included)
    static constexpr int NSTAGE = PX * PY, NCENTRE = SC * CY, NINCR = SD * DY;

    // Work items of the phases (item e of a workgroup's round-robin walk):
    // phase 0 stages node-cell (x, y) of P (cells x - 2, y - 2 of the tile),
    static AF_HD bool stage_item(int e, int& x, int& y) {
        x = e % PX;
        y = e / PX;
        return e < PX * PY;
    }
    // phase 1 recovers the centre of tile cell (x, y), x, y in [-2, T + 2),
    static AF_HD bool centre_item(int e, int& x, int& y) {
        x = e % SC - 2;
        y = e / SC - 2;
        return e < SC * CY && x + 2 < CX;
    }
    // phase 2 the increments of node-cell (x, y), x, y in [-1, T + 2),
    static AF_HD bool incr_item(int e, int& x, int& y) {
        x = e % SD - 1;
        y = e / SD - 1;
        return e < SD * DY && x + 1 < DX;
    }
    // phase 3 the point update of target family fam at node-cell (x, y) in [0, T]: V
    // targets (VX x VY), then Ev (VX x TY), then Eh (TX x VY), each family in rows of
    // RW lanes (0: rows as wide as the family's row of targets; lanes past it idle),
    template <int RW>
    struct Points {
        static constexpr int WV = RW ? RW : VX, WE = RW ? RW : VX, WH = RW ? RW : TX;
        static constexpr int NV = WV * VY, NE = WE * TY, NH = WH * VY, N = NV + NE + NH;
        static AF_HD bool item(int e, int& fam, int& x, int& y) {
            if (e >= N) return false;
            if (e < NV) { fam = F_V; x = e % WV; y = e / WV; return x < VX; }
            if (e < NV + NE) { fam = F_EV; x = (e - NV) % WE; y = (e - NV) / WE; return x < VX; }
            fam = F_EH; x = (e - NV - NE) % WH; y = (e - NV - NE) / WH;
            return x < TX;
        }
    };
    // and phase 4 updates the average of tile cell (x, y).
    static AF_HD bool update_item(int e, int& x, int& y) {
        x = e % TX;
        y = e / TX;
        return e < TX * TY;
    }
};

// The same tile packed for two workgroups per CU (TX = 15, T double): the planes of a row
// lie side by side ([y][plane][x]), and the planes that nothing reads in the last row (Ev of
// the primitives, C of the increments) come last in a row, so that the staged Ev of that
// row may fall on the centres' place (written after them) and the increments end early.
// A row of all planes is an odd multiple of 16 doubles, so that the two rows of 16 items
// that a half-wavefront of phase 3 touches fall on different banks; phases 1 and 2 walk their
// regions in columns [0, 16) row by row, then the columns left over, two or three to a row,
// which lie on few banks: most of the 0.98 conflict cycles per LDS instruction that the counters
// show (2048^2; 0.14 for the 31x10 tile, whose reads were merged).  The price of two workgroups
// on a CU; it is paid in the LDS, which is busy less than the vector units.
template <class T, int TX, int TY>
struct PackedTile {
    using S = T;
    using Full = FusedTile<T, TX, TY>;
    static constexpr int X = TX, Y = TY, W = TX >= 13 ? 16 : 8;
    static constexpr int PX = Full::PX, PY = Full::PY, CX = Full::CX, CY = Full::CY, DX = Full::DX, DY = Full::DY;
    static constexpr int VX = Full::VX, VY = Full::VY;
    static constexpr int SC = PX, SD = DX;           // row strides of C, D
    static constexpr int OC = (PY * 12 - 4) * PX;    // start of the centres
    T PC[OC + CY * 4 * SC];
    union {
        T Db[(DY * 24 - 6) * SD];
        struct {
            T FV[8][VY][VX];
            T FE[4][TY][VX];
            T GE[4][VY][TX];
        } F;
    };
    static_assert(DX >= W && CX >= W, "regions hold the walk's W columns");
    static_assert(4 * PX <= CY * 4 * SC, "the Ev row without a place falls on the centres");
    // planes of a row: V, Eh, Ev; increments V, Eh, Ev, C (each family's durations together)
    static AF_HD constexpr int slot(int fam) { return fam == F_EH ? 1 : (fam == F_EV ? 2 : fam); }
    static AF_HD constexpr int ps(int k) { return 4 * slot(k / 4) + k % 4; }
    static AF_HD constexpr int ds(int t, int q) { return 6 * slot(q / 3) + 3 * t + q % 3; }
    AF_HD T& p(int k, int y, int x) { return PC[(y * 12 + ps(k)) * PX + x]; }
    AF_HD T& c(int k, int y, int x) { return PC[OC + (y * 4 + k) * SC + x]; }
    AF_HD T& d(int t, int q, int y, int x) { return Db[(y * 24 + ds(t, q)) * SD + x]; }
    AF_HD const T& p(int k, int y, int x) const { return PC[(y * 12 + ps(k)) * PX + x]; }
    AF_HD const T& c(int k, int y, int x) const { return PC[OC + (y * 4 + k) * SC + x]; }
    AF_HD const T& d(int t, int q, int y, int x) const { return Db[(y * 24 + ds(t, q)) * SD + x]; }
    static AF_HD constexpr bool has_d(int q, int y) { return q / 3 != F_C || y < DY - 1; }

    // item e of a region of NX x NY: columns [0, W) in rows of W, then the rest
    template <int NX, int NY>
    static AF_HD bool split_item(int e, int& x, int& y) {
        if (e < W * NY) {
            x = e % W;
            y = e / W;
        } else {
            x = W + (e - W * NY) % (NX - W);
            y = (e - W * NY) / (NX - W);
        }
        return e < NX * NY;
    }
    static constexpr int NSTAGE = PX * PY, NCENTRE = CX * CY, NINCR = DX * DY;
    static AF_HD bool stage_item(int e, int& x, int& y) { return Full::stage_item(e, x, y); }
    static AF_HD bool centre_item(int e, int& x, int& y) {
        const bool in = split_item<CX, CY>(e, x, y);
        x -= 2;
        y -= 2;
        return in;
    }
    static AF_HD bool incr_item(int e, int& x, int& y) {
        const bool in = split_item<DX, DY>(e, x, y);
        x -= 1;
        y -= 1;
        return in;
    }
    template <int RW>
    using Points = typename Full::template Points<RW>;
    static AF_HD bool update_item(int e, int& x, int& y) { return Full::update_item(e, x, y); }
};

template <class Tile>
struct TileAcc {
    const Tile* t;
    AF_HD Prim<typename Tile::S> node(int fam, int x, int y) const {
        if (fam == F_C) return {t->c(0, y + 2, x + 2), t->c(1, y + 2, x + 2), t->c(2, y + 2, x + 2), t->c(3, y + 2, x + 2)};
        const int b = 4 * fam;
        return {t->p(b, y + 2, x + 2), t->p(b + 1, y + 2, x + 2), t->p(b + 2, y + 2, x + 2), t->p(b + 3, y + 2, x + 2)};
    }
};

template <class Tile>
struct TileInc {
    const Tile* t;
    int tau;
    AF_HD typename Tile::S inc(int fam, int x, int y, int var) const { return t->d(tau, fam * 3 + var, y + 1, x + 1); }
};

template <class T, int TX, int TY>
using LdsAcc = TileAcc<FusedTile<T, TX, TY>>;
template <class T, int TX, int TY>
using LdsInc = TileInc<FusedTile<T, TX, TY>>;

// The launches that take a grid's ntiles tiles, a workgroup of NT threads to each:
// launch(first tile, number).  HIP takes fewer than 2^32 work-items along an axis of a
// launch, and a grid of 2^31 cells has up to 2^31 / 40 tiles of 15 x 10 (four columns), 2.7e10
// work-items; at most 2^31 of them to a launch.
template <int NT, class F>
void tile_runs(int ntiles, const F& launch) {
    constexpr int most = (1 << 30) / NT * 2;
    for (int t = 0; t < ntiles; t += most) launch(t, ntiles - t < most ? ntiles - t : most);
}

AF_HD int wrap_any(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

// Periodic index of the tile window: one conditional shift when the grid is at least
// as large as the window (the usual case, decided per launch), else a modulo.
AF_HD int wrap_win(int v, int n, bool one) {
    if (one) return v < 0 ? v + n : (v >= n ? v - n : v);
    return wrap_any(v, n);
}

}  // namespace af
