// Node-level pieces of the RB-TAI step expressed against an accessor, shared by
// the multi-kernel path and the fused LDS-tiled kernel.
//
// An accessor A provides
//   Prim<T> A.node(fam, ci, cj)       primitive value of node family fam of cell
//                                     (ci, cj) (fam = F_C: the recovered centre),
// and an increment accessor D provides
//   T D.inc(fam, ci, cj, var)         acoustic increment (var 0: du, 1: dv, 2: dp)
//                                     of the node for the tau being processed.
// Cell indices are relative to whatever origin the accessor uses.
#pragma once
#include "af_device.h"

namespace af {

// Node freezing (Sec. 6.1 step 1): c_K, Z_K and 1 / Z_K.  Sets SB_CFL if c_K dt / h > 1/2
// (lam1 = dt / h) and SB_NONPHYS if the node state is not physical.
template <class T>
struct Freeze { T c, Z, iZ; };

template <class T, class Pol>
AF_HD Freeze<T> freeze_node(const Prim<T>& Wn, const Pol& pol, T lam1, unsigned& st) {
    const T rK = pol.rho(Wn.r), pK = pol.pr(Wn.p);
    if (!(rK > T(0)) || !(pK > T(0))) st |= SB_NONPHYS;
    // c = sqrt(gamma p / rho) and Z = rho c from one reciprocal square root:
    // 1 / Z = (gamma p rho)^(-1/2), c = gamma p / Z, Z = gamma p rho / Z
    const T gp = pol.gamma * pK, q = gp * rK;
    const T iZ = rsqrt_of(q);
    const Freeze<T> z{gp * iZ, q * iZ, iZ};
    if (!(z.c * lam1 <= T(0.5))) st |= SB_CFL;
    return z;
}

// Fence between stages whose live values together exceed a wave's registers: the sums so
// far are complete here (pinned to registers), and nothing moves across.
template <class T>
AF_HD void pin(T& x) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
}

template <class T>
AF_HD void stage_fence(T (&a1)[3][4], T (&a2)[3][4]) {
#pragma unroll
    for (int o = 0; o < 3; ++o)
#pragma unroll
        for (int m = 0; m < 4; ++m) { pin(a1[o][m]); pin(a2[o][m]); }
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// Values read before this point are read again after it instead of being kept.
AF_HD void reload_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// Variable VAR (0: p, 1: u, 2: v, 3: rho) at (a, b) half cells from the vertex of cell (i, j).
template <int VAR, class T, class A>
AF_HD T lattice(const A& acc, int i, int j, int a, int b) {
    const int fam = (a & 1) ? ((b & 1) ? F_C : F_EH) : ((b & 1) ? F_EV : F_V);
    const Prim<T> n = acc.node(fam, i + (a - (a & 1)) / 2, j + (b - (b & 1)) / 2);
    return VAR == 0 ? n.p : (VAR == 1 ? n.u : (VAR == 2 ? n.v : n.r));
}

// The nine nodal values [x-node][y-node] of one variable (0: p, 1: u, 2: v, 3: rho) of
// cell (ci, cj), and those of one increment.
template <int VAR, class T, class A>
AF_HD void cell_field(const A& acc, int ci, int cj, T f[3][3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) f[a][b] = lattice<VAR, T>(acc, ci, cj, a, b);
}

template <class T, class D>
AF_HD void cell_inc(const D& dinc, int ci, int cj, int var, T g[3][3]) {
    g[0][0] = dinc.inc(F_V, ci, cj, var);      g[1][0] = dinc.inc(F_EH, ci, cj, var);
    g[2][0] = dinc.inc(F_V, ci + 1, cj, var);  g[0][1] = dinc.inc(F_EV, ci, cj, var);
    g[1][1] = dinc.inc(F_C, ci, cj, var);      g[2][1] = dinc.inc(F_EV, ci + 1, cj, var);
    g[0][2] = dinc.inc(F_V, ci, cj + 1, var);  g[1][2] = dinc.inc(F_EH, ci, cj + 1, var);
    g[2][2] = dinc.inc(F_V, ci + 1, cj + 1, var);
}

// One coefficient along x (A) of every row, taken along y for both nodes of a pair.
template <int NX, bool FIRST, bool SECOND, int VAR, int A, class T>
AF_HD void pair_column(const T (&row)[5][NX], T (&a1)[3][4], T (&a2)[3][4]) {
    constexpr int W1 = NX == 5 ? W_V_NE : W_EH_U, W2 = NX == 5 ? W_EV_R : W_C;
    if constexpr (FIRST) {
        const T f[5] = {row[0][A], row[1][A], row[2][A], row[3][A], row[4][A]};
        T c[5];
        line<5, A == 0>(f, c);
        block_acc<W1, NX, 5, VAR, A>(c, a1);
    }
    if constexpr (SECOND) {
        const T f[3] = {row[2][A], row[3][A], row[4][A]};
        T c[3];
        line<3, true>(f, c);
        block_acc<W2, NX, 3, VAR, A>(c, a2);
    }
}

// Block sums of one variable for a pair of node families that read the same lines of
// nodes along x: NX = 5, the vertex (i, j) (first, full reach in y) and the vertical-edge
// midpoint (i, j + 1/2) (second, rows j .. j + 1) over x in [i - 1, i + 1]; NX = 3, the
// horizontal-edge midpoint (i + 1/2, j) and the centre (i + 1/2, j + 1/2) over x in
// [i, i + 1].
template <int NX, bool FIRST, bool SECOND, int VAR, class T, class A>
AF_HD void pair_blocks(const A& acc, int i, int j, T (&a1)[3][4], T (&a2)[3][4]) {
    constexpr int X0 = NX == 5 ? -2 : 0;
    T row[5][NX];
#pragma unroll
    for (int b = FIRST ? 0 : 2; b < 5; ++b) {
        T f[NX];
#pragma unroll
        for (int a = 0; a < NX; ++a) f[a] = lattice<VAR, T>(acc, i, j, X0 + a, b - 2);
        line<NX, true>(f, row[b]);
    }
    pair_column<NX, FIRST, SECOND, VAR, 0>(row, a1, a2);
    pair_column<NX, FIRST, SECOND, VAR, 1>(row, a1, a2);
    pair_column<NX, FIRST, SECOND, VAR, 2>(row, a1, a2);
    if constexpr (NX == 5) {
        pair_column<NX, FIRST, SECOND, VAR, 3>(row, a1, a2);
        pair_column<NX, FIRST, SECOND, VAR, 4>(row, a1, a2);
    }
}

// The node increments of a pair of families (NX as above) for both durations: inc1 of
// the first family's node, inc2 of the second's; [duration][du, dv, dp].  The sums are
// formed with the velocities first, in units of p / Z, then scaled to those of p.
template <int NX, bool FIRST = true, bool SECOND = true, class T, class A, class Pol>
AF_HD void pair_increments(const A& acc, int i, int j, const Pol& pol, T lam0, T lam1, T inc1[2][3], T inc2[2][3],
                           unsigned& st) {
    constexpr int F1 = NX == 5 ? F_V : F_EH, F2 = NX == 5 ? F_EV : F_C;
    T a1[3][4], a2[3][4];
    zero_acc(a1);
    zero_acc(a2);
    pair_blocks<NX, FIRST, SECOND, 1>(acc, i, j, a1, a2);
    stage_fence(a1, a2);
    pair_blocks<NX, FIRST, SECOND, 2>(acc, i, j, a1, a2);
    stage_fence(a1, a2);
    Freeze<T> z1{}, z2{};
    if constexpr (FIRST) {
        z1 = freeze_node(acc.node(F1, i, j), pol, lam1, st);
        scale_acc(a1, z1.Z);
    }
    if constexpr (SECOND) {
        z2 = freeze_node(acc.node(F2, i, j), pol, lam1, st);
        scale_acc(a2, z2.Z);
    }
    pair_blocks<NX, FIRST, SECOND, 0>(acc, i, j, a1, a2);
    stage_fence(a1, a2);
    if constexpr (FIRST) {
        block_increment(a1, z1.c * lam0, z1.iZ, inc1[0]);
        block_increment(a1, z1.c * lam1, z1.iZ, inc1[1]);
    }
    if constexpr (SECOND) {
        block_increment(a2, z2.c * lam0, z2.iZ, inc2[0]);
        block_increment(a2, z2.c * lam1, z2.iZ, inc2[1]);
    }
}

// The increments of one pair of families of cell (i, j), put(plane, value) with plane
// [duration][family * 3 + (du, dv, dp)].
template <int NX, class T, class A, class Pol, class Put>
AF_HD void put_pair(const A& acc, int i, int j, const Pol& pol, T lam0, T lam1, unsigned& st, const Put& put) {
    constexpr int F1 = NX == 5 ? F_V : F_EH, F2 = NX == 5 ? F_EV : F_C;
    T d1[2][3], d2[2][3];
    pair_increments<NX>(acc, i, j, pol, lam0, lam1, d1, d2, st);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            put(t * 12 + F1 * 3 + v, d1[t][v]);
            put(t * 12 + F2 * 3 + v, d2[t][v]);
        }
}

// All four nodes of cell (i, j).  One pair of families at a time: interleaving the pairs
// takes more registers than a wave holds at the kernels' occupancies.  Lines shared
// within a pair and each block entry applied once per node: 935 vector instructions and
// 91 LDS reads per node-cell in the FP64 step kernel, against 1470 and 130 with every
// wedge transformed on its own (FP64 step 2048^2 0.98 -> 0.86 ms, FP32 4096^2 1.87 ->
// 1.64 ms).
template <class T, class A, class Pol, class Put>
AF_HD void cell_increments(const A& acc, int i, int j, const Pol& pol, T lam0, T lam1, unsigned& st, const Put& put) {
    put_pair<5>(acc, i, j, pol, lam0, lam1, st, put);
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
#endif
    put_pair<3>(acc, i, j, pol, lam0, lam1, st, put);
}

// One family alone (the same operations, the lines not shared).
template <int FAM, class T, class A, class Pol>
AF_HD void node_increments(const A& acc, int i, int j, const Pol& pol, T lam0, T lam1, T inc[2][3],
                           unsigned& st) {
    T unused[2][3];
    if constexpr (FAM == F_V) pair_increments<5, true, false>(acc, i, j, pol, lam0, lam1, inc, unused, st);
    else if constexpr (FAM == F_EV) pair_increments<5, false, true>(acc, i, j, pol, lam0, lam1, unused, inc, st);
    else if constexpr (FAM == F_EH) pair_increments<3, true, false>(acc, i, j, pol, lam0, lam1, inc, unused, st);
    else pair_increments<3, false, true>(acc, i, j, pol, lam0, lam1, unused, inc, st);
}

template <int FAM>
struct FamOffset;
template <> struct FamOffset<F_V> { static constexpr double ox = 0.0, oy = 0.0; };
template <> struct FamOffset<F_EV> { static constexpr double ox = 0.0, oy = 0.5; };
template <> struct FamOffset<F_EH> { static constexpr double ox = 0.5, oy = 0.0; };

// The same offsets for a target family known only at run time (cell units).
template <class T>
AF_HD T fam_ox(int fam) { return fam == F_EH ? T(0.5) : T(0); }
template <class T>
AF_HD T fam_oy(int fam) { return fam == F_EV ? T(0.5) : T(0); }

// Locate an offset (cell units, relative to the target's own cell) in its cell:
// integer shift and local coordinate in [-1, 1].  A displacement of one cell or
// more (or NaN) raises SB_FOOT and is replaced by the node itself, which keeps
// every gather inside the two-cell halo.
template <class T>
AF_HD void locate(T off, T o, int& cell, T& xi, unsigned& st) {
    if (!(fabs(off - o) < T(1))) { st |= SB_FOOT; off = o; }
    T fl = floor(off);
    cell = (int)fl;
    xi = T(2) * (off - fl) - T(1);
}

// Transported (SCHEME 0, eq. transported-update) or additive (SCHEME 1,
// eq. barsukow-additive) point update of the target of family fam (F_V, F_EV or
// F_EH) at (i, j) for duration tau = lam h (Sec. 6.1 steps 3-4).  The family may be
// a run-time value (lanes of one wavefront then share one instruction stream) or a
// constant (point_update<FAM, ...>).
// The convective foot of the target of family fam at (i, j) (node value WP) after
// tau = lam h, by the two Picard stages (eq. adv-footpoint; Sec. 6.1 step 3): the
// foot's cell (ci, cj) and its local coordinates (xi, eta) in [-1, 1].
template <class T, class A, class Pol>
AF_HD void picard_foot(const A& acc, int fam, int i, int j, const Pol& pol, T lam, const Prim<T>& WP, int& ci,
                       int& cj, T& xi, T& eta, unsigned& st) {
    const T ox = fam_ox<T>(fam), oy = fam_oy<T>(fam);
    int cx, cy;
    T xm, xp, ym, yp;
    // first Picard step: at a node the reconstruction equals the node value
    locate(ox - lam * pol.vu(WP.u), ox, cx, xi, st);
    locate(oy - lam * pol.vv(WP.v), oy, cy, eta, st);
    lag_pm(xi, xm, xp);
    lag_pm(eta, ym, yp);
    T fu[3][3], fv[3][3];
    cell_field<1>(acc, i + cx, j + cy, fu);
    cell_field<2>(acc, i + cx, j + cy, fv);
    T u1 = q2(xm, xp, ym, yp, fu), v1 = q2(xm, xp, ym, yp, fv);
    // second Picard step from P with the velocity at the first foot
    locate(ox - lam * pol.vu(u1), ox, cx, xi, st);
    locate(oy - lam * pol.vv(v1), oy, cy, eta, st);
    ci = i + cx;
    cj = j + cy;
}

//
// SUM (SCHEME 0): the increment accessor holds u + du and v + dv in place of du and dv.
// Interpolation is linear and both velocities are read at the same foot, so one Q2
// evaluation of the sum gives the new velocity: five evaluations per duration at the
// second foot instead of seven.
template <int SCHEME, bool SUM = false, class T, class A, class D, class Pol>
AF_HD Prim<T> point_update_f(const A& acc, const D& dinc, int fam, int i, int j, const Pol& pol, T lam,
                             unsigned& st) {
    Prim<T> WP = acc.node(fam, i, j);
    int ci, cj;
    T xi, eta, xm, xp, ym, yp;
    picard_foot(acc, fam, i, j, pol, lam, WP, ci, cj, xi, eta, st);
    lag_pm(xi, xm, xp);
    lag_pm(eta, ym, yp);
    T g[3][3];
    Prim<T> Wf;
    cell_field<3>(acc, ci, cj, g);
    Wf.r = q2(xm, xp, ym, yp, g);
    cell_field<0>(acc, ci, cj, g);
    Wf.p = q2(xm, xp, ym, yp, g);
    if constexpr (!SUM) {
        cell_field<1>(acc, ci, cj, g);
        Wf.u = q2(xm, xp, ym, yp, g);
        cell_field<2>(acc, ci, cj, g);
        Wf.v = q2(xm, xp, ym, yp, g);
    }
    T du, dv, dp, rho_over_c2;
    if constexpr (SCHEME == 0) {
        cell_inc(dinc, ci, cj, 0, g);
        du = q2(xm, xp, ym, yp, g);
        cell_inc(dinc, ci, cj, 1, g);
        dv = q2(xm, xp, ym, yp, g);
        cell_inc(dinc, ci, cj, 2, g);
        dp = q2(xm, xp, ym, yp, g);
        rho_over_c2 = quot(pol.rho(Wf.r), pol.gamma * pol.pr(Wf.p));    // 1 / c^2 at the foot
    } else {
        du = dinc.inc(fam, i, j, 0);
        dv = dinc.inc(fam, i, j, 1);
        dp = dinc.inc(fam, i, j, 2);
        rho_over_c2 = quot(pol.rho(WP.r), pol.gamma * pol.pr(WP.p));    // frozen 1 / c^2 at P
    }
    if constexpr (SUM) return Prim<T>{Wf.r + dp * rho_over_c2, du, dv, Wf.p + dp};
    else return Prim<T>{Wf.r + dp * rho_over_c2, Wf.u + du, Wf.v + dv, Wf.p + dp};
}

template <int FAM, int SCHEME, class T, class A, class D, class Pol>
AF_HD Prim<T> point_update(const A& acc, const D& dinc, int i, int j, const Pol& pol, T lam, unsigned& st) {
    return point_update_f<SCHEME>(acc, dinc, FAM, i, j, pol, lam, st);
}

// Both durations of one target at once.  The two Picard stages of both durations
// normally stay in one cell, fixed by the sign of the node velocity; that cell's
// nine nodes and both increment sets are gathered once and every stage is checked
// to stay in it.  Lanes whose feet leave it take the general path above, which
// performs the same arithmetic (so the results do not depend on the path).
template <int SCHEME, bool SUM = false, class T, class A, class D, class Pol>
AF_HD void point_update_pair_f(const A& acc, const D& d0, const D& d1, int fam, int i, int j, const Pol& pol,
                               T lam0, T lam1, unsigned& st, Prim<T>& wh, Prim<T>& w1) {
    const T ox = fam_ox<T>(fam), oy = fam_oy<T>(fam);
    const Prim<T> WP = acc.node(fam, i, j);
    // candidate cell from the longer first-stage displacement
    const T uP = pol.vu(WP.u), vP = pol.vv(WP.v);
    const T ex = ox - lam1 * uP, ey = oy - lam1 * vP;
    bool fast = (fabs(ex - ox) < T(1)) && (fabs(ey - oy) < T(1));
    int cx = 0, cy = 0;
    Prim<T> wr[2];
    if (fast) {
        const T fcx = floor(ex), fcy = floor(ey);
        cx = (int)fcx;
        cy = (int)fcy;
        const int ci = i + cx, cj = j + cy;
        // field by field, so that nine nodal values are live at a time: the velocities (both
        // Picard stages' positions), then density, pressure and the increments at the feet
        T xm[2], xp[2], ym[2], yp[2], g[3][3];
        Prim<T> Wf[2];
        {
            T fu[3][3], fv[3][3];
            cell_field<1>(acc, ci, cj, fu);
            cell_field<2>(acc, ci, cj, fv);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const T lam = t ? lam1 : lam0;
                T xi, eta, fl;
                // first Picard stage
                const T o1x = ox - lam * uP, o1y = oy - lam * vP;
                fl = floor(o1x); fast = fast && (fl == fcx); xi = T(2) * (o1x - fl) - T(1);
                fl = floor(o1y); fast = fast && (fl == fcy); eta = T(2) * (o1y - fl) - T(1);
                lag_pm(xi, xm[t], xp[t]);
                lag_pm(eta, ym[t], yp[t]);
                const T u1 = q2(xm[t], xp[t], ym[t], yp[t], fu), v1 = q2(xm[t], xp[t], ym[t], yp[t], fv);
                // second stage
                const T o2x = ox - lam * pol.vu(u1), o2y = oy - lam * pol.vv(v1);
                fast = fast && (fabs(o2x - ox) < T(1)) && (fabs(o2y - oy) < T(1));
                fl = floor(o2x); fast = fast && (fl == fcx); xi = T(2) * (o2x - fl) - T(1);
                fl = floor(o2y); fast = fast && (fl == fcy); eta = T(2) * (o2y - fl) - T(1);
                lag_pm(xi, xm[t], xp[t]);
                lag_pm(eta, ym[t], yp[t]);
            }
        }
        if constexpr (!SUM) {
            // the velocities gathered a second time: kept from the first stage they would
            // exceed the 128 registers of the FP64 15x10 kernel (the FP32 additive kernels, of
            // 119 to 128 registers, take the second gather with it)
            reload_fence();
            cell_field<1>(acc, ci, cj, g);
#pragma unroll
            for (int t = 0; t < 2; ++t) Wf[t].u = q2(xm[t], xp[t], ym[t], yp[t], g);
            cell_field<2>(acc, ci, cj, g);
#pragma unroll
            for (int t = 0; t < 2; ++t) Wf[t].v = q2(xm[t], xp[t], ym[t], yp[t], g);
        }
        cell_field<3>(acc, ci, cj, g);
#pragma unroll
        for (int t = 0; t < 2; ++t) Wf[t].r = q2(xm[t], xp[t], ym[t], yp[t], g);
        cell_field<0>(acc, ci, cj, g);
#pragma unroll
        for (int t = 0; t < 2; ++t) Wf[t].p = q2(xm[t], xp[t], ym[t], yp[t], g);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const D& dd = t ? d1 : d0;
            T d[3];
            if constexpr (SCHEME == 0) {
#pragma unroll
                for (int var = 0; var < 3; ++var) {
                    cell_inc(dd, ci, cj, var, g);
                    d[var] = q2(xm[t], xp[t], ym[t], yp[t], g);
                }
            } else {
#pragma unroll
                for (int var = 0; var < 3; ++var) d[var] = dd.inc(fam, i, j, var);
            }
            // 1 / c^2 at the foot (transported) or frozen at the target (additive)
            const T rho_over_c2 = SCHEME == 0 ? quot(pol.rho(Wf[t].r), pol.gamma * pol.pr(Wf[t].p))
                                              : quot(pol.rho(WP.r), pol.gamma * pol.pr(WP.p));
            if constexpr (SUM) wr[t] = Prim<T>{Wf[t].r + d[2] * rho_over_c2, d[0], d[1], Wf[t].p + d[2]};
            else wr[t] = Prim<T>{Wf[t].r + d[2] * rho_over_c2, Wf[t].u + d[0], Wf[t].v + d[1], Wf[t].p + d[2]};
        }
    }
    if (fast) {
        wh = wr[0];
        w1 = wr[1];
    } else {
        wh = point_update_f<SCHEME, SUM>(acc, d0, fam, i, j, pol, lam0, st);
        w1 = point_update_f<SCHEME, SUM>(acc, d1, fam, i, j, pol, lam1, st);
    }
}

template <int FAM, int SCHEME, bool SUM = false, class T, class A, class D, class Pol>
AF_HD void point_update_pair(const A& acc, const D& d0, const D& d1, int i, int j, const Pol& pol, T lam0, T lam1,
                             unsigned& st, Prim<T>& wh, Prim<T>& w1) {
    point_update_pair_f<SCHEME, SUM>(acc, d0, d1, FAM, i, j, pol, lam0, lam1, st, wh, w1);
}

}  // namespace af
