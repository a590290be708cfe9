// Arithmetic of the reverse-mode step (transposed Sec. 6.1 dataflow), written once
// for the scalar type T and against small accessor types, so that the adjoint
// kernels (af_adjoint.hip, T = double, LDS windows) and the host operation count
// (count_flops.cpp, an operation-counting scalar) run the very same code.
//
// Accessors:
//   S  staged forward state: S.base(i, j), S.at(plane, base, off) with the window
//      plane numbering (0..11 point values fam * 4 + (rho, u, v, p), 12..15 recovered
//      centres, 16..39 increments tau * 12 + fam * 3 + (u, v, p)); row stride S_::kRX.
//   O  scatter target with the same plane numbering (its own row stride O_::kRX):
//      O.base(i, j), O.addb(plane, base, off, value), O.node(fam, i, j, g[4]); every
//      add is one accumulation.
//   A  forward nodes by cell: A.node(fam, i, j) (fam = F_C: recovered centre).
//   CT cotangent of the step's output: CT.get(plane, i, j) (periodic).
// The floor() that locates a foot is piecewise constant: its derivative is zero.
#pragma once
#include "af_kernels.h"

namespace af {

// Family of node [a][b] of a cell, and its first plane in the scatter window (point
// values fam * 4, centre 12).
AF_HD constexpr int fam_of(int a, int b) {
    return (a == 1 && b == 1) ? F_C : (a == 1 ? F_EH : (b == 1 ? F_EV : F_V));
}
AF_HD constexpr int win_plane(int fam) { return fam == F_C ? 12 : 4 * fam; }

template <class T>
AF_HD void lagr(T s, T l[3], T dl[3]) {
    l[0] = T(0.5) * s * (s - T(1));
    l[1] = T(1) - s * s;
    l[2] = T(0.5) * s * (s + T(1));
    dl[0] = s - T(0.5);
    dl[1] = T(-2) * s;
    dl[2] = s + T(0.5);
}

// Flux Jacobians transposed: g += (dF/dW)^T nu, W = (rho, u, v, p).
// (Each product shared by several terms is formed once, as the compiled code does; the
// one quotient, 1 / (gamma - 1), is the same in every call and formed once per thread.)
template <class T>
AF_HD void flux_x_T(const Prim<T>& w, T gamma, const T nu[4], T g[4]) {
    const T gm1i = T(1) / (gamma - T(1));
    const T uu = w.u * w.u, uv = w.u * w.v, ru = w.r * w.u;
    const T q2 = T(0.5) * (uu + w.v * w.v);
    const T E = w.p * gm1i + w.r * q2;
    g[0] += nu[0] * w.u + nu[1] * uu + nu[2] * uv + nu[3] * w.u * q2;
    g[1] += nu[0] * w.r + nu[1] * T(2) * ru + nu[2] * w.r * w.v + nu[3] * (E + w.p + ru * w.u);
    g[2] += nu[2] * ru + nu[3] * ru * w.v;
    g[3] += nu[1] + nu[3] * w.u * gamma * gm1i;
}

template <class T>
AF_HD void flux_y_T(const Prim<T>& w, T gamma, const T nu[4], T g[4]) {
    const T gm1i = T(1) / (gamma - T(1));
    const T vv = w.v * w.v, uv = w.u * w.v, rv = w.r * w.v;
    const T q2 = T(0.5) * (w.u * w.u + vv);
    const T E = w.p * gm1i + w.r * q2;
    g[0] += nu[0] * w.v + nu[1] * uv + nu[2] * vv + nu[3] * w.v * q2;
    g[1] += nu[1] * rv + nu[3] * rv * w.u;
    g[2] += nu[0] * w.r + nu[1] * w.r * w.u + nu[2] * T(2) * rv + nu[3] * (E + w.p + rv * w.v);
    g[3] += nu[2] + nu[3] * w.v * gamma * gm1i;
}

// Transposed point update of target FAM at (i, j) for the duration tau_t = lam h;
// WP = the target's time-n value.  SCHEME 0: transported update (the increments are
// interpolated at the foot, the density closure uses c^2 at the foot); the increment planes
// hold u + du, v + dv and dp, as in the step, and so do their cotangents: what the
// velocities themselves get from the foot is the sum of those planes' cotangents over the
// durations, which the increments' kernel adds.  SCHEME 1: additive update (the
// target's own increments, c^2 frozen at the target).
// The forward value w is recomputed here and its cotangent formed from the flux
// cotangents: lw = ws * (dF/dW)^T nuF + ws * (dG/dW)^T nuG (+ extra: the cotangent
// of the new point value itself, for the full step).  The contributions to the target's own
// node (through the first foot position) are added to gself, those to the increments go to
// the window; those to the nodes of the two foot cells are returned (FootAdj).  MODE 1
// returns them only.
template <class T>
struct FootAdj {
    T lx1[3], ly1[3], lx2[3], ly2[3];   // Lagrange weights of the two Picard stages' positions
    T l[4], lu1, lv1;                   // adjoint of Q2(W) at the second, of Q2(u), Q2(v) at the first
    int wb1, wb2;                       // window offsets of their cells
};

template <int FAM, int SCHEME, int MODE, class T, class S_, class O_>
AF_HD void point_update_adj(const S_& S, const O_& O, int t, int i, int j, const Prim<T>& WP, T gamma, T lam,
                            const T nuF[4], const T nuG[4], T ws, const T* extra, T gself[4], FootAdj<T>& R) {
    const T ox = T(FamOffset<FAM>::ox), oy = T(FamOffset<FAM>::oy);
    constexpr int RX = O_::kRX, SRX = S_::kRX;   // row strides of the window and of the staged state
    constexpr bool SUM = SCHEME == 0;
    unsigned st = 0;
    // ---- forward recomputation ----
    int cx, cy;
    T xi, eta, dlx[3], dly[3];
    locate(ox - lam * WP.u, ox, cx, xi, st);
    locate(oy - lam * WP.v, oy, cy, eta, st);
    lagr(xi, R.lx1, dlx);
    lagr(eta, R.ly1, dly);
    T u1 = T(0), v1 = T(0), du1x = T(0), du1y = T(0), dv1x = T(0), dv1y = T(0);
    R.wb1 = O.base(i + cx, j + cy);
    const int sb1 = S.base(i + cx, j + cy);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const int f = fam_of(a, b), soff = (b == 2 ? SRX : 0) + (a == 2 ? 1 : 0);
            const T nu_ = S.at(win_plane(f) + 1, sb1, soff), nv_ = S.at(win_plane(f) + 2, sb1, soff);
            const T w = R.lx1[a] * R.ly1[b], wx = dlx[a] * R.ly1[b], wy = R.lx1[a] * dly[b];
            u1 += w * nu_;
            v1 += w * nv_;
            du1x += wx * nu_;
            du1y += wy * nu_;
            dv1x += wx * nv_;
            dv1y += wy * nv_;
        }
    locate(ox - lam * u1, ox, cx, xi, st);
    locate(oy - lam * v1, oy, cy, eta, st);
    lagr(xi, R.lx2, dlx);
    lagr(eta, R.ly2, dly);
    R.wb2 = O.base(i + cx, j + cy);
    const int sb2 = S.base(i + cx, j + cy);
    T Wf[4] = {T(0), T(0), T(0), T(0)}, dWx[4] = {T(0), T(0), T(0), T(0)}, dWy[4] = {T(0), T(0), T(0), T(0)};
    T Df[3] = {T(0), T(0), T(0)}, dDx[3] = {T(0), T(0), T(0)}, dDy[3] = {T(0), T(0), T(0)};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const T w = R.lx2[a] * R.ly2[b], wx = dlx[a] * R.ly2[b], wy = R.lx2[a] * dly[b];
            const int f = fam_of(a, b), soff = (b == 2 ? SRX : 0) + (a == 2 ? 1 : 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (SUM && (q == 1 || q == 2)) continue;
                const T v = S.at(win_plane(f) + q, sb2, soff);
                Wf[q] += w * v; dWx[q] += wx * v; dWy[q] += wy * v;
            }
            if constexpr (SUM) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const T v = S.at(16 + t * 12 + f * 3 + q, sb2, soff);
                    Df[q] += w * v; dDx[q] += wx * v; dDy[q] += wy * v;
                }
            }
        }
    const int wbP = O.base(i, j);
    if constexpr (!SUM) {
        const int sbP = S.base(i, j);
#pragma unroll
        for (int q = 0; q < 3; ++q) Df[q] = S.at(16 + t * 12 + FAM * 3 + q, sbP, 0);
    }
    // ---- reverse ----
    // compose: rho = rho_f + dp rho_K / (gamma p_K), u = u_f + du, v = v_f + dv, p = p_f + dp,
    // with K the foot (SCHEME 0) or the target (SCHEME 1)
    const T rK = SUM ? Wf[0] : WP.r, pK = SUM ? Wf[3] : WP.p;
    const T qinv = T(1) / (gamma * pK), rq = rK * qinv;
    T lw[4] = {T(0), T(0), T(0), T(0)};
    {
        const Prim<T> w{Wf[0] + Df[2] * rq, SUM ? Df[0] : Wf[1] + Df[0], SUM ? Df[1] : Wf[2] + Df[1], Wf[3] + Df[2]};
        T nu[4];
        if constexpr (FAM != F_EH) {
#pragma unroll
            for (int k = 0; k < 4; ++k) nu[k] = ws * nuF[k];
            flux_x_T(w, gamma, nu, lw);
        }
        if constexpr (FAM != F_EV) {
#pragma unroll
            for (int k = 0; k < 4; ++k) nu[k] = ws * nuG[k];
            flux_y_T(w, gamma, nu, lw);
        }
        if (extra)
#pragma unroll
            for (int k = 0; k < 4; ++k) lw[k] += extra[k];
    }
    const T lDf[3] = {lw[1], lw[2], lw[3] + lw[0] * rq};
    const T ldq = lw[0] * Df[2] * qinv;
    R.l[1] = SUM ? T(0) : lw[1];
    R.l[2] = SUM ? T(0) : lw[2];
    if constexpr (SUM) {
        R.l[0] = lw[0] + ldq;
        R.l[3] = lw[3] - ldq * gamma * rq;   // rho_K / p_K = gamma rq
    } else {
        R.l[0] = lw[0];
        R.l[3] = lw[3];
        // the frozen rho_K / (gamma p_K) at the target, and its own increments
        if constexpr (MODE == 0) {
            gself[0] += ldq;
            gself[3] -= ldq * gamma * rq;
#pragma unroll
            for (int q = 0; q < 3; ++q) O.addb(16 + t * 12 + FAM * 3 + q, wbP, 0, lDf[q]);
        }
    }
    // foot position: xi2 = 2 (off - floor(off)) - 1, off = ox - lam u1
    T lxi2 = T(0), leta2 = T(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (SUM && (q == 1 || q == 2)) continue;
        lxi2 += R.l[q] * dWx[q];
        leta2 += R.l[q] * dWy[q];
    }
    if constexpr (SUM) {
#pragma unroll
        for (int q = 0; q < 3; ++q) { lxi2 += lDf[q] * dDx[q]; leta2 += lDf[q] * dDy[q]; }
    }
    R.lu1 = T(-2) * lam * lxi2;
    R.lv1 = T(-2) * lam * leta2;
    if constexpr (MODE == 1) return;
    if constexpr (SUM) {
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const T w = R.lx2[a] * R.ly2[b];
                const int f = fam_of(a, b), off = (b == 2 ? RX : 0) + (a == 2 ? 1 : 0);
#pragma unroll
                for (int q = 0; q < 3; ++q) O.addb(16 + t * 12 + f * 3 + q, R.wb2, off, w * lDf[q]);
            }
    }
    const T lxi1 = R.lu1 * du1x + R.lv1 * dv1x, leta1 = R.lu1 * du1y + R.lv1 * dv1y;
    gself[1] += T(-2) * lam * lxi1;
    gself[2] += T(-2) * lam * leta1;
}

// Contributions to the nodes of a foot cell at window offset wb: the second stage of SECOND and
// the first stage of FIRST of N durations that share the cell, one addition per node and plane.
template <bool SUM, int N, bool FIRST, bool SECOND, class T, class O_>
AF_HD void foot_scatter(const O_& O, int wb, const FootAdj<T>* R) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            T g[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
            for (int t = 0; t < N; ++t) {
                if constexpr (SECOND) {
                    const T w = R[t].lx2[a] * R[t].ly2[b];
                    g[0] += w * R[t].l[0];
                    if constexpr (!SUM) { g[1] += w * R[t].l[1]; g[2] += w * R[t].l[2]; }
                    g[3] += w * R[t].l[3];
                }
                if constexpr (FIRST) {
                    const T w = R[t].lx1[a] * R[t].ly1[b];
                    g[1] += w * R[t].lu1;
                    g[2] += w * R[t].lv1;
                }
            }
            const int pl = win_plane(fam_of(a, b)), off = (b == 2 ? O_::kRX : 0) + (a == 2 ? 1 : 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((q == 1 || q == 2) ? (FIRST || (SECOND && !SUM)) : SECOND) O.addb(pl + q, wb, off, g[q]);
        }
}

// Reverse sweep of one target (family FAM of node-cell (i, j)): the adjoints of the
// edge fluxes it feeds, from the averages' cotangents, then of its three time levels
// (w^n directly, w^{n+1/2} and w^{n+1} through the transposed point update).
// The two Picard stages of both durations normally lie in one foot cell: each node then
// gets one addition per plane for all four.  MODE 0 does that and returns 1 for a target
// whose feet lie in different cells, whose contributions to the foot cells it leaves out;
// MODE 1 recomputes such a target and scatters those, stage by stage (the caller runs it for
// the rare wavefronts that need it, so that the common path keeps one scatter per node and
// plane and nothing live for the other).
template <int FAM, int SCHEME, int MODE, class T, class S_, class CT, class O_>
AF_HD unsigned point_adj_target(const S_& S, const CT& cot1, const O_& O, int i, int j, T gamma, T lam0, T lam1,
                                unsigned fix = 0) {
    constexpr bool SUM = SCHEME == 0;
    // cotangents of the time-integrated edge fluxes at this node: F at V and Ev, G at
    // V and Eh; spatial Simpson weights 1/6 (V, two edges each) and 4/6 (edge midpoints)
    T nuF[4] = {T(0), T(0), T(0), T(0)}, nuG[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const T lij = cot1.get(k, i, j);
        const T muF_ij = lam1 * (lij - cot1.get(k, i - 1, j));
        const T muG_ij = lam1 * (lij - cot1.get(k, i, j - 1));
        if constexpr (FAM == F_V) {
            const T lijm = cot1.get(k, i, j - 1), limj = cot1.get(k, i - 1, j), limjm = cot1.get(k, i - 1, j - 1);
            const T muF_ijm = lam1 * (lijm - limjm);
            const T muG_imj = lam1 * (limj - limjm);
            nuF[k] = (muF_ij + muF_ijm) * T(1.0 / 6.0);
            nuG[k] = (muG_ij + muG_imj) * T(1.0 / 6.0);
        } else if constexpr (FAM == F_EV) {
            nuF[k] = muF_ij * T(4.0 / 6.0);
        } else {
            nuG[k] = muG_ij * T(4.0 / 6.0);
        }
    }
    const int wb = O.base(i, j), sb = S.base(i, j);
    const int pl = win_plane(FAM);
    const Prim<T> w0{S.at(pl, sb, 0), S.at(pl + 1, sb, 0), S.at(pl + 2, sb, 0), S.at(pl + 3, sb, 0)};
    T g[4] = {T(0), T(0), T(0), T(0)};
    if (MODE == 1 && !fix) return 0u;
    // time level n (time-Simpson weight 1/6): the node itself
    if constexpr (MODE == 0) {
        T nu[4];
        if constexpr (FAM != F_EH) {
#pragma unroll
            for (int k = 0; k < 4; ++k) nu[k] = nuF[k] * T(1.0 / 6.0);
            flux_x_T(w0, gamma, nu, g);
        }
        if constexpr (FAM != F_EV) {
#pragma unroll
            for (int k = 0; k < 4; ++k) nu[k] = nuG[k] * T(1.0 / 6.0);
            flux_y_T(w0, gamma, nu, g);
        }
    }
    // n + 1/2 (weight 4/6) and n + 1 (weight 1/6; also an output of the step)
    FootAdj<T> R[2];
    point_update_adj<FAM, SCHEME, MODE>(S, O, 0, i, j, w0, gamma, lam0, nuF, nuG, T(4.0 / 6.0), (const T*)nullptr, g,
                                        R[0]);
    const T extra[4] = {cot1.get(4 + 4 * FAM, i, j), cot1.get(5 + 4 * FAM, i, j), cot1.get(6 + 4 * FAM, i, j),
                        cot1.get(7 + 4 * FAM, i, j)};
    point_update_adj<FAM, SCHEME, MODE>(S, O, 1, i, j, w0, gamma, lam1, nuF, nuG, T(1.0 / 6.0), extra, g, R[1]);
    if constexpr (MODE == 1) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            foot_scatter<SUM, 1, false, true>(O, R[t].wb2, R + t);
            foot_scatter<SUM, 1, true, false>(O, R[t].wb1, R + t);
        }
        return 0u;
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) O.addb(pl + q, wb, 0, g[q]);
        const bool same = R[0].wb1 == R[0].wb2 && R[1].wb1 == R[0].wb2 && R[1].wb2 == R[0].wb2;
        if (same) foot_scatter<SUM, 2, true, true>(O, R[0].wb2, R);
        return same ? 0u : 1u;
    }
}

// Transposed line transform (see line): coefficients' adjoint -> nodes' adjoint.
template <int N, class T>
AF_HD void line_T(const T* c, T* f) {
    if constexpr (N == 5) {
        const T e1 = T(4) * c[1] - T(2) * c[2], e2 = c[2] - c[1];
        const T o1 = T(4) * c[3] - T(2) * c[4], o2 = c[4] - c[3];
        f[0] = e2 - o2;
        f[1] = e1 - o1;
        f[2] = c[0] - T(2) * (e1 + e2);
        f[3] = e1 + o1;
        f[4] = e2 + o2;
    } else {
        f[0] = c[2] - c[1];
        f[1] = c[0] - T(2) * c[2];
        f[2] = c[2] + c[1];
    }
}

// Transposed block (see block_acc): adjoint of the sums -> adjoint of the coefficients
// along y of variable VAR's coefficient A along x.
template <int W, int NX, int NY, int VAR, int A, int B, int OUT, class T>
AF_HD void block_term_T(const T (&la)[3][4], T (&c)[NY]) {
    constexpr LineTerm x = LineTerms<NX>::t[A], y = LineTerms<NY>::t[B];
    constexpr bool match = x.odd == ((OUT == 1) != (VAR == 1)) && y.odd == ((OUT == 2) != (VAR == 2));
    if constexpr (match && x.pow + y.pow > 0) {
        constexpr double w = kBlk[W][x.pow][y.pow][3 * OUT + VAR] * x.scale * y.scale;
        if constexpr (w != 0.0) c[B] += T(w) * la[OUT][x.pow + y.pow - 1];
    }
}

template <int W, int NX, int NY, int VAR, int A, class T, int... K>
AF_HD void block_terms_T(const T (&la)[3][4], T (&c)[NY], std::integer_sequence<int, K...>) {
    (block_term_T<W, NX, NY, VAR, A, K / 3, K % 3>(la, c), ...);
}

// One coefficient along x (A) of every row of the lines shared by a pair of families
// (see pair_column), from the adjoint of both nodes' sums.
template <int NX, int VAR, int A, class T>
AF_HD void pair_column_T(const T (&la1)[3][4], const T (&la2)[3][4], T (&row)[5][NX]) {
    constexpr int W1 = NX == 5 ? W_V_NE : W_EH_U, W2 = NX == 5 ? W_EV_R : W_C;
    T c1[5] = {T(0), T(0), T(0), T(0), T(0)}, c2[3] = {T(0), T(0), T(0)}, f1[5], f2[3];
    block_terms_T<W1, NX, 5, VAR, A>(la1, c1, std::make_integer_sequence<int, 15>());
    block_terms_T<W2, NX, 3, VAR, A>(la2, c2, std::make_integer_sequence<int, 9>());
    line_T<5>(c1, f1);
    line_T<3>(c2, f2);
#pragma unroll
    for (int b = 0; b < 5; ++b) row[b][A] = b >= 2 ? f1[b] + f2[b - 2] : f1[b];
}

// Adjoint of the nodal values of one variable (0: p, 1: u, 2: v) from a pair's sums, each
// node's share scattered once; own1, own2: what the two nodes themselves get besides.
template <int NX, int VAR, class T, class O_>
AF_HD void pair_scatter(const O_& O, int i, int j, const T (&la1)[3][4], const T (&la2)[3][4], T own1, T own2) {
    constexpr int X0 = NX == 5 ? -2 : 0, MID = NX / 2;
    T row[5][NX];
    pair_column_T<NX, VAR, 0>(la1, la2, row);
    pair_column_T<NX, VAR, 1>(la1, la2, row);
    pair_column_T<NX, VAR, 2>(la1, la2, row);
    if constexpr (NX == 5) {
        pair_column_T<NX, VAR, 3>(la1, la2, row);
        pair_column_T<NX, VAR, 4>(la1, la2, row);
    }
    const int wb = O.base(i, j);
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        T f[NX];
        line_T<NX>(row[b], f);
        if (b == 2) f[MID] += own1;
        if (b == 3) f[MID] += own2;
#pragma unroll
        for (int a = 0; a < NX; ++a) {
            const int x = X0 + a, y = b - 2;
            const int fam = (x & 1) ? ((y & 1) ? F_C : F_EH) : ((y & 1) ? F_EV : F_V);
            O.addb(win_plane(fam) + (VAR == 0 ? 3 : VAR), wb, (y - (y & 1)) / 2 * O_::kRX + (x - (x & 1)) / 2, f[a]);
        }
    }
}

// Transposed increments of one node: from the cotangents li of its increments and its
// block sums (velocities' share auv in units of p / Z, pressure's share ap), the adjoint la
// of the sums in units of p and those of the frozen c and Z.
template <class T>
AF_HD void node_adj(const T li[2][3], const T (&auv)[3][4], const T (&ap)[3][4], const Freeze<T>& z, T lam0, T lam1,
                    T (&la)[3][4], T& lc, T& lZ) {
    T a[3][4];
#pragma unroll
    for (int o = 0; o < 3; ++o)
#pragma unroll
        for (int m = 0; m < 4; ++m) a[o][m] = z.Z * auv[o][m] + ap[o][m];
    zero_acc(la);
    T liZ = T(0);
    lc = T(0);
    lZ = T(0);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const T lam = t ? lam1 : lam0, r = z.c * lam;
        // inc = (r / Z S_u, r / Z S_v, r S_pi), S_o = sum_m a[o][m] r^m; lq: adjoint of r S_o
        const T lq[3] = {li[t][2], li[t][0] * z.iZ, li[t][1] * z.iZ};
        T s[3], lr = T(0);
#pragma unroll
        for (int o = 0; o < 3; ++o) {
            s[o] = ((a[o][3] * r + a[o][2]) * r + a[o][1]) * r + a[o][0];
            const T ds = (T(3) * a[o][3] * r + T(2) * a[o][2]) * r + a[o][1];
            lr += lq[o] * (s[o] + r * ds);
            T w = lq[o] * r;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                la[o][m] += w;
                if (m < 3) w = w * r;
            }
        }
        lc += lam * lr;
        liZ += r * (li[t][0] * s[1] + li[t][1] * s[2]);
    }
    lZ = -z.iZ * z.iZ * liZ;
#pragma unroll
    for (int o = 0; o < 3; ++o)
#pragma unroll
        for (int m = 0; m < 4; ++m) lZ += la[o][m] * auv[o][m];
}

// Transposed increments of a pair of families at cell (i, j) (NX as in pair_blocks).  The
// lines and blocks are those of the forward operator transposed, so every node of the
// stencil gets one contribution per pair and variable: 128 scattered additions per cell
// for the two pairs, against 251 with one per wedge.  l1, l2: the cotangents of the two nodes'
// increments [duration][u, v, p]; a node whose six are all zero contributes nothing.
// sum: the point kernel's increment planes held u + du and v + dv, so the nodes' velocities get
// the cotangents of both durations besides (SCHEME 0).
template <int NX, class T, class A_, class O_>
AF_HD void incr_adj(const A_& A, const O_& O, int i, int j, const T (&l1)[2][3], const T (&l2)[2][3], bool sum, T gamma,
                    T lam0, T lam1) {
    constexpr int F1 = NX == 5 ? F_V : F_EH, F2 = NX == 5 ? F_EV : F_C;
    bool any1 = false, any2 = false;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            any1 = any1 || (l1[t][q] != T(0));
            any2 = any2 || (l2[t][q] != T(0));
        }
    if (!any1 && !any2) return;
    T u1[3][4], u2[3][4], p1[3][4], p2[3][4];
    zero_acc(u1);
    zero_acc(u2);
    pair_blocks<NX, true, true, 1>(A, i, j, u1, u2);
    stage_fence(u1, u2);
    pair_blocks<NX, true, true, 2>(A, i, j, u1, u2);
    stage_fence(u1, u2);
    zero_acc(p1);
    zero_acc(p2);
    pair_blocks<NX, true, true, 0>(A, i, j, p1, p2);
    stage_fence(p1, p2);
    const int wb = O.base(i, j);
    T la1[3][4], la2[3][4], Z1 = T(0), Z2 = T(0), own1 = T(0), own2 = T(0);
    zero_acc(la1);
    zero_acc(la2);
    // c = sqrt(gamma p / rho), Z = rho c: dc/drho = -c / (2 rho) = -c^2 / (2 Z),
    // dc/dp = c / (2 p) = gamma / (2 Z), dZ/drho = c / 2, dZ/dp = Z / (2 p) = gamma rho / (2 Z)
    const PolAbs<T> pol{gamma, T(0)};
    unsigned st = 0;
    auto reduce = [&](int fam, const T (&li)[2][3], const T (&auv)[3][4], const T (&ap)[3][4], T (&la)[3][4], T& Z, T& own) {
        const Prim<T> W = A.node(fam, i, j);
        const Freeze<T> z = freeze_node(W, pol, lam1, st);
        T lc, lZ;
        node_adj(li, auv, ap, z, lam0, lam1, la, lc, lZ);
        const T hiZ = T(0.5) * z.iZ;
        O.addb(win_plane(fam), wb, 0, lc * (-z.c * z.c * hiZ) + lZ * (T(0.5) * z.c));
        own = lc * (gamma * hiZ) + lZ * (gamma * W.r * hiZ);
        Z = z.Z;
    };
    if (any1) reduce(F1, l1, u1, p1, la1, Z1, own1);
    if (any2) reduce(F2, l2, u2, p2, la2, Z2, own2);
    stage_fence(la1, la2);
    pair_scatter<NX, 0>(O, i, j, la1, la2, own1, own2);
    scale_acc(la1, Z1);
    scale_acc(la2, Z2);
    stage_fence(la1, la2);
    pair_scatter<NX, 1>(O, i, j, la1, la2, sum ? l1[0][0] + l1[1][0] : T(0), sum ? l2[0][0] + l2[1][0] : T(0));
    stage_fence(la1, la2);
    pair_scatter<NX, 2>(O, i, j, la1, la2, sum ? l1[0][1] + l1[1][1] : T(0), sum ? l2[0][1] + l2[1][1] : T(0));
}

template <class T>
AF_HD void cons_T(const Prim<T>& w, T gamma, const T lU[4], T g[4]) {
    // U = (rho, rho u, rho v, p/(gamma-1) + rho (u^2+v^2)/2)
    const T q2 = T(0.5) * (w.u * w.u + w.v * w.v);
    g[0] = lU[0] + w.u * lU[1] + w.v * lU[2] + q2 * lU[3];
    g[1] = w.r * lU[1] + w.r * w.u * lU[3];
    g[2] = w.r * lU[2] + w.r * w.v * lU[3];
    g[3] = lU[3] / (gamma - T(1));
}

// Transposed centre recovery of cell (i, j) for the centre cotangent lW: the averages'
// cotangent (plane 16 + k of the window, weight 9/4) and the point values of the cell's
// eight boundary nodes (through U(W) at corners, weight -1/16, and edge midpoints, -1/4).
template <class T, class A_, class O_>
AF_HD void centre_adj(const A_& A, const O_& O, int i, int j, const T lW[4], T gamma) {
    const Prim<T> Wc = A.node(F_C, i, j);
    // W = prim(U_c): rho = U0, u = U1/U0, v = U2/U0, p = (g-1)(U3 - (U1 u + U2 v)/2)
    const T ir = T(1) / Wc.r, gm1 = gamma - T(1);
    T lU[4];
    lU[0] = lW[0] - lW[1] * Wc.u * ir - lW[2] * Wc.v * ir + lW[3] * gm1 * T(0.5) * (Wc.u * Wc.u + Wc.v * Wc.v);
    lU[1] = lW[1] * ir - lW[3] * gm1 * Wc.u;
    lU[2] = lW[2] * ir - lW[3] * gm1 * Wc.v;
    lU[3] = lW[3] * gm1;
    // U_c = 9/4 [Ubar - sum_corners U / 36 - sum_edges U / 9]
    const int wb = O.base(i, j);
#pragma unroll
    for (int k = 0; k < 4; ++k) O.addb(16 + k, wb, 0, T(2.25) * lU[k]);
    T lc[4], le[4], g[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) { lc[k] = -lU[k] * T(1.0 / 16.0); le[k] = -lU[k] * T(0.25); }
    cons_T(A.node(F_V, i, j), gamma, lc, g);          O.node(F_V, i, j, g);
    cons_T(A.node(F_V, i + 1, j), gamma, lc, g);      O.node(F_V, i + 1, j, g);
    cons_T(A.node(F_V, i, j + 1), gamma, lc, g);      O.node(F_V, i, j + 1, g);
    cons_T(A.node(F_V, i + 1, j + 1), gamma, lc, g);  O.node(F_V, i + 1, j + 1, g);
    cons_T(A.node(F_EH, i, j), gamma, le, g);         O.node(F_EH, i, j, g);
    cons_T(A.node(F_EH, i, j + 1), gamma, le, g);     O.node(F_EH, i, j + 1, g);
    cons_T(A.node(F_EV, i, j), gamma, le, g);         O.node(F_EV, i, j, g);
    cons_T(A.node(F_EV, i + 1, j), gamma, le, g);     O.node(F_EV, i + 1, j, g);
}

}  // namespace af
