// Device building blocks of the RB-TAI Active Flux step for gfx950 (FP64 and FP32).
//
// Every function here is a small, fully inlined piece of the algorithm of Sec. 6.1:
//   centre recovery from the conservative Simpson constraint (eq. center-node),
//   the node-centred exact acoustic operator in compact monomial-block form
//   (App. D, eq. compact-monomial-block), the Q2 evaluation used for the convective
//   foot and for the increment interpolant (Sec. 4, R_Delta), the transported point
//   update (Sec. 6.1 steps 3-4) and the Euler fluxes (Sec. 3).
// Data access goes through an accessor type (global planes or an LDS tile) so that
// the multi-kernel and the fused kernels share the arithmetic.
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

#include "af_blocks.h"
#include "af_internal.h"

// Helpers are host+device so that the operation-counting build (count_flops.cpp)
// can run the very same arithmetic on the host.
#ifndef AF_HD
#define AF_HD __host__ __device__ __forceinline__
#endif

namespace af {

// 1 / sqrt(x): the device's reciprocal square root (one hardware estimate and its
// refinement in FP64, the hardware instruction in FP32); the host builds that check
// indexing and count operations take the plain quotient.
AF_HD double rsqrt_of(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return rsqrt(x);
#else
    return 1.0 / sqrt(x);
#endif
}
AF_HD float rsqrt_of(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
    return rsqrtf(x);
#else
    return 1.0f / sqrtf(x);
#endif
}

// a / b: the correctly rounded quotient in FP64; in FP32 the product with the hardware
// reciprocal (within 1 ulp; a few instructions against the division's scaled iteration),
// whose rounding is far inside the FP32 form's stated error; the host builds divide.
AF_HD double quot(double a, double b) { return a / b; }
AF_HD float quot(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return a * __builtin_amdgcn_rcpf(b);
#else
    return a / b;
#endif
}

enum Fam { F_V = 0, F_EV = 1, F_EH = 2, F_C = 3 };

template <class T>
struct Prim { T r, u, v, p; };

// ---------------------------------------------------------------------------
// Conservative <-> primitive (Sec. 2)
// ---------------------------------------------------------------------------
template <class T>
AF_HD void cons_of(const Prim<T>& w, T gm1inv, T U[4]) {
    U[0] = w.r;
    U[1] = w.r * w.u;
    U[2] = w.r * w.v;
    U[3] = w.p * gm1inv + T(0.5) * w.r * (w.u * w.u + w.v * w.v);
}

// Recovered centre node (eq. center-node), written about the anchor U_a = U(V_ij)
// so that uniform data returns the anchor exactly (free-stream preservation):
//   U_c = U_a + 9/4 [ (Ubar - U_a) - sum_corners (U - U_a)/36 - sum_edges (U - U_a)/9 ].
template <class T>
AF_HD Prim<T> recover_centre(const T Ub[4], const Prim<T>& v00, const Prim<T>& v10,
                                                  const Prim<T>& v01, const Prim<T>& v11, const Prim<T>& eh0,
                                                  const Prim<T>& eh1, const Prim<T>& ev0, const Prim<T>& ev1,
                                                  T gamma) {
    const T gm1inv = T(1) / (gamma - T(1));
    T Ua[4], U[4], sc[4], se[4];
    cons_of(v00, gm1inv, Ua);
    cons_of(v10, gm1inv, U);
#pragma unroll
    for (int k = 0; k < 4; ++k) sc[k] = U[k] - Ua[k];
    cons_of(v01, gm1inv, U);
#pragma unroll
    for (int k = 0; k < 4; ++k) sc[k] += U[k] - Ua[k];
    cons_of(v11, gm1inv, U);
#pragma unroll
    for (int k = 0; k < 4; ++k) sc[k] += U[k] - Ua[k];
    cons_of(eh0, gm1inv, U);
#pragma unroll
    for (int k = 0; k < 4; ++k) se[k] = U[k] - Ua[k];
    cons_of(eh1, gm1inv, U);
#pragma unroll
    for (int k = 0; k < 4; ++k) se[k] += U[k] - Ua[k];
    cons_of(ev0, gm1inv, U);
#pragma unroll
    for (int k = 0; k < 4; ++k) se[k] += U[k] - Ua[k];
    cons_of(ev1, gm1inv, U);
#pragma unroll
    for (int k = 0; k < 4; ++k) se[k] += U[k] - Ua[k];
    T Uc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        Uc[k] = Ua[k] + T(2.25) * ((Ub[k] - Ua[k]) - sc[k] * T(1.0 / 36.0) - se[k] * T(1.0 / 9.0));
    Prim<T> w;
    w.r = Uc[0];
    T ir = T(1) / Uc[0];
    w.u = Uc[1] * ir;
    w.v = Uc[2] * ir;
    w.p = (gamma - T(1)) * (Uc[3] - T(0.5) * (Uc[1] * w.u + Uc[2] * w.v));
    return w;
}

// ---------------------------------------------------------------------------
// Exact node-centred acoustic operator (App. D)
// ---------------------------------------------------------------------------
// The compact monomial blocks in folded form.  The wedges of a node are mirror images of one
// another, and so are their blocks (a factor -1 per odd power and per odd channel), so
// the sum over them needs the data only in even and odd parts: along a line of five
// nodes f at X = -1, -1/2, 0, 1/2, 1 about the node the monomial coefficients in |X| of
// f(X) + f(-X) and f(X) - f(-X), along a line of three nodes at X = -1/2, 0, 1/2 (one
// cell) the coefficients in X.  Each block entry is then applied once per node instead of
// once per wedge, and lines along x are shared by the nodes above one another.
// Coefficients are stored without a factor 2 that the block constants take (LineTerm).
struct LineTerm { int pow; bool odd; double scale; };
template <int N> struct LineTerms;
template <> struct LineTerms<5> {
    static constexpr LineTerm t[5] = {{0, false, 2.0}, {1, false, 1.0}, {2, false, 2.0}, {1, true, 1.0}, {2, true, 2.0}};
};
template <> struct LineTerms<3> {
    static constexpr LineTerm t[3] = {{0, false, 1.0}, {1, true, 1.0}, {2, false, 2.0}};
};

// Line transform, in differences so that constants give exact zeros.  DIFF: differences
// from the middle node first (node values); otherwise fewer operations (for values that
// are differences along the other direction already).
template <int N, bool DIFF, class T>
AF_HD void line(const T* f, T* c) {
    if constexpr (N == 5) {
        T e1, e2;
        const T o1 = f[3] - f[1], o2 = f[4] - f[0];
        if constexpr (DIFF) {
            e1 = (f[3] - f[2]) + (f[1] - f[2]);
            e2 = (f[4] - f[2]) + (f[0] - f[2]);
        } else {
            e1 = (f[3] + f[1]) - T(2) * f[2];
            e2 = (f[4] + f[0]) - T(2) * f[2];
        }
        c[0] = f[2];
        c[1] = T(4) * e1 - e2;
        c[2] = e2 - T(2) * e1;
        c[3] = T(4) * o1 - o2;
        c[4] = o2 - T(2) * o1;
    } else {
        c[0] = f[1];
        c[1] = f[2] - f[0];
        c[2] = (f[2] - f[1]) + (f[0] - f[1]);
    }
}

// acc[out][m] += the r^(m+1) coefficient of channel out (0: pi, 1: u, 2: v) from the
// coefficients c along y of variable VAR's (0: pi, 1: u, 2: v) coefficient A along x; W:
// the node's wedge with X, Y > 0.
template <int W, int NX, int NY, int VAR, int A, int B, int OUT, class T>
AF_HD void block_term(const T (&c)[NY], T (&acc)[3][4]) {
    constexpr LineTerm x = LineTerms<NX>::t[A], y = LineTerms<NY>::t[B];
    // odd in x where exactly one of the two is u, odd in y where one is v
    constexpr bool match = x.odd == ((OUT == 1) != (VAR == 1)) && y.odd == ((OUT == 2) != (VAR == 2));
    if constexpr (match && x.pow + y.pow > 0) {
        constexpr double w = kBlk[W][x.pow][y.pow][3 * OUT + VAR] * x.scale * y.scale;
        if constexpr (w != 0.0) acc[OUT][x.pow + y.pow - 1] += T(w) * c[B];
    }
}

template <int W, int NX, int NY, int VAR, int A, class T, int... K>
AF_HD void block_terms(const T (&c)[NY], T (&acc)[3][4], std::integer_sequence<int, K...>) {
    (block_term<W, NX, NY, VAR, A, K / 3, K % 3>(c, acc), ...);
}

template <int W, int NX, int NY, int VAR, int A, class T>
AF_HD void block_acc(const T (&c)[NY], T (&acc)[3][4]) {
    block_terms<W, NX, NY, VAR, A>(c, acc, std::make_integer_sequence<int, 3 * NY>());
}

template <class T>
AF_HD void zero_acc(T (&acc)[3][4]) {
#pragma unroll
    for (int o = 0; o < 3; ++o)
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[o][m] = T(0);
}

template <class T>
AF_HD void scale_acc(T (&acc)[3][4], T s) {
#pragma unroll
    for (int o = 0; o < 3; ++o)
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[o][m] = acc[o][m] * s;
}

// Increments (du, dv, dp) at radius r from the sums (channels in units of p).
template <class T>
AF_HD void block_increment(const T a[3][4], T r, T iZ, T inc[3]) {
    T s[3];
#pragma unroll
    for (int o = 0; o < 3; ++o) s[o] = ((a[o][3] * r + a[o][2]) * r + a[o][1]) * r + a[o][0];
    inc[0] = (r * iZ) * s[1];
    inc[1] = (r * iZ) * s[2];
    inc[2] = r * s[0];
}

// ---------------------------------------------------------------------------
// Q2 evaluation and the transported point update
// ---------------------------------------------------------------------------
// Lagrange weights at -1 and +1 (the middle one is implied by the difference form).
template <class T>
AF_HD void lag_pm(T s, T& lm, T& lp) {
    T hs = T(0.5) * s;
    lm = hs * (s - T(1));
    lp = hs * (s + T(1));
}

// sum_a l_a f_a written as f_1 + l_-(f_0 - f_1) + l_+(f_2 - f_1): exact on constants.
template <class T>
AF_HD T q1(T lm, T lp, T f0, T f1, T f2) {
    return f1 + lm * (f0 - f1) + lp * (f2 - f1);
}

template <class T>
AF_HD T q2(T xm, T xp, T ym, T yp, const T f[3][3]) {
    T g0 = q1(xm, xp, f[0][0], f[1][0], f[2][0]);
    T g1 = q1(xm, xp, f[0][1], f[1][1], f[2][1]);
    T g2 = q1(xm, xp, f[0][2], f[1][2], f[2][2]);
    return q1(ym, yp, g0, g1, g2);
}

// FP32: the tensor weights lx[a] ly[b] (lx = (xm, 1 - xm - xp, xp)) times the nodal values,
// nine products whose weights every evaluation at the same point shares (the compiler
// forms them once), against sixteen operations per evaluation in the difference form.
// The FP32 form's values are perturbations about a uniform background, which stays exact
// (a zero perturbation stays zero); the FP64 path keeps the difference form, exact on
// constants.
template <>
AF_HD float q2<float>(float xm, float xp, float ym, float yp, const float f[3][3]) {
    const float lx[3] = {xm, 1.0f - xm - xp, xp}, ly[3] = {ym, 1.0f - ym - yp, yp};
    float s = 0.0f;
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a) s += (lx[a] * ly[b]) * f[a][b];
    return s;
}

template <class T>
AF_HD void flux_x(const Prim<T>& w, T gm1inv, T F[4]) {
    T E = w.p * gm1inv + T(0.5) * w.r * (w.u * w.u + w.v * w.v);
    T m = w.r * w.u;
    F[0] = m;
    F[1] = m * w.u + w.p;
    F[2] = m * w.v;
    F[3] = w.u * (E + w.p);
}

template <class T>
AF_HD void flux_y(const Prim<T>& w, T gm1inv, T F[4]) {
    T E = w.p * gm1inv + T(0.5) * w.r * (w.u * w.u + w.v * w.v);
    T m = w.r * w.v;
    F[0] = m;
    F[1] = m * w.u;
    F[2] = m * w.v + w.p;
    F[3] = w.v * (E + w.p);
}

// ---------------------------------------------------------------------------
// Variable policies.  PolAbs: the state holds the physical values (FP64 path).
// PolPert: the state holds perturbations about a uniform background W_bg and
// U(W_bg) (FP32 path); every conversion and flux below is the exact difference
// F(W_bg + W') - F(W_bg), so no large background value is ever rounded away.
// The increments of the acoustic operator and the Q2 evaluations are linear in
// the data and shift-invariant, so they act on perturbations unchanged.
// ---------------------------------------------------------------------------
template <class T>
struct PolAbs {
    T gamma, gm1inv;
    AF_HD T rho(T r) const { return r; }
    AF_HD T vu(T u) const { return u; }
    AF_HD T vv(T v) const { return v; }
    AF_HD T pr(T p) const { return p; }
    AF_HD Prim<T> centre(const T Ub[4], const Prim<T>& v00, const Prim<T>& v10, const Prim<T>& v01,
                         const Prim<T>& v11, const Prim<T>& eh0, const Prim<T>& eh1, const Prim<T>& ev0,
                         const Prim<T>& ev1) const {
        return recover_centre(Ub, v00, v10, v01, v11, eh0, eh1, ev0, ev1, gamma);
    }
    AF_HD void fx(const Prim<T>& w, T F[4]) const { flux_x(w, gm1inv, F); }
    AF_HD void fy(const Prim<T>& w, T F[4]) const { flux_y(w, gm1inv, F); }
};

template <class T>
struct PolPert {
    T gamma, gm1inv, r0, u0, v0, p0;
    T m0x, m0y, H0;    // background momentum and total enthalpy density E + p
    AF_HD T rho(T r) const { return r0 + r; }
    AF_HD T vu(T u) const { return u0 + u; }
    AF_HD T vv(T v) const { return v0 + v; }
    AF_HD T pr(T p) const { return p0 + p; }
    // E(W) - E(W_bg) from a perturbation
    AF_HD T energy(const Prim<T>& w) const {
        const T uu = u0 + w.u, vv = v0 + w.v;
        return w.p * gm1inv +
               T(0.5) * (w.r * (uu * uu + vv * vv) + r0 * (w.u * (T(2) * u0 + w.u) + w.v * (T(2) * v0 + w.v)));
    }
    AF_HD void cons(const Prim<T>& w, T U[4]) const {
        U[0] = w.r;
        U[1] = r0 * w.u + w.r * (u0 + w.u);
        U[2] = r0 * w.v + w.r * (v0 + w.v);
        U[3] = energy(w);
    }
    AF_HD Prim<T> centre(const T Ub[4], const Prim<T>& v00, const Prim<T>& v10, const Prim<T>& v01,
                         const Prim<T>& v11, const Prim<T>& eh0, const Prim<T>& eh1, const Prim<T>& ev0,
                         const Prim<T>& ev1) const {
        T Ua[4], U[4], sc[4], se[4];
        cons(v00, Ua);
        const Prim<T>* corners[3] = {&v10, &v01, &v11};
        const Prim<T>* edges[4] = {&eh0, &eh1, &ev0, &ev1};
#pragma unroll
        for (int k = 0; k < 4; ++k) { sc[k] = T(0); se[k] = T(0); }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            cons(*corners[c], U);
#pragma unroll
            for (int k = 0; k < 4; ++k) sc[k] += U[k] - Ua[k];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            cons(*edges[c], U);
#pragma unroll
            for (int k = 0; k < 4; ++k) se[k] += U[k] - Ua[k];
        }
        T Uc[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            Uc[k] = Ua[k] + T(2.25) * ((Ub[k] - Ua[k]) - sc[k] * T(1.0 / 36.0) - se[k] * T(1.0 / 9.0));
        Prim<T> w;
        w.r = Uc[0];
        const T ir = quot(T(1), r0 + Uc[0]);
        w.u = (Uc[1] - u0 * Uc[0]) * ir;
        w.v = (Uc[2] - v0 * Uc[0]) * ir;
        const T uu = u0 + w.u, vv = v0 + w.v;
        w.p = (gamma - T(1)) *
              (Uc[3] - T(0.5) * (w.r * (uu * uu + vv * vv) + r0 * (w.u * (T(2) * u0 + w.u) + w.v * (T(2) * v0 + w.v))));
        return w;
    }
    AF_HD void fx(const Prim<T>& w, T F[4]) const {
        const T uu = u0 + w.u, vv = v0 + w.v;
        const T m = r0 * w.u + w.r * uu;                 // rho u - rho0 u0
        const T Hp = energy(w) + w.p;                    // H - H0
        F[0] = m;
        F[1] = m0x * w.u + m * uu + w.p;
        F[2] = m0x * w.v + m * vv;
        F[3] = u0 * Hp + w.u * (H0 + Hp);
    }
    AF_HD void fy(const Prim<T>& w, T F[4]) const {
        const T uu = u0 + w.u, vv = v0 + w.v;
        const T m = r0 * w.v + w.r * vv;                 // rho v - rho0 v0
        const T Hp = energy(w) + w.p;
        F[0] = m;
        F[1] = m0y * w.u + m * uu;
        F[2] = m0y * w.v + m * vv + w.p;
        F[3] = v0 * Hp + w.v * (H0 + Hp);
    }
};

}  // namespace af
