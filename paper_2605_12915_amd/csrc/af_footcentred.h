// Foot-centred exact frozen-acoustic point update (App. C; Sec. 4, the paragraph on an
// exact frozen acoustic update), FP64, for the multi-kernel path (af_f64.hip); host and
// device code, so that a host build can check it against the oracle (tests/fc_host.cpp).
//
// For a target P and a duration tau: the convective foot F by the two Picard stages of
// the transported update (eq. adv-footpoint), the frozen state W* = W_h^n(F) of the
// cellwise Q2 reconstruction, c* = sqrt(gamma p* / rho*), Z* = rho* c*, and the disk
// of radius R = c* tau / h (cell units) about F, which must stay inside the half-cell
// footprint |F - P| + R < 1/2 in each direction (eq. fc-half-footprint).  With pi = p / Z*
// the exact solution of the frozen acoustic system at F after tau is written with
// spherical means M_r[f] = (1 / 2 pi) int_{|z| < 1} f(F + r z) (1 - |z|^2)^(-1/2) dz of
// the continuous piecewise-Q2 data:
//   pi(F) = M_R[pi_0] + R M_R[z . grad pi_0] - R M_R[g],        g = div u_0,
//   u(F)  = u_0(F) - R M_R[grad pi_0] + int_0^R r M_r[grad g] dr.
// The last integral (grad g distributional: g jumps across grid lines) equals, after
// exchanging the integration order and integrating by parts over the disk's pieces,
// (R / 2 pi) int_0^{2 pi} e_theta int_0^{pi/2} g(F + R sin(psi) e_theta) dpsi dtheta:
// one more sum over the nodes of M_R.  Density from the transported update's linear
// closure rho* + (p - p*) / c*^2.
//
// Quadrature: polar coordinates about F with |z| = sin(psi) (absorbing the weight), the
// angle split at multiples of pi/4, where a grid line touches the circle (with cuts
// graded towards the tangency) and where a ray passes through a grid corner, and each
// ray's psi range split where it crosses a grid line, so that every piece lies in one
// cell; 32 Gauss points per angular piece, clustered towards both ends by
// theta = t0 + (t1 - t0)(1 - cos(pi s)) / 2 (square-root behaviour at a tangency).  Along a
// ray's piece the integrands are polynomials in |z| (the Q2 data of one cell), so the
// radial integrals are exact sums of the moments of sin(psi)^k.  The footprint keeps the
// disk inside the 2 x 2 cells around P, so at most one vertical and one horizontal grid line
// cut it.
//
// On the device one half-wavefront takes a target and duration (fc_point_group): a lane
// computes one of the (at most 25) cuts, which are sorted across the lanes, loads one of the
// 25 lattice nodes, and is one of the 32 angular nodes of every piece.  The host build runs
// the same pieces and nodes one after the other.
#pragma once
#include <hip/hip_runtime.h>

#include "af_gauss.h"
#include "af_internal.h"
#include "af_kernels.h"

namespace af {

constexpr double kFcPi = 3.14159265358979323846;

// Polynomials of one cell about the foot in the unit disk's coordinates z (offsets divided
// by R), from the nodal values minus the frozen state: p[a][b] of z_x^a z_y^b, and R times
// the divergence g = du/dx + dv/dy, whose coefficients combine along a ray with
// (c, s) = (cos, sin): g0, g1c c + g1s s, g2cc c^2 + g2cs c s + g2ss s^2, g3css c s^2 + g3ccs c^2 s.
struct FcPoly { double p[3][3], g0, g1c, g1s, g2cc, g2cs, g2ss, g3css, g3ccs; };

// Sums over the disk, from which the point value follows: m = M_R[p - p*] + R M_R[z . grad p],
// and R times M_R[g], M_R[grad p] and the history term (1 / 2 pi) int int g e_theta dpsi dtheta.
struct FcSums { double m, g, x, y, hx, hy; };

// Coefficients of z^k of the quadratic through f at 0, 1/2, 1, about x, scaled by R.
AF_HD void fc_shift(double f0, double f1, double f2, double x, double R, double c[3]) {
    const double d1 = f1 - f0, d2 = f2 - f0, a = 4.0 * d1 - d2, b = 2.0 * d2 - 4.0 * d1;
    c[0] = f0 + x * (a + b * x);
    c[1] = R * (a + 2.0 * b * x);
    c[2] = R * R * b;
}

// n(var, a, b): nodal value (0: p, 1: u, 2: v) [x-node][y-node] of the cell whose lower left
// corner is (x0, y0) from the foot.
template <class N>
AF_HD void fc_poly(const N& n, double x0, double y0, double R, FcPoly& c) {
    double k[3][3][3];
#pragma unroll
    for (int v = 0; v < 3; ++v) {
        double row[3][3];
#pragma unroll
        for (int b = 0; b < 3; ++b) fc_shift(n(v, 0, b), n(v, 1, b), n(v, 2, b), -x0, R, row[b]);
#pragma unroll
        for (int a = 0; a < 3; ++a) fc_shift(row[0][a], row[1][a], row[2][a], -y0, R, k[v][a]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) c.p[a][b] = k[0][a][b];
    const double(&u)[3][3] = k[1];
    const double(&w)[3][3] = k[2];
    c.g0 = u[1][0] + w[0][1];
    c.g1c = 2.0 * u[2][0] + w[1][1];
    c.g1s = u[1][1] + 2.0 * w[0][2];
    c.g2cc = w[2][1];
    c.g2cs = 2.0 * (u[2][1] + w[1][2]);
    c.g2ss = u[1][2];
    c.g3css = 2.0 * u[2][2];
    c.g3ccs = 2.0 * w[2][2];
}

// The disk about the foot (X, Y) (relative to the target's cell, cell units) of radius R,
// 0 < R, |X - ox| + R < 1/2, |Y - oy| + R < 1/2, and the grid lines that cut it: at most one
// in each direction, at lam, mu (units of R).
struct FcDisk {
    double X, Y, R, lam, mu;
    int kx, ky;
    bool hx, hy;
};

AF_HD FcDisk fc_disk_of(double X, double Y, double R) {
    FcDisk d;
    d.X = X; d.Y = Y; d.R = R;
    d.kx = (int)floor(X + R);
    d.ky = (int)floor(Y + R);
    d.hx = (double)d.kx > X - R && (double)d.kx < X + R;
    d.hy = (double)d.ky > Y - R && (double)d.ky < Y + R;
    d.lam = d.hx ? ((double)d.kx - X) / R : 0.0;
    d.mu = d.hy ? ((double)d.ky - Y) / R : 0.0;
    return d;
}

constexpr int kFcCuts = 25;   // candidates for a cut of the angle, fc_cut(d, 0 .. kFcCuts - 1)

// Candidate q for a cut, in [0, 2 pi]; 2 pi where there is none.
AF_HD double fc_cut(const FcDisk& d, int q) {
    constexpr double full = 2.0 * kFcPi;
    double c = full;
    if (q < 8) return q * (0.25 * kFcPi);
    if (q < 24) {
        // tangencies of the vertical (8 .. 15) and the horizontal line (16 .. 23): the two
        // angles, then cuts graded towards them
        const bool vert = q < 16;
        const double l = vert ? d.lam : d.mu;
        if (!(vert ? d.hx : d.hy)) return full;
        const double base = (vert ? 0.0 : 0.5 * kFcPi) + (l > 0.0 ? 0.0 : kFcPi), a = acos(fmin(1.0, fabs(l)));
        const int g = (q & 7) >> 1;
        const double gr = g == 0 ? 0.0 : (g == 1 ? 0.25 : (g == 2 ? 1.0 : 4.0)), t = gr * fabs(l);
        if (g > 0 && !(t < a)) return full;
        c = (q & 1) ? base + a - t : base - a + t;
    } else {
        if (!(d.hx && d.hy)) return full;
        const double dx = (double)d.kx - d.X, dy = (double)d.ky - d.Y;
        if (!(dx * dx + dy * dy < d.R * d.R)) return full;
        c = atan2(dy, dx);
    }
    if (c < 0.0) c += full;
    if (c >= full) c -= full;
    return c;
}

// cos and sin of tm + d for |d| <= pi/8 + rounding, from those of tm: the Taylor series of
// cos d - 1 and sin d (terms left out below 1e-17 at 0.4) and the addition theorem.
AF_HD void fc_turn(double cm, double sm, double d, double& c, double& s) {
    const double x = d * d;
    double sd = -1.0 / 1307674368000.0;                 // -1/15!
    sd = fma(sd, x, 1.0 / 6227020800.0);
    sd = fma(sd, x, -1.0 / 39916800.0);
    sd = fma(sd, x, 1.0 / 362880.0);
    sd = fma(sd, x, -1.0 / 5040.0);
    sd = fma(sd, x, 1.0 / 120.0);
    sd = fma(sd, x, -1.0 / 6.0);
    sd = fma(sd * x, d, d);
    double cd = 1.0 / 20922789888000.0;                 // 1/16!
    cd = fma(cd, x, -1.0 / 87178291200.0);
    cd = fma(cd, x, 1.0 / 479001600.0);
    cd = fma(cd, x, -1.0 / 3628800.0);
    cd = fma(cd, x, 1.0 / 40320.0);
    cd = fma(cd, x, -1.0 / 720.0);
    cd = fma(cd, x, 1.0 / 24.0);
    cd = fma(cd, x, -0.5) * x;                          // cos d - 1
    c = cm + (cm * cd - sm * sd);
    s = sm + (sm * cd + cm * sd);
}

// cos and sin of an angle in [0, 2 pi], turned from the nearest multiple of pi/4.
AF_HD void fc_angle(double t, double& c, double& s) {
    constexpr double h = 0.70710678118654752440, lo = 3.061616997868383e-17;   // pi/4 - (double)(pi/4)
    const double m = floor(t * (4.0 / kFcPi) + 0.5);
    const int q = (int)m & 7, r = q & 3;
    const double a = r == 0 ? 1.0 : (r == 2 ? 0.0 : (r == 1 ? h : -h)), b = r == 0 ? 0.0 : (r == 2 ? 1.0 : h);
    fc_turn(q < 4 ? a : -a, q < 4 ? b : -b, fma(-m, 0.25 * kFcPi, t) - m * lo, c, s);
}

// One angular piece [t0, t0 + dt]: cos and sin of its middle, and a code of the lines that its
// rays cross in the order of increasing radius (the same for every ray of the piece): bits
// 0-1 their number, bit 2 set if the horizontal line comes first, bits 4-5, 6-7 and 8-9 the cells
// of the radial pieces as indices into the 2 x 2 cells around (kx, ky), 2 (upper row) +
// (right column).
struct FcPiece { double dt, cm, sm; int code; };

AF_HD FcPiece fc_piece(const FcDisk& d, double t0, double t1) {
    FcPiece w;
    w.dt = t1 - t0;
    const double tm = 0.5 * (t0 + t1);
    fc_angle(tm, w.cm, w.sm);
    const double qx = d.lam / w.cm, qy = d.mu / w.sm;
    const bool cx = d.hx && qx > 0.0 && qx < 1.0, cy = d.hy && qy > 0.0 && qy < 1.0;
    const int n = (cx ? 1 : 0) + (cy ? 1 : 0);
    const bool yfirst = cy && (!cx || qy < qx);
    const double q0 = n == 0 ? 1.0 : (yfirst ? qy : qx), q1 = n < 2 ? 1.0 : (yfirst ? qx : qy);
    const double q[4] = {0.0, q0, q1, 1.0};
    w.code = n + (yfirst ? 4 : 0);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        // the middle (in radius) of the radial piece on the middle ray
        const double r = 0.5 * (q[s] + q[s + 1]);
        const int ix = (int)floor(d.X + d.R * r * w.cm) - (d.kx - 1), iy = (int)floor(d.Y + d.R * r * w.sm) - (d.ky - 1);
        w.code += (2 * (iy > 0 ? 1 : 0) + (ix > 0 ? 1 : 0)) << (4 + 2 * s);
    }
    return w;
}

// Antiderivatives at psi (s = sin psi, c = cos psi) of sin^k, k = 0 .. 5.
struct FcMom { double v[6]; };

AF_HD FcMom fc_moments(double psi, double s, double c) {
    FcMom m;
    m.v[0] = psi;
    m.v[1] = -c;
    double e = s;
#pragma unroll
    for (int k = 2; k < 6; ++k) {
        m.v[k] = ((k - 1) * m.v[k - 2] - e * c) * (1.0 / k);
        e *= s;
    }
    return m;
}

// The radial piece between the moments lo and hi on the ray (c, s), weight w, in one cell.
AF_HD void fc_ray(const FcPoly& P, double c, double s, double w, const FcMom& lo, const FcMom& hi, FcSums& S) {
    double I[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) I[k] = w * (hi.v[k] - lo.v[k]);
    const double cc = c * c, cs = c * s, ss = s * s;
    // R grad p along the ray by powers of |z|, and R g
    const double x[4] = {P.p[1][0], 2.0 * P.p[2][0] * c + P.p[1][1] * s, 2.0 * P.p[2][1] * cs + P.p[1][2] * ss,
                         2.0 * P.p[2][2] * c * ss};
    const double y[4] = {P.p[0][1], P.p[1][1] * c + 2.0 * P.p[0][2] * s, P.p[2][1] * cc + 2.0 * P.p[1][2] * cs,
                         2.0 * P.p[2][2] * cc * s};
    const double g[4] = {P.g0, P.g1c * c + P.g1s * s, P.g2cc * cc + P.g2cs * cs + P.g2ss * ss,
                         P.g3css * c * ss + P.g3ccs * cc * s};
    double m = P.p[0][0] * I[1], gm = 0.0, xm = 0.0, ym = 0.0, hm = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // p's coefficient of |z|^(k+1) is (c x_k + s y_k) / (k + 1); z . grad p has k + 1 times it
        m += (c * x[k] + s * y[k]) * ((1.0 + 1.0 / (k + 1)) * I[k + 2]);
        gm += g[k] * I[k + 1];
        xm += x[k] * I[k + 1];
        ym += y[k] * I[k + 1];
        hm += g[k] * I[k];
    }
    S.m += m;
    S.g += gm;
    S.x += xm;
    S.y += ym;
    S.hx += hm * c;
    S.hy += hm * s;
}

// Angular node (position xc = cos(pi x), weight wt = w pi sin(pi x) / 2 of the clustered rule)
// of a piece: every radial piece of its ray.  poly(cell): the cell's polynomials.
template <class P>
AF_HD void fc_node(const FcDisk& d, const FcPiece& w, double xc, double wt, const P& poly, FcSums& S) {
    double c, s;
    fc_turn(w.cm, w.sm, -0.5 * w.dt * xc, c, s);
    const double wk = wt * w.dt * (1.0 / (2.0 * kFcPi));
    const int n = w.code & 3;
    FcMom lo = fc_moments(0.0, 0.0, 1.0);
#pragma unroll 1
    for (int q = 0; q <= n; ++q) {
        double psi = 0.5 * kFcPi, sp = 1.0, cp = 0.0;   // the ray's end
        if (q < n) {
            const bool horizontal = ((w.code >> 2) & 1) != q;
            sp = fmin(1.0, fmax(0.0, (horizontal ? d.mu : d.lam) / (horizontal ? s : c)));
            psi = asin(sp);
            cp = sqrt((1.0 - sp) * (1.0 + sp));
        }
        const FcMom hi = fc_moments(psi, sp, cp);
        fc_ray(poly((w.code >> (4 + 2 * q)) & 3), c, s, wk, lo, hi, S);
        lo = hi;
    }
}

// What precedes the disk: foot, frozen state, radius and the footprint check.  Returns false
// where the value is ws as it stands.
template <class A>
AF_HD bool fc_foot(const A& acc, int fam, int i, int j, double gamma, double lam, unsigned& st, Prim<double>& ws,
                   double& c2, FcDisk& d) {
    const PolAbs<double> pol{gamma, 1.0 / (gamma - 1.0)};
    const Prim<double> WP = acc.node(fam, i, j);
    int ci, cj;
    double xi, eta, xm, xp, ym, yp;
    picard_foot(acc, fam, i, j, pol, lam, WP, ci, cj, xi, eta, st);
    lag_pm(xi, xm, xp);
    lag_pm(eta, ym, yp);
    double f[3][3];
    cell_field<3>(acc, ci, cj, f);
    ws.r = q2(xm, xp, ym, yp, f);
    cell_field<1>(acc, ci, cj, f);
    ws.u = q2(xm, xp, ym, yp, f);
    cell_field<2>(acc, ci, cj, f);
    ws.v = q2(xm, xp, ym, yp, f);
    cell_field<0>(acc, ci, cj, f);
    ws.p = q2(xm, xp, ym, yp, f);
    if (!(ws.r > 0.0) || !(ws.p > 0.0)) {
        st |= SB_NONPHYS;
        return false;
    }
    c2 = gamma * ws.p / ws.r;
    const double R = sqrt(c2) * lam;
    // foot relative to the target's cell, and its displacement from the target
    const double Xf = (double)(ci - i) + 0.5 * (xi + 1.0), Yf = (double)(cj - j) + 0.5 * (eta + 1.0);
    const double dx = Xf - fam_ox<double>(fam), dy = Yf - fam_oy<double>(fam);
    if (!(fabs(dx) + R < 0.5) || !(fabs(dy) + R < 0.5)) {
        st |= SB_FOOTPRINT;
        return false;
    }
    if (!(R > 0.0)) return false;
    d = fc_disk_of(Xf, Yf, R);
    return true;
}

AF_HD Prim<double> fc_value(const Prim<double>& ws, double c2, const FcSums& S) {
    const double Z = ws.r * sqrt(c2);
    const double p = ws.p + S.m - Z * S.g;
    return Prim<double>{ws.r + (p - ws.p) / c2, ws.u - S.x / Z + S.hx, ws.v - S.y / Z + S.hy, p};
}

// Lattice node n (0 .. 24) of the 2 x 2 cells around (kx, ky): half cells (n % 5, n / 5) from the
// vertex of cell (kx - 1, ky - 1).
template <class A>
AF_HD Prim<double> fc_lattice(const A& acc, const FcDisk& d, int i, int j, int n) {
    const int a = n % 5, b = n / 5;
    const int fam = (a & 1) ? ((b & 1) ? F_C : F_EH) : ((b & 1) ? F_EV : F_V);
    return acc.node(fam, i + d.kx - 1 + a / 2, j + d.ky - 1 + b / 2);
}

// Polynomials of cell q (0 .. 3) of the 2 x 2, from the lattice's values nd[3][25] (p, u, v) minus
// the frozen state.
AF_HD void fc_cell_poly(const FcDisk& d, const double* nd, int q, FcPoly& P) {
    const int cx = q & 1, cy = q >> 1;
    fc_poly([&](int v, int a, int b) { return nd[v * 25 + (2 * cy + b) * 5 + 2 * cx + a]; }, (double)(d.kx - 1 + cx) - d.X,
            (double)(d.ky - 1 + cy) - d.Y, d.R, P);
}

// New point value of the target of family fam at (i, j) after tau = lam h, one piece and
// node after the other (host build).
template <class A>
AF_HD Prim<double> fc_point_update(const A& acc, int fam, int i, int j, double gamma, double lam, unsigned& st) {
    Prim<double> ws;
    double c2;
    FcDisk d;
    if (!fc_foot(acc, fam, i, j, gamma, lam, st, ws, c2, d)) return ws;
    double nd[75];
    for (int n = 0; n < 25; ++n) {
        const Prim<double> w = fc_lattice(acc, d, i, j, n);
        nd[n] = w.p - ws.p;
        nd[25 + n] = w.u - ws.u;
        nd[50 + n] = w.v - ws.v;
    }
    FcPoly P[4];
    for (int q = 0; q < 4; ++q) fc_cell_poly(d, nd, q, P[q]);
    double cut[kFcCuts + 1];
    for (int q = 0; q < kFcCuts; ++q) {
        const double c = fc_cut(d, q);
        int k = q;
        for (; k > 0 && cut[k - 1] > c; --k) cut[k] = cut[k - 1];
        cut[k] = c;
    }
    cut[kFcCuts] = 2.0 * kFcPi;
    FcSums S{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int q = 0; q < kFcCuts; ++q) {
        if (cut[q + 1] - cut[q] < 1e-15) continue;
        const FcPiece w = fc_piece(d, cut[q], cut[q + 1]);
        for (int k = 0; k < 32; ++k)
            fc_node(d, w, kGaussCos32[k], 0.5 * kFcPi * kGaussW32[k] * kGaussSin32[k],
                    [&](int c) -> const FcPoly& { return P[c]; }, S);
    }
    return fc_value(ws, c2, S);
}

#if defined(__HIPCC__)
// The same by one half-wavefront: lane = threadIdx.x & 31 of 32 lanes that agree on the
// target; sh: LDS of this group.  The value is valid in every lane.
struct FcShared { double nd[75]; FcPoly P[4]; };

template <class A>
__device__ __forceinline__ Prim<double> fc_point_group(const A& acc, int fam, int i, int j, double gamma, double lam,
                                                       unsigned& st, FcShared& sh, int lane) {
    Prim<double> ws;
    double c2;
    FcDisk d;
    if (!fc_foot(acc, fam, i, j, gamma, lam, st, ws, c2, d)) return ws;
    if (lane < 25) {
        const Prim<double> w = fc_lattice(acc, d, i, j, lane);
        sh.nd[lane] = w.p - ws.p;
        sh.nd[25 + lane] = w.u - ws.u;
        sh.nd[50 + lane] = w.v - ws.v;
    }
    __builtin_amdgcn_wave_barrier();
    __threadfence_block();
    if (lane < 4) fc_cell_poly(d, sh.nd, lane, sh.P[lane]);
    __builtin_amdgcn_wave_barrier();
    __threadfence_block();
    // bitonic sort of the cuts across the group
    double cut = lane < kFcCuts ? fc_cut(d, lane) : 2.0 * kFcPi;
#pragma unroll
    for (int k = 2; k <= 32; k *= 2)
#pragma unroll
        for (int m = k / 2; m > 0; m /= 2) {
            const double o = __shfl_xor(cut, m, 32);
            const bool up = (lane & k) == 0, low = (lane & m) == 0;
            cut = up == low ? fmin(cut, o) : fmax(cut, o);
        }
    const double xc = kGaussCos32[lane], wt = 0.5 * kFcPi * kGaussW32[lane] * kGaussSin32[lane];
    // lane q prepares piece q (cut[25 ..] = 2 pi: empty pieces)
    const double next = __shfl_down(cut, 1, 32);
    const FcPiece mine = fc_piece(d, cut, lane < 31 ? next : 2.0 * kFcPi);
    FcSums S{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int q = 0; q < kFcCuts; ++q) {
        const FcPiece w{__shfl(mine.dt, q, 32), __shfl(mine.cm, q, 32), __shfl(mine.sm, q, 32), __shfl(mine.code, q, 32)};
        if (w.dt < 1e-15) continue;
        fc_node(d, w, xc, wt, [&](int c) -> const FcPoly& { return sh.P[c]; }, S);
    }
#pragma unroll
    for (int m = 16; m > 0; m /= 2) {
        S.m += __shfl_xor(S.m, m, 32);
        S.g += __shfl_xor(S.g, m, 32);
        S.x += __shfl_xor(S.x, m, 32);
        S.y += __shfl_xor(S.y, m, 32);
        S.hx += __shfl_xor(S.hx, m, 32);
        S.hy += __shfl_xor(S.hy, m, 32);
    }
    return fc_value(ws, c2, S);
}
#endif

}  // namespace af
