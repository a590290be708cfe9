// Host walk of the adjoint kernels' arithmetic (af_adjoint.h) over one block's items: every target
// of an 8 x 8 point block, both passes, and every pair and centre of a 16 x 8 increments block, on
// random states whose velocities reach 1.5 cells a step.  Every read of the staged state and
// every addition must lie in the block's window ([-1, B + 2) and [-2, B + 2)), plane by plane.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "af_adjoint.h"

using namespace af;

static int g_fail = 0;

// A window of node-cells [-H, B + H2): plane pl at offset b = (j + H) kRX + (i + H).
template <int H, int NX, int NY>
struct Win {
    static constexpr int kRX = 4096;   // rows far apart: an offset that leaves a row is seen
    std::vector<double>* a;
    int planes;
    int base(int i, int j) const { return (j + H) * kRX + (i + H); }
    bool ok(int pl, int b) const {
        const int x = b % kRX, y = b / kRX;
        const bool in = b >= 0 && pl >= 0 && pl < planes && x < NX && y < NY;
        if (!in && !g_fail++) std::fprintf(stderr, "plane %d, offset (%d, %d) outside %d x %d\n", pl, x, y, NX, NY);
        return in;
    }
    double& ref(int pl, int b) const { return (*a)[(size_t)pl * NX * NY + (size_t)(b / kRX) * NX + b % kRX]; }
    double at(int pl, int b, int off) const { return ok(pl, b + off) ? ref(pl, b + off) : 0.0; }
    void addb(int pl, int b, int off, double v) const {
        if (ok(pl, b + off)) ref(pl, b + off) += v;
    }
    void node(int fam, int i, int j, const double g[4]) const {
        for (int q = 0; q < 4; ++q) addb(win_plane(fam) + q, base(i, j), 0, g[q]);
    }
};

struct Cot {
    std::vector<double> v;
    double get(int k, int i, int j) const { return v[(size_t)(k * 31 + (i + 3) * 7 + (j + 3)) % v.size()]; }
};

template <int H, int NX, int NY>
struct Nodes {
    Win<H, NX, NY> w;
    Prim<double> node(int fam, int i, int j) const {
        const int b = w.base(i, j), p = win_plane(fam);
        return {w.at(p, b, 0), w.at(p + 1, b, 0), w.at(p + 2, b, 0), w.at(p + 3, b, 0)};
    }
};

template <int SCHEME>
static int points(double vmax, unsigned seed) {
    constexpr int B = 8, R = B + 3;
    std::mt19937 rng(seed);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    const double lam1 = 0.3, lam0 = 0.15;
    std::vector<double> s(40 * R * R), o(40 * R * R, 0.0);
    for (int pl = 0; pl < 40; ++pl)
        for (int e = 0; e < R * R; ++e) {
            const int q = pl < 16 ? pl % 4 : 4 + (pl - 16) % 3;
            s[(size_t)pl * R * R + e] = q == 0 || q == 3 ? 1.0 + 0.1 * U(rng) : (q == 6 ? 0.01 * U(rng) : vmax / lam1 * U(rng));
        }
    Cot c;
    for (int k = 0; k < 997; ++k) c.v.push_back(U(rng));
    const Win<1, R, R> S{&s, 40}, O{&o, 40};
    int split = 0;
    for (int j = 0; j < B; ++j)
        for (int i = 0; i < B; ++i) {
            const unsigned v = point_adj_target<F_V, SCHEME, 0>(S, c, O, i, j, 1.4, lam0, lam1);
            const unsigned e = point_adj_target<F_EV, SCHEME, 0>(S, c, O, i, j, 1.4, lam0, lam1);
            const unsigned h = point_adj_target<F_EH, SCHEME, 0>(S, c, O, i, j, 1.4, lam0, lam1);
            point_adj_target<F_V, SCHEME, 1>(S, c, O, i, j, 1.4, lam0, lam1, v);
            point_adj_target<F_EV, SCHEME, 1>(S, c, O, i, j, 1.4, lam0, lam1, e);
            point_adj_target<F_EH, SCHEME, 1>(S, c, O, i, j, 1.4, lam0, lam1, h);
            split += v + e + h;
        }
    for (double x : o)
        if (!std::isfinite(x)) ++g_fail;
    return split;
}

static void incr(double vmax, unsigned seed) {
    constexpr int BX = 16, BY = 8, NX = BX + 4, NY = BY + 4;
    std::mt19937 rng(seed);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    std::vector<double> s(16 * NX * NY), o(20 * NX * NY, 0.0);
    for (int pl = 0; pl < 16; ++pl)
        for (int e = 0; e < NX * NY; ++e) s[(size_t)pl * NX * NY + e] = pl % 4 == 0 || pl % 4 == 3 ? 1.0 + 0.1 * U(rng) : vmax * U(rng);
    const Win<2, NX, NY> S{&s, 16}, O{&o, 20};
    const Nodes<2, NX, NY> A{S};
    for (int j = -1; j < BY + 1; ++j)
        for (int i = -1; i < BX + 1; ++i) {
            double l[4][2][3], lW[4];
            for (auto& f : l)
                for (auto& t : f)
                    for (double& q : t) q = U(rng);
            for (double& q : lW) q = U(rng);
            incr_adj<5>(A, O, i, j, l[F_V], l[F_EV], true, 1.4, 0.15, 0.3);
            incr_adj<3>(A, O, i, j, l[F_EH], l[F_C], false, 1.4, 0.15, 0.3);
            if (i < BX && j < BY) centre_adj(A, O, i, j, lW, 1.4);
        }
    for (double x : o)
        if (!std::isfinite(x)) ++g_fail;
}

int main() {
    unsigned seed = 1;
    for (double vmax : {0.02, 0.4, 0.95, 1.5}) {
        const int a = points<0>(vmax, seed++), b = points<1>(vmax, seed++);
        std::printf("velocities to %.2f cells: %d and %d targets with feet in different cells\n", vmax, a, b);
        if (vmax >= 0.4 && (a < 20 || b < 20)) return 2;
        incr(vmax, seed++);
    }
    return g_fail != 0;
}
