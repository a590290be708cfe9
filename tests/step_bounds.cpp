// Host walk of the step kernels' tiles as they are launched: every phase of every tile of a grid
// through the arithmetic that the kernels run (the pairs of families, u + du in the velocities'
// increment planes of the transported update), with the LDS tile as an object of its own.
// Built with address and undefined-behaviour sanitizers; besides, the tile starts as NaN, so that
// a value read before it is written, or from a place that nothing writes, reaches a result.
// Grids ragged, smaller than the window, and whole multiples of the tiles; node velocities up to 1.5 cells a
// step, so that feet leave the window's reach and the foot guard must clamp them.
#include <cmath>
#include <cstdio>
#include <limits>
#include <memory>
#include <random>
#include <vector>

#include "af_tile.h"

using namespace af;

static int g_fail = 0;

#define REQUIRE(cond, ...)                                   \
    do {                                                     \
        if (!(cond)) {                                       \
            std::fprintf(stderr, __VA_ARGS__);               \
            std::fprintf(stderr, "\n");                      \
            ++g_fail;                                        \
            return;                                          \
        }                                                    \
    } while (0)

template <class T>
static bool finite(const Prim<T>& w) {
    return std::isfinite((double)w.r) && std::isfinite((double)w.u) && std::isfinite((double)w.v) && std::isfinite((double)w.p);
}

template <class Tile, int RW, int NT, int SCHEME>
static void walk(int nx, int ny, double vmax, unsigned seed) {
    using T = typename Tile::S;
    constexpr int TX = Tile::X, TY = Tile::Y;
    constexpr bool kSum = SCHEME == 0;
    std::unique_ptr<Tile> L(new Tile());
    std::mt19937 rng(seed);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    const PolAbs<T> pol{T(1.4), T(1.0 / 0.4)};
    const T lam1 = T(0.3), lam0 = T(0.15);
    const size_t N = (size_t)nx * ny;
    const bool onex = nx >= Tile::PX, oney = ny >= Tile::PY;
    const TileAcc<Tile> A{L.get()};
    for (int j0 = 0; j0 < ny; j0 += TY)
        for (int i0 = 0; i0 < nx; i0 += TX) {
            unsigned st = 0;
            static_assert(sizeof(Tile) % sizeof(T) == 0, "a tile is an array of T");
            for (size_t k = 0; k < sizeof(Tile) / sizeof(T); ++k) ((T*)L.get())[k] = std::numeric_limits<T>::quiet_NaN();
            int x, y;
            for (int e = 0; e < Tile::NSTAGE + NT; ++e) {
                if (!Tile::stage_item(e, x, y)) continue;
                const size_t g = (size_t)wrap_win(j0 + y - 2, ny, oney) * nx + wrap_win(i0 + x - 2, nx, onex);
                REQUIRE(g < N, "stage: global index %zu outside %zu (grid %dx%d, tile %d,%d)", g, N, nx, ny, i0, j0);
                for (int k = 0; k < 12; ++k)
                    L->p(k, y, x) = k % 4 == 0 || k % 4 == 3 ? T(1.0 + 0.1 * U(rng)) : T(vmax / (double)lam1 * U(rng));
            }
            for (int e = 0; e < Tile::NCENTRE + NT; ++e) {
                if (!Tile::centre_item(e, x, y)) continue;
                const size_t g = (size_t)wrap_win(j0 + y, ny, oney) * nx + wrap_win(i0 + x, nx, onex);
                REQUIRE(g < N, "centre: global index %zu outside %zu", g, N);
                const T Ub[4] = {T(1), T(0.1), T(-0.1), T(2.6)};
                const Prim<T> n[8] = {A.node(F_V, x, y), A.node(F_V, x + 1, y), A.node(F_V, x, y + 1), A.node(F_V, x + 1, y + 1),
                                      A.node(F_EH, x, y), A.node(F_EH, x, y + 1), A.node(F_EV, x, y), A.node(F_EV, x + 1, y)};
                for (const auto& w : n) REQUIRE(finite(w), "centre (%d, %d) reads a node that is not staged", x, y);
                (void)pol.centre(Ub, n[0], n[1], n[2], n[3], n[4], n[5], n[6], n[7]);
                // (a physical centre of the same velocities, for the later phases)
                L->c(0, y + 2, x + 2) = T(1);
                L->c(1, y + 2, x + 2) = T(vmax / (double)lam1 * U(rng));
                L->c(2, y + 2, x + 2) = T(vmax / (double)lam1 * U(rng));
                L->c(3, y + 2, x + 2) = T(1);
            }
            bool good = true;
            auto put = [&](int pl, T v) {
                const int fam = (pl % 12) / 3, q = pl % 3;
                if (kSum && q == 0) v = A.node(fam, x, y).u + v;
                if (kSum && q == 1) v = A.node(fam, x, y).v + v;
                good = good && std::isfinite((double)v);
                if (Tile::has_d(pl % 12, y + 1)) L->d(pl / 12, pl % 12, y + 1, x + 1) = v;
            };
            constexpr int NI = (Tile::NINCR + 63) / 64 * 64;
            for (int e = 0; e < (NT >= 2 * NI ? NT : Tile::NINCR + NT); ++e) {
                if constexpr (NT >= 2 * NI) {
                    if (e < NI) {
                        if (Tile::incr_item(e, x, y)) put_pair<5>(A, x, y, pol, lam0, lam1, st, put);
                    } else if (e < 2 * NI) {
                        if (Tile::incr_item(e - NI, x, y)) put_pair<3>(A, x, y, pol, lam0, lam1, st, put);
                    }
                } else if (Tile::incr_item(e, x, y)) {
                    cell_increments(A, x, y, pol, lam0, lam1, st, put);
                }
                REQUIRE(good, "item %d: increments not finite", e);
            }
            using Pts = typename Tile::template Points<RW>;
            const TileInc<Tile> D0{L.get(), 0}, D1{L.get(), 1};
            std::vector<int> item;
            for (int e = 0; e < Pts::N + NT; ++e) {
                int fam;
                if (!Pts::item(e, fam, x, y)) continue;
                REQUIRE(x >= 0 && x <= TX && y >= 0 && y <= TY, "point item (%d, %d) outside [0, T]", x, y);
                Prim<T> wh, w1;
                point_update_pair_f<SCHEME, kSum>(A, D0, D1, fam, x, y, pol, lam0, lam1, st, wh, w1);
                REQUIRE(finite(wh) && finite(w1), "target %d (%d, %d): value not finite", fam, x, y);
                item.push_back(fam);
                item.push_back(x);
                item.push_back(y);
            }
            for (size_t q = 0; q < item.size(); q += 3) {
                const int fam = item[q], tx = item[q + 1], ty = item[q + 2];
                if (fam == F_V)
                    for (int k = 0; k < 8; ++k) L->F.FV[k][ty][tx] = T(0.5);
                else if (fam == F_EV)
                    for (int k = 0; k < 4; ++k) L->F.FE[k][ty][tx] = T(0.5);
                else
                    for (int k = 0; k < 4; ++k) L->F.GE[k][ty][tx] = T(0.5);
            }
            for (int e = 0; e < TX * TY + NT; ++e) {
                if (!Tile::update_item(e, x, y) || i0 + x >= nx || j0 + y >= ny) continue;
                for (int k = 0; k < 4; ++k) {
                    const T s = L->F.FV[k][y][x] + L->F.FE[k][y][x] + L->F.FV[k][y + 1][x] + L->F.FV[k][y][x + 1] +
                                L->F.FE[k][y][x + 1] + L->F.FV[k][y + 1][x + 1] + L->F.FV[4 + k][y][x] + L->F.GE[k][y][x] +
                                L->F.GE[k][y + 1][x] + L->F.FV[4 + k][y + 1][x + 1];
                    REQUIRE(s == T(5), "update (%d, %d) reads a flux that is not stored", x, y);
                }
            }
            if (vmax >= 1.0) REQUIRE((st & SB_FOOT) != 0, "large velocities did not raise the foot flag");
        }
}

template <class Tile, int RW, int NT>
static void both(int nx, int ny, double vmax, unsigned& seed) {
    walk<Tile, RW, NT, 0>(nx, ny, vmax, seed++);
    walk<Tile, RW, NT, 1>(nx, ny, vmax, seed++);
}

int main() {
    const int grids[][2] = {{4, 4}, {5, 7}, {30, 20}, {33, 12}, {9, 40}};
    unsigned seed = 1;
    for (const auto& g : grids)
        for (double vmax : {0.4, 1.5}) {
            both<PackedTile<double, 15, 10>, 16, 512>(g[0], g[1], vmax, seed);
            both<FusedTile<double, 31, 10>, 32, 512>(g[0], g[1], vmax, seed);
            both<PackedTile<double, 8, 8>, 0, 256>(g[0], g[1], vmax, seed);
            both<FusedTile<double, 4, 4>, 0, 128>(g[0], g[1], vmax, seed);
            both<PackedTile<float, 8, 8>, 0, 256>(g[0], g[1], vmax, seed);
            both<FusedTile<float, 4, 4>, 0, 128>(g[0], g[1], vmax, seed);
            both<FusedTile<float, 31, 10>, 32, 512>(g[0], g[1], vmax, seed);
            both<FusedTile<float, 31, 10>, 32, 1024>(g[0], g[1], vmax, seed);
            if (g_fail) return 1;
        }
    std::printf("step tiles: every access in bounds, every value read was written\n");
    return 0;
}
