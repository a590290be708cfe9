// Host walk of the packed tile (af_tile.h): every element gets a number of its own in the
// phase that writes it, and every read of the later phases must find the number of the
// element it names.  Catches an index outside the tile (subscripts are checked, the
// build is sanitized), two elements that share a place while both are read, an element
// that is read but never written, and work items that miss or repeat a node-cell.
#include <cstdio>
#include <memory>
#include <set>
#include <utility>

#include "af_tile.h"

using namespace af;

static int g_bad = 0;

template <class T>
static void expect(T got, int want, const char* what, int x, int y) {
    if ((int)got == want) return;
    if (++g_bad < 10) std::fprintf(stderr, "%s at (%d, %d): holds %d, expected %d\n", what, x, y, (int)got, want);
}

template <class T, int TX, int TY, int RW, int NT>
static void walk() {
    using Tile = PackedTile<T, TX, TY>;
    std::unique_ptr<Tile> L(new Tile());
    auto idp = [](int k, int x, int y) { return 1 + (k * 64 + y + 2) * 64 + x + 2; };
    auto idc = [](int k, int x, int y) { return 100000 + (k * 64 + y + 2) * 64 + x + 2; };
    auto idd = [](int t, int q, int x, int y) { return 200000 + ((t * 12 + q) * 64 + y + 2) * 64 + x + 2; };
    std::set<std::pair<int, int>> seen;
    int x, y;
    for (int e = 0; e < Tile::NSTAGE + NT; ++e) {
        if (!Tile::stage_item(e, x, y)) continue;
        seen.insert({x, y});
        for (int k = 0; k < 12; ++k) L->p(k, y, x) = T(idp(k, x - 2, y - 2));
    }
    expect((int)seen.size(), Tile::PX * Tile::PY, "staged node-cells", 0, 0);
    const TileAcc<Tile> A{L.get()};
    auto node = [&](int fam, int i, int j) {
        const Prim<T> n = A.node(fam, i, j);
        const T v[4] = {n.r, n.u, n.v, n.p};
        for (int k = 0; k < 4; ++k) expect(v[k], fam == F_C ? idc(k, i, j) : idp(4 * fam + k, i, j), "node", i, j);
    };
    seen.clear();
    for (int e = 0; e < Tile::NCENTRE + NT; ++e) {
        if (!Tile::centre_item(e, x, y)) continue;
        seen.insert({x, y});
        for (int k = 0; k < 4; ++k) L->c(k, y + 2, x + 2) = T(idc(k, x, y));
    }
    expect((int)seen.size(), Tile::CX * Tile::CY, "centres", 0, 0);
    // phase 1 reads the boundary nodes of every centre after other centres are written
    for (const auto& c : seen)
        for (int b = 0; b < 3; ++b)
            for (int a = 0; a < 3; ++a) node((a & 1) ? ((b & 1) ? F_C : F_EH) : ((b & 1) ? F_EV : F_V), c.first + a / 2, c.second + b / 2);
    seen.clear();
    for (int e = 0; e < Tile::NINCR + NT; ++e) {
        if (!Tile::incr_item(e, x, y)) continue;
        seen.insert({x, y});
        for (int b = -2; b <= 2; ++b)
            for (int a = -2; a <= 2; ++a)
                node((a & 1) ? ((b & 1) ? F_C : F_EH) : ((b & 1) ? F_EV : F_V), x + (a - (a & 1)) / 2, y + (b - (b & 1)) / 2);
        for (int t = 0; t < 2; ++t)
            for (int q = 0; q < 12; ++q)
                if (Tile::has_d(q, y + 1)) L->d(t, q, y + 1, x + 1) = T(idd(t, q, x, y));
    }
    expect((int)seen.size(), Tile::DX * Tile::DY, "increments", 0, 0);
    using Pts = typename Tile::template Points<RW>;
    std::set<std::pair<int, int>> targets[3];
    for (int e = 0; e < Pts::N + NT; ++e) {
        int fam;
        if (!Pts::item(e, fam, x, y)) continue;
        targets[fam].insert({x, y});
        node(fam, x, y);
        for (int t = 0; t < 2; ++t) {
            const TileInc<Tile> D{L.get(), t};
            for (int v = 0; v < 3; ++v) {
                if (x < TX + 1 && y < TY + 1) expect(D.inc(fam, x, y, v), idd(t, 3 * fam + v, x, y), "own increment", x, y);
                // the cells a foot within one cell can fall in
                for (int cy = -1; cy <= (fam == F_EV ? 1 : 0); ++cy)
                    for (int cx = -1; cx <= (fam == F_EH ? 1 : 0); ++cx)
                        for (int b = 0; b < 3; ++b)
                            for (int a = 0; a < 3; ++a) {
                                const int f = (a & 1) ? ((b & 1) ? F_C : F_EH) : ((b & 1) ? F_EV : F_V);
                                const int i = x + cx + a / 2, j = y + cy + b / 2;
                                expect(D.inc(f, i, j, v), idd(t, 3 * f + v, i, j), "increment", i, j);
                                node(f, i, j);
                            }
            }
        }
    }
    expect((int)targets[F_V].size(), (TX + 1) * (TY + 1), "V targets", 0, 0);
    expect((int)targets[F_EV].size(), (TX + 1) * TY, "Ev targets", 0, 0);
    expect((int)targets[F_EH].size(), TX * (TY + 1), "Eh targets", 0, 0);
}

int main() {
    walk<double, 15, 10, 16, 512>();
    walk<double, 8, 8, 0, 256>();
    walk<float, 8, 8, 0, 256>();
    if (g_bad) return 1;
    std::printf("packed tile: every read finds its element\n");
    return 0;
}
