// Host check of tile_runs (af_tile.h): over the grids a context accepts (up to 2^31 cells, four
// cells or more a side) every tile belongs to exactly one launch, in order, and no launch has
// 2^32 work-items or more.
#include <cstdio>

#include "af_tile.h"

template <int NT>
static int check(long long nx, long long ny, int TX, int TY) {
    const long long tiles = ((nx + TX - 1) / TX) * ((ny + TY - 1) / TY);
    long long next = 0;
    int bad = tiles > 2147483647LL, runs = 0;
    af::tile_runs<NT>((int)tiles, [&](int first, int count) {
        bad |= first != next || count < 1 || (unsigned long long)count * NT >= 1ull << 32;
        next += count;
        ++runs;
    });
    bad |= next != tiles || (tiles * NT < 1LL << 31 && runs != 1);
    if (bad) std::fprintf(stderr, "%lldx%lld tile %dx%d/%d: %d launches, %lld of %lld tiles\n", nx, ny, TX, TY, NT, runs, next, tiles);
    return bad;
}

int main() {
    const long long g[][2] = {{4, 4},       {64, 64},         {2048, 2048},     {130000000, 4},  {4, 130000000}, {536870912, 4},
                              {4, 536870912}, {16, 134217728}, {46340, 46340},  {126000000, 4},  {62914560, 10}, {62914575, 10}};
    int bad = 0;
    for (const auto& s : g) {
        bad |= check<512>(s[0], s[1], 15, 10);
        bad |= check<512>(s[0], s[1], 31, 10);
        bad |= check<1024>(s[0], s[1], 31, 10);
    }
    return bad;
}
