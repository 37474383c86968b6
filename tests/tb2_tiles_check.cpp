// tb2_tiles_check.cpp — host test of the two-step kernel's work plans for both of its
// tile shapes (paper_2512_23116_amd/csrc/lbm_tb2_plan.hpp), built with address and
// undefined-behaviour sanitizers by tests/test_tb2_tiles_cpu.py.
//
// Each plan is made as the launch makes it: tile counts and costs of the one tile shape.
// Every cell column of the lattice lies in exactly one tile, and every (tile, plane)
// unit is taken by exactly one workgroup, inside its XCD's range.  The tile a lattice
// takes is the one that was measured faster.
//
// Exit status 0 and a summary line on success, a message and status 1 otherwise.
#include <stdint.h>
#include <stdio.h>

#include <vector>

#include "lbm_tb2_plan.hpp"

static uint64_t plans = 0;

static int fail(const char* what, uint32_t nx, uint32_t ny, uint32_t nz, uint64_t a) {
    fprintf(stderr, "FAIL %s: shape %u x %u x %u, %llu\n", what, nx, ny, nz, (unsigned long long)a);
    return 1;
}

template <class Tile>
static int check(uint32_t nx, uint32_t ny, uint32_t nz, uint32_t groups, uint32_t cus) {
    const uint32_t tx = (nx + Tile::TX - 1) / Tile::TX, ty = (ny + Tile::TY - 1) / Tile::TY;
    const uint32_t tiles = tx * ty;
    if ((tx - 1) * Tile::TX >= nx || (ty - 1) * Tile::TY >= ny) return fail("an empty tile", nx, ny, nz, tiles);
    std::vector<uint8_t> column((size_t)nx * ny, 0);
    for (uint32_t t = 0; t < tiles; ++t)
        for (uint32_t y = t / tx * Tile::TY; y < ny && y < (t / tx + 1) * Tile::TY; ++y)
            for (uint32_t x = t % tx * Tile::TX; x < nx && x < (t % tx + 1) * Tile::TX; ++x)
                if (column[x + (size_t)nx * y]++) return fail("column in two tiles", nx, ny, nz, t);
    for (uint8_t c : column)
        if (!c) return fail("column in no tile", nx, ny, nz, tiles);
    // a full tile costs 1, a partial one less, none less than its first phase alone
    for (uint32_t t = 0; t < tiles; ++t) {
        const double c = lbm::tile_cost(t, tx, nx, ny, Tile::TX, Tile::TY);
        const bool full = (t % tx + 1) * Tile::TX <= nx && (t / tx + 1) * Tile::TY <= ny;
        if (!(c > 0.65 && (full ? c > 0.9999 && c < 1.0001 : c < 1.0)))
            return fail("tile cost", nx, ny, nz, t);
    }
    const lbm::Tb2Plan P = lbm::make_plan(nx, ny, nz, tx, ty, groups, cus, Tile::TX, Tile::TY);
    if (P.w.cut[0] != 0 || P.w.cut[groups] != tiles) return fail("tile ranges", nx, ny, nz, groups);
    std::vector<uint8_t> seen((size_t)tiles * nz, 0);
    for (uint64_t h = 0; h < (uint64_t)groups * P.per_group; ++h) {
        uint32_t tile = 0, z0 = 0, n = 0;
        if (!lbm::tb2_item(P.w, nz, (uint32_t)h, tile, z0, n)) continue;
        const uint32_t g = (uint32_t)(h % groups);
        if (tile < P.w.cut[g] || tile >= P.w.cut[g + 1]) return fail("tile outside its group", nx, ny, nz, h);
        if (n < 1 || z0 + n > nz) return fail("chunk outside the lattice", nx, ny, nz, h);
        for (uint32_t z = z0; z < z0 + n; ++z)
            if (seen[(size_t)tile * nz + z]++) return fail("unit taken twice", nx, ny, nz, h);
    }
    for (uint8_t s : seen)
        if (!s) return fail("unit never taken", nx, ny, nz, groups);
    ++plans;
    return 0;
}

template <class Tile>
static int all() {
    static_assert(Tile::EX == Tile::TX + 2 && Tile::EY == Tile::TY + 2, "one cell of halo");
    static_assert(Tile::kThreads <= 1024, "threads of a workgroup");
    const uint32_t xs[] = {1, 2, 61, 62, 63, 64, 65, 93, 94, 124, 125, 127, 128, 129, 186};
    const uint32_t ys[] = {1, 2, 12, 13, 14, 15, 25, 26, 27, 28, 29, 40};
    const uint32_t zs[] = {1, 2, 3, 4, 17, 64, 131};
    for (uint32_t nx : xs)
        for (uint32_t ny : ys)
            for (uint32_t nz : zs)
                for (uint32_t groups : {1u, 8u})
                    for (uint32_t cus : {1u, 256u})
                        if (check<Tile>(nx, ny, nz, groups, cus)) return 1;
    const uint32_t large[][3] = {{800, 800, 800}, {1290, 1290, 1290}, {512, 512, 512}, {400, 400, 400},
                                 {256, 256, 256}, {331, 331, 331}, {100, 100, 100}, {48, 48, 48},
                                 {800, 800, 1}, {1, 1, 1290}, {3, 700, 1000}, {1000, 3, 700}};
    for (const auto& s : large)
        for (uint32_t groups : {1u, 8u})
            if (check<Tile>(s[0], s[1], s[2], groups, 256)) return 1;
    return 0;
}

// The tile each of these lattices takes: the faster one of two that were timed, where
// they differ by more than 5 %.
static int choice() {
    struct Case {
        uint32_t n, bytes;
        bool wide;
    };
    const Case cases[] = {{64, 4, true},   {100, 4, false}, {112, 4, false}, {176, 4, false},
                          {184, 4, false}, {216, 4, false}, {245, 4, true},  {248, 4, false},
                          {256, 4, true},  {260, 4, false}, {288, 4, false}, {300, 4, true},
                          {306, 4, true},  {320, 4, true},  {331, 4, false}, {352, 4, false},
                          {360, 4, true},  {370, 4, true},  {384, 4, true},  {392, 4, false},
                          {420, 4, true},  {434, 4, true},  {440, 4, true},  {492, 4, true},
                          {512, 4, true},  {576, 4, true},  {608, 4, true},  {640, 4, true},
                          {672, 4, true},  {704, 4, true},  {800, 4, true},  {64, 2, true},   {128, 2, true},  {184, 2, false},
                          {240, 2, false}, {256, 2, true},  {260, 2, false}, {320, 2, true},
                          {331, 2, false}, {384, 2, true},  {400, 2, false}, {450, 2, false},
                          {512, 2, true},  {640, 2, false}, {704, 2, false}};
    for (const Case& c : cases) {
        using W = lbm::Tb2Tile<true>;
        using N = lbm::Tb2Tile<false>;
        const double wide = lbm::make_plan(c.n, c.n, c.n, (c.n + W::TX - 1) / W::TX,
                                           (c.n + W::TY - 1) / W::TY, 8, 256, W::TX, W::TY).makespan;
        const double narrow = lbm::make_plan(c.n, c.n, c.n, (c.n + N::TX - 1) / N::TX,
                                             (c.n + N::TY - 1) / N::TY, 8, 256, N::TX, N::TY).makespan;
        if (lbm::wide_tile(c.n, c.n, c.bytes, wide, narrow) != c.wide)
            return fail("tile", c.n, c.n, c.n, c.bytes);
    }
    return 0;
}

int main() {
    if (choice()) return 1;
    if (all<lbm::Tb2Tile<true>>() || all<lbm::Tb2Tile<false>>()) return 1;
    printf("ok: %llu plans\n", (unsigned long long)plans);
    return 0;
}
