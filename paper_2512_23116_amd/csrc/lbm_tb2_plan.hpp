// lbm_tb2_plan.hpp — which (tile, z chunk) each workgroup of the two-step
// kernel takes, and the host's choice of that plan for a lattice shape.
// The item lookup is plain integer code shared by the kernel and the host test
// of the plan (built with address and undefined-behaviour sanitizers).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <functional>
#include <queue>
#include <vector>

namespace lbm {

// Tile of one workgroup, extended by a one-cell halo, in one of two shapes: 64 x 13
// columns with the halo columns in a wave of their own, or 62 x 14 (64 x 16 with the
// halo) in a wave per row.  lbm_tb2.hip says which lattice takes which, and why.
template <bool kWave>
struct Tb2Tile {
    static constexpr int TX = kWave ? 64 : 62, TY = kWave ? 13 : 14;
    static constexpr int EX = TX + 2, EY = TY + 2;
    static constexpr int kThreads = 64 * (EY + (kWave ? 1 : 0));
};
// The tile of make_plan where none is named: 64 x 13.  tiles_x, tiles_y and the tile have to
// belong together; a launch names its own.
constexpr int TB_TX = Tb2Tile<true>::TX, kTbTY = Tb2Tile<true>::TY;
constexpr int TB_MAX_CHUNKS = 64;

// Work plan of a launch: the tiles are split into `groups` contiguous ranges
// cut[g] .. cut[g+1] (one per XCD; workgroup h runs on XCD h % 8), every tile
// into the same z chunks of zlen planes, the last one shorter: chunk k is planes
// k zlen .. min((k+1) zlen, nz) - 1.  Workgroup h takes item h / groups of its
// group, items ordered chunk-major: chunk k of every tile of the range, in tile
// order, then chunk k + 1.  Groups with fewer items pad with workgroups that
// exit at once.
struct Tb2Work {
    uint32_t groups, nchunk, zlen;
    uint32_t cut[9];
};

// Tile index, first plane and plane count of workgroup h of a lattice nz planes
// deep; false for padding.
__host__ __device__ inline bool tb2_item(const Tb2Work& W, uint32_t nz, uint32_t h,
                                         uint32_t& tile, uint32_t& z0, uint32_t& nzc) {
    const uint32_t grp = h % W.groups, item = h / W.groups;
    const uint32_t t0 = W.cut[grp], nt = W.cut[grp + 1] - t0;
    if (item >= nt * W.nchunk) return false;
    const uint32_t chunk = item / nt;
    tile = t0 + (item - chunk * nt);
    z0 = chunk * W.zlen;
    nzc = (nz - z0 < W.zlen) ? nz - z0 : W.zlen;
    return true;
}

struct Tb2Plan {
    Tb2Work w{};
    uint32_t per_group = 0;   // workgroups per group: the launch has groups * per_group
    double makespan = 0.0;    // estimated finishing time, in planes of a full tile
};

// Relative cost of one plane of a tile: phase 1 runs on all its columns,
// phase 2 on the interior only, about 35 % of a full tile's time (a 62 x 14
// tile with 2 of its 14 interior rows takes 0.70 of a full one at 800^3).
inline double tile_cost(uint32_t tile, uint32_t tiles_x, uint32_t nx, uint32_t ny,
                        uint32_t tw, uint32_t th) {
    const uint32_t x = tile % tiles_x, y = tile / tiles_x;
    const uint32_t w = std::min<uint32_t>(tw, nx - x * tw);
    const uint32_t h = std::min<uint32_t>(th, ny - y * th);
    return 0.65 + 0.35 * double(w * h) / double(tw * th);
}

// Finishing time of the slowest group when each group's CUs take its items in
// order as they free up (list scheduling), an item costing its planes plus
// three: the two planes a chunk starts with and the workgroup's start-up (at
// 800^3 an item takes about 10 us plus 5.7 us per plane, and about 5 us pass
// between two items on a CU), times its tile's cost.
inline double plan_makespan(const Tb2Plan& P, uint32_t nz, const std::vector<double>& cost,
                            uint32_t cus_per_group) {
    double worst = 0.0;
    std::vector<double> cu;
    for (uint32_t g = 0; g < P.w.groups; ++g) {
        cu.assign(std::max<uint32_t>(1, cus_per_group), 0.0);
        std::priority_queue<double, std::vector<double>, std::greater<double>> q(cu.begin(),
                                                                               cu.end());
        for (uint32_t k = 0; k < P.w.nchunk; ++k) {
            const uint32_t z0 = k * P.w.zlen, n = std::min(P.w.zlen, nz - z0);
            const double planes = double(n + 3);
            for (uint32_t t = P.w.cut[g]; t < P.w.cut[g + 1]; ++t) {
                const double free_at = q.top();
                q.pop();
                q.push(free_at + planes * cost[t]);
            }
        }
        while (!q.empty()) {
            worst = std::max(worst, q.top());
            q.pop();
        }
    }
    return worst;
}

// The plan for a lattice shape: tiles cut into `groups` ranges of equal total
// cost, and of the chunk lengths tried (every length from 2 planes up to nz
// that changes the chunk count or the last chunk's length by a step: below 256^3 the
// tiles alone are too few for the CUs, and chunks of 16 planes at least had left 100^3
// at 112 workgroups and 80 us per launch where 240 take 49) the one
// with the smallest estimated finishing time.
inline Tb2Plan make_plan(uint32_t nx, uint32_t ny, uint32_t nz, uint32_t tiles_x,
                         uint32_t tiles_y, uint32_t groups, uint32_t cus,
                         uint32_t tw = TB_TX, uint32_t th = kTbTY) {
    const uint32_t tiles = tiles_x * tiles_y;
    std::vector<double> cost(tiles), cum(tiles + 1, 0.0);
    for (uint32_t t = 0; t < tiles; ++t) {
        cost[t] = tile_cost(t, tiles_x, nx, ny, tw, th);
        cum[t + 1] = cum[t] + cost[t];
    }
    Tb2Plan best;
    best.w.groups = groups;
    for (uint32_t g = 0; g <= groups; ++g) {
        const double target = cum[tiles] * g / groups;
        uint32_t t = 0;
        while (t < tiles && cum[t] < target) ++t;
        best.w.cut[g] = (g == groups) ? tiles : t;
    }
    const uint32_t cus_per_group = std::max<uint32_t>(1, cus / groups);
    // more than 64 items per CU gain nothing and cost planning time
    const uint64_t max_items = 64ull * std::max<uint32_t>(1, cus);
    double best_ms = -1.0;
    auto consider = [&](uint32_t zlen) {
        Tb2Plan P = best;
        P.w.zlen = zlen;
        P.w.nchunk = (nz + zlen - 1) / zlen;
        if (P.w.nchunk > (uint32_t)TB_MAX_CHUNKS) return;
        if (P.w.nchunk > 1 && (uint64_t)tiles * P.w.nchunk > max_items) return;
        const double ms = plan_makespan(P, nz, cost, cus_per_group);
        if (best_ms < 0.0 || ms < best_ms * (1.0 - 1e-9)) {
            best_ms = ms;
            best = P;
            best.makespan = ms;
        }
    };
    consider(nz);                          // one chunk: always possible
    const uint32_t step = std::max<uint32_t>(1, nz / 256);
    for (uint32_t zlen = 2; zlen < nz; zlen += step) consider(zlen);
    for (uint32_t g = 0; g < groups; ++g) {
        const uint32_t items = (best.w.cut[g + 1] - best.w.cut[g]) * best.w.nchunk;
        best.per_group = std::max(best.per_group, items);
    }
    return best;
}

// Which tile a lattice takes, 64 x 13 (true) or 62 x 14, from the finishing times that
// their plans estimate.  ms per launch at n^3, 64 x 13 / 62 x 14:
//  * Rows of whole 128-byte lines: 64 x 13, whose rows are whole lines too, unless its
//    plan is the longer one (the last tile column or row mostly empty).
//      FP32  256: 0.61/0.69  320: 1.09/1.30  512: 4.36/4.85;  288: 0.88/0.80  352: 2.12/1.62
//      FP16  256: 0.46/0.51  512: 3.39/3.60;  640: 7.1/6.5  704: 8.9/8.3
//    In FP32 by 2 % (640: 9.3/9.9, 704: 12.2/13.8, of plans 1.006 and 1.004 times as long),
//    or where 62 x 14 has a full last column (below; 608: 7.5/8.4, 800: 17.8/18.8).
//  * Other rows, 16-bit: 62 x 14.  245: 0.48/0.38  331: 1.20/0.95  400: 2.05/1.89
//  * Other rows, FP32, while a plane of the 19 populations fits the 4 MB L2 of an XCD,
//    where tiles find the lines they share: 62 x 14.
//      100: 0.047/0.044  112: 0.081/0.050  184: 0.32/0.27  232: 0.52/0.47
//  * Past that 62 x 14 loses those lines where its last tile column is more than three
//    quarters full (with a narrower one the neighbours keep step): 64 x 13 then, if its
//    plan is not much the longer one, and wherever its plan is the shorter one.
//      245: 0.63/0.68  306: 1.10/1.33  370: 2.10/2.69  434: 3.0/3.9  492: 4.9/5.4
//      440: 3.04/3.35 (shorter plan);  248: 0.71/0.58 (plan 1.16 times as long)
//      260: 0.80/0.75  331: 1.63/1.31  392: 2.59/2.22  450: 3.87/3.68  475: 4.7/4.6
// (wide_possible: the plans need not be asked where it is false; at 800^3 one takes 18 ms.)
inline bool wide_possible(uint32_t nx, uint32_t ny, uint32_t elem_bytes) {
    return (uint64_t)nx * elem_bytes % 128 == 0 ||
           (elem_bytes == 4 && (uint64_t)nx * ny * 19 * elem_bytes > (4u << 20));
}
inline bool wide_tile(uint32_t nx, uint32_t ny, uint32_t elem_bytes, double wide, double narrow) {
    if (!wide_possible(nx, ny, elem_bytes)) return false;
    const uint32_t tx = Tb2Tile<false>::TX;
    const bool lines = (uint64_t)nx * elem_bytes % 128 == 0;
    if (elem_bytes != 4) return wide <= narrow;
    const bool full = 4 * ((nx - 1) % tx + 1) > 3 * tx;
    return wide < (lines ? 1.02 : 1.0) * narrow || (full && wide < 1.12 * narrow);
}

}  // namespace lbm
