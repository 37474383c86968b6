// lbm_tb2.hip — two time steps per pass over HBM (A/B pull streaming).
//
// A single step moves 2 * 19 * b bytes per cell through HBM, and the
// single-step kernel runs at the ceiling of that access pattern.  This kernel
// keeps the intermediate time level on chip instead: a workgroup owns a tile of
// (x, y) columns (64 x 13 or 62 x 14) plus a one-cell halo, 1024 threads, and
// marches along z through a chunk of planes.  Which (tile,
// chunk) a workgroup takes is planned on the host once per lattice shape
// (lbm_tb2_plan.hpp): each XCD owns a contiguous range of tiles and runs
// their chunks in order, the long ones first and one short chunk per tile
// last, so that its CUs run out of work at nearly the same time.
//   phase 1  each of the extended tile's columns pulls f(t) of plane z+1 from A
//            (eq. mrt_dns_guo, periodic) and collides; of the post-collision
//            values it keeps in LDS exactly what phase 2 will pull: the 5
//            populations with c_z = -1 (needed now), the 9 with c_z = 0
//            (needed one plane later, 2 slots) and the 5 with c_z = +1
//            (needed two planes later, 3 slots): 38 floats per column,
//            150-156 KB of the 160 KB LDS of a CDNA4 CU;
//   phase 2  each interior column pulls the step-(t+1) populations of plane z
//            from those buffers (planes z+1, z, z-1 and the neighbouring
//            columns), collides and writes B at its own cell.
// The loads of a phase-1 plane are issued two planes ahead.  HBM traffic per two
// cell updates: A is read once per extended column (1.18-1.19 of the interior,
// plus 2 planes per chunk) and B is written once, instead of two full reads and
// writes.
// Per cell the arithmetic is the single-step collision, instruction for instruction,
// and for 16-bit storage the LDS buffers hold the intermediate level in the storage
// format: the result has the bits of two single steps.  It does not depend on the
// tile or the work plan.
#include <algorithm>
#include <array>
#include <atomic>
#include <map>
#include <mutex>
#include <utility>

#include "lbm_device.hpp"
#include "lbm_tb2_plan.hpp"

namespace lbm {

// Position of direction i within its class of c_z (-1: 5, 0: 9, +1: 5).
__host__ __device__ constexpr int zclass_index(int i) {
    int n = 0;
    for (int k = 0; k < i; ++k) n += (cz_of(k) == cz_of(i)) ? 1 : 0;
    return n;
}

struct TB2Args {
    LatticeArgs L;
    uint32_t tiles_x, tiles_y;
    Tb2Work W;
};

__device__ __forceinline__ uint32_t wrap_add(uint32_t base, int d, uint32_t n) {
    // (base + d) mod n for base < n and -1 <= d <= 64 (n >= 1)
    int v = (int)base + d;
    if (v < 0) v += (int)n;
    return (uint32_t)v % n;
}

// What holds this kernel is the cache lines it moves, not its instructions: with the
// loads and stores taken out it takes 1.7 of 6.1 ms (512^3 FP32), loads alone 3.2 and
// stores alone 3.1, and their times add.  Hence the two tiles (Tb2Tile):
//   - kHaloWave: 64 x 13 columns, a wave per row of the extended tile, and the columns
//     left and right of the rows in a wave of their own.  Where a lattice row is a whole
//     number of 128-byte lines the tile's rows are whole lines too.  Row pieces of 62
//     columns start anywhere, so that two of the three lines of every stored piece are
//     written in parts by two workgroups.
//   - 62 x 14 columns, 64 x 16 with the halo, a wave per row, where rows start anywhere
//     in a line in any case: the halo columns cost no lines of their own.
// wide_tile says which lattice takes which, with both measured.  Before there were two,
// the kernel took 6.1 ms at 512^3 FP32 (4.4 now), 0.83 / 0.56 at 256^3 FP32 / FP16 (0.61 /
// 0.46), 2.26 at 400^3 BF16 (1.98), 14.0 at 800^3 FP16 (12.9).  Of 48 FP32 and 28 16-bit
// lattices timed against that kernel, FP32 ones with rows of no whole 32-byte sectors are
// slower in two places: 236^3 to 245^3 by 2 to 3 % (it fetches two planes ahead, and the
// lines that neighbours share leave the L2 sooner), 470^3 and 475^3 by 3 to 5 %.
// What a plane's pulls wait for matters next.  Loads and stores of a wave complete in
// order under one counter, so nothing in the loop is loaded to be used at once (a
// force-table load per plane, waited for, had drained every pull and store in flight),
// a pull is kept as stored and decoded where it is used, and pulls are never skipped
// (past the last plane they repeat it): a wait counts the accesses that are certain.
// That and the addressing took 800^3 FP16 from 13.9 to 11.9 ms.  FP32 pulls after the
// stores and the second barrier of a plane: reads and writes then reach memory in turns,
// not mixed (512^3 4.9 -> 4.3 ms, 320^3 1.20 -> 1.05); 16-bit storage, with half the
// bytes, loses more to the later start (256^3 FP16 0.48 -> 0.51).
template <class Cd, bool kHaloWave>
__global__ __launch_bounds__(Tb2Tile<kHaloWave>::kThreads) void k_step_tb2(TB2Args A) {
    using Tile = Tb2Tile<kHaloWave>;
    constexpr int TB_TX = Tile::TX, TB_TY = Tile::TY, TB_EX = Tile::EX, TB_EY = Tile::EY;
    constexpr int TB_E = TB_EX * TB_EY;
    static_assert((kHaloWave ? TB_TX : TB_EX) == 64 && 2 * TB_EY <= 64, "lanes per row and halo");
    using T = typename Cd::T;
    using R = typename Cd::R;
    static_assert(std::is_same_v<R, float>, "the collision runs in FP32");
    // 16-bit storage: the intermediate level stays in LDS in the storage format
    // (the values a single step would store), at 2 B per value.  That leaves room
    // to rotate the buffers over more slots (down 2, mid 3, up 4: 57 values per
    // column) so that phase 1 of the next plane may overwrite no slot
    // phase 2 of this plane still reads: one barrier per plane.  FP32 storage
    // keeps FP32 values in the minimal 38 slots and two barriers.
    constexpr bool k16 = sizeof(T) == 2;
    using LT = std::conditional_t<k16, T, R>;
    constexpr int ND = k16 ? 2 : 1, NM = k16 ? 3 : 2, NU = k16 ? 4 : 3;
    __shared__ LT down[ND][5][TB_E];   // c_z = -1 populations of plane z+1
    __shared__ LT mid[NM][9][TB_E];    // c_z =  0 populations, planes z+1, z (, z-1)
    __shared__ LT up[NU][5][TB_E];     // c_z = +1 populations, planes z+1, z, z-1 (, z-2)
    __shared__ R rowbuf[2][TB_EY][16];  // force row coefficients of two phase-1 planes

    const LatticeArgs& L = A.L;
    uint32_t tile, Z0, nplanes;
    if (!tb2_item(A.W, L.nz, blockIdx.x, tile, Z0, nplanes)) return;   // padding: all leave
    // (divisions run on the VALU: bring their uniform results back to scalar registers)
    tile = __builtin_amdgcn_readfirstlane(tile);
    Z0 = __builtin_amdgcn_readfirstlane(Z0);
    nplanes = __builtin_amdgcn_readfirstlane(nplanes);
    const uint32_t tile_x = tile % A.tiles_x, tile_y = tile / A.tiles_x;
    const uint32_t X0 = tile_x * TB_TX, Y0 = tile_y * TB_TY;
    const int niter = (int)nplanes + 2;   // output planes of this chunk, and two ahead

    // phase-1 column (ex, ey) of the extended tile: a wave per row, either of all its
    // columns or of the tile's own; then the last wave takes the columns left and
    // right of every row (its lanes past those repeat one)
    const int t = threadIdx.x, lane = t & 63;
    const bool main = !kHaloWave || t < 64 * TB_EY;
    const int q = lane % (2 * TB_EY);
    const int ex = !kHaloWave ? lane : (main ? lane + 1 : (q & 1) * (TB_EX - 1));
    const int ey = main ? t >> 6 : q >> 1;
    const int col = ex + TB_EX * ey;
    // wrapped onto the lattice (columns past its far edges too: letting them repeat the
    // last one that is needed reads fewer lines but measured 5-10 % slower, 331^3 and
    // 450^3 FP32)
    const uint32_t x1 = wrap_add(X0, ex - 1, L.nx), y1 = wrap_add(Y0, ey - 1, L.ny);
    // phase-2 column: interior only, never wrapped (x1, y1 are its own coordinates)
    const bool inner = main && ex >= 1 && ex <= TB_TX && ey >= 1 && ey <= TB_TY &&
                       X0 + (uint32_t)ex - 1u < L.nx && Y0 + (uint32_t)ey - 1u < L.ny;

    // 16-bit storage: populations and force in units of 1/sigma (collide's
    // kScaled), so that every pass through the storage format is a conversion
    const R inv_s = inv_scale_of<R>(L), s_st = scale_of<R>(L);
    const R load_s = k16 ? R(1) : inv_s, store_s = k16 ? R(1) : s_st;
    const CollideConst<R>& k = collide_const<R>(L);
    auto to_lds = [&](R v) -> LT {
        if constexpr (k16) return enc<Cd>(v, R(1));
        else return v;
    };
    auto from_lds = [&](LT v) -> R {
        if constexpr (k16) return dec<Cd>(v, R(1));
        else return v;
    };

    // Addressing: the plane of a direction and the z of its source are the same for
    // the whole workgroup and go into the scalar base of each access; the lane's part
    // is its (x, y) column, whose nine neighbour offsets (in bytes, periodic) are
    // formed once per workgroup.  The march then computes no vector address at all.
    const uint64_t pbytes = L.plane * (uint64_t)sizeof(T);
    const uint32_t zbytes = L.nxy * (uint32_t)sizeof(T);   // < 2^32 (plane bytes are)
    uint32_t off[3][3];   // [1 + dy][1 + dx]
    {
        const uint32_t xs[3] = {x1 == 0 ? L.nx - 1 : x1 - 1, x1, x1 + 1 == L.nx ? 0 : x1 + 1};
        const uint32_t ys[3] = {y1 == 0 ? L.ny - 1 : y1 - 1, y1, y1 + 1 == L.ny ? 0 : y1 + 1};
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
                off[dy][dx] = (xs[dx] + L.nx * ys[dy]) * (uint32_t)sizeof(T);
    }
    // The bases are formed per use from values the compiler cannot see through: kept
    // live across the loop, the 38 of them would spill scalar registers to vector
    // lanes.
    auto opaque = [](uint64_t v) -> uint64_t {
        uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
        uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        asm volatile("" : "+s"(lo), "+s"(hi));
        return ((uint64_t)hi << 32) | lo;
    };
    auto plane_at = [&](const void* array, uint32_t z) -> uint64_t {
        return opaque((uint64_t)array + (uint64_t)z * zbytes);
    };
    // (defines an offset anew, for the 32-bit lane offset of an access to be seen
    // where the access is: hoisted as 64-bit values they cost an addition per access)
    auto refresh = [](uint32_t& o) { asm volatile("" : "+v"(o)); };

    auto plane1 = [&](int j) {   // z of the phase-1 plane of iteration j: Z0 - 1 + j, wrapped
        int z = (int)Z0 - 1 + min(j, niter - 1);   // (past the last plane: that one again)
        if (z < 0) z += (int)L.nz;
        if (z >= (int)L.nz) z -= (int)L.nz;
        return (uint32_t)z;
    };
    // Force (eq. forcing_pattern, force_sum).  The x harmonics stay in registers; a row's
    // coefficients are pulled by the row's own wave (one value a lane) with the
    // populations of the plane before, and go through LDS to the wave and the halo
    // columns of that row.
    const bool forced = L.rowc != nullptr;
    R h1 = R(0), h2 = R(0), h3 = R(0), h4 = R(0);
    if (forced) {
        const R* xt = (const R*)L.xtab + (uint64_t)x1 * 4;
        h1 = xt[0];
        h2 = xt[1];
        h3 = xt[2];
        h4 = xt[3];
    }
    auto row_coeff = [&](int j) -> R {
        return ((const R*)L.rowc)[(uint64_t)(y1 + L.ny * plane1(j)) * 16 + (lane & 15)];
    };
    const bool row_writer = main && lane < 16;

    struct Pulled {   // what iteration j consumes: populations of its plane, as stored,
        T g[19];      // and its row coefficient of the next
        R row;
    };
    auto pull = [&](int j, Pulled& P) {
        const uint32_t z = plane1(j);
        const uint64_t pb = opaque(pbytes);
        const PlaneStride src[3] = {
            {(char*)plane_at(L.a, z == 0 ? L.nz - 1 : z - 1), pb},
            {(char*)plane_at(L.a, z), pb},
            {(char*)plane_at(L.a, z + 1 == L.nz ? 0 : z + 1), pb}};
#pragma unroll
        for (int e = 0; e < 9; ++e) refresh(off[e / 3][e % 3]);
        if (forced) P.row = row_coeff(j + 1);
        static_for<19>([&](auto I) {
            constexpr int i = decltype(I)::value;
            P.g[i] = *(LBM_GLOBAL_SPACE const T*)(src[1 - cz_of(i)](i) +
                                                  off[1 - cy_of(i)][1 - cx_of(i)]);
        });
    };

    // One iteration j: phase 1 on the prefetched pulls P of plane Z0 - 1 + j,
    // then phase 2 on plane Z0 + j - 2, and before it (16-bit) or after it (FP32) the
    // pulls of plane j + 2 are issued into P (two planes of prefetch in flight).
    // The phase-2 cell of iteration j is the phase-1 cell of iteration j - 1 (same
    // column, plane Z0 + j - 2): its force is carried over instead of recomputed.
    R Fpx = R(0), Fpy = R(0), Fpz = R(0);
    auto iteration = [&](int j, Pulled& P) {
        const uint32_t uj = (uint32_t)j;
        R Fx = R(0), Fy = R(0), Fz = R(0);
        {   // phase 1: step t at plane Z0 - 1 + j for every extended column
            R g[19];
#pragma unroll
            for (int i = 0; i < 19; ++i) g[i] = dec<Cd>(P.g[i], load_s);
            if (forced) {
                force_sum<R>(rowbuf[uj & 1][ey], h1, h2, h3, h4, Fx, Fy, Fz);
                if constexpr (k16) {
                    Fx *= s_st;
                    Fy *= s_st;
                    Fz *= s_st;
                }
                // read in the next iteration, after the barrier; last read in phase 1
                // of the one before, which every wave has left
                if (row_writer) rowbuf[(uj + 1) & 1][ey][lane] = P.row;
            }
            collide<R, k16>(g, Fx, Fy, Fz, k, inv_s);
            const uint32_t sd = uj % ND, sm = uj % NM, su = uj % NU;
            static_for<19>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cz = cz_of(i), ii = zclass_index(i);
                const LT v = to_lds(g[i]);
                if constexpr (cz < 0) down[sd][ii][col] = v;
                else if constexpr (cz == 0) mid[sm][ii][col] = v;
                else up[su][ii][col] = v;
            });
        }
        __syncthreads();
        if constexpr (k16) pull(j + 2, P);
        if (j >= 2 && j < niter && inner) {   // phase 2: step t+1 at plane Z0 + j - 2
            R g[19];
            // planes z2 + 1, z2 and z2 - 1: phase 1 of iterations j, j - 1, j - 2
            const uint32_t sd = uj % ND, sm = (uj - 1) % NM, su = (uj - 2) % NU;
            // one address per class of c_z, at the first column of the neighbourhood:
            // every read is at a constant offset >= 0 from it
            const LT* const rd = &down[sd][0][col - 1 - TB_EX];
            const LT* const rm = &mid[sm][0][col - 1 - TB_EX];
            const LT* const ru = &up[su][0][col - 1 - TB_EX];
            static_for<19>([&](auto I) {
                constexpr int i = decltype(I)::value;
                constexpr int cz = cz_of(i);
                constexpr int o = zclass_index(i) * TB_E + (1 - cx_of(i)) + TB_EX * (1 - cy_of(i));
                if constexpr (cz < 0) g[i] = from_lds(rd[o]);
                else if constexpr (cz == 0) g[i] = from_lds(rm[o]);
                else g[i] = from_lds(ru[o]);
            });
            collide<R, k16>(g, Fpx, Fpy, Fpz, k, inv_s);
            refresh(off[1][1]);
            const PlaneStride out{(char*)plane_at(L.b, Z0 + (uint32_t)(j - 2)), opaque(pbytes)};
            static_for<19>([&](auto I) {
                constexpr int i = decltype(I)::value;
                *(LBM_GLOBAL_SPACE T*)(out(i) + off[1][1]) = enc<Cd>(g[i], store_s);
            });
        }
        Fpx = Fx;
        Fpy = Fy;
        Fpz = Fz;
        // With the rotating 16-bit slots, phase 1 of iteration j + 1 writes no
        // slot that phase 2 of iteration j reads, and phase 1 of j + 2 waits at
        // the barrier of j + 1 for every phase 2 of j: no second barrier.
        if constexpr (!k16) {
            __syncthreads();
            pull(j + 2, P);
        }
    };

    Pulled pa{}, pb{};
    if (forced) {
        if (row_writer) rowbuf[0][ey][lane] = row_coeff(0);
        __syncthreads();
    }
    pull(0, pa);
    pull(1, pb);    // niter >= 3, so plane 1 always exists
    for (int j = 0; j < niter; j += 2) {   // unrolled by two: pa, pb stay in registers
        iteration(j, pa);
        iteration(j + 1, pb);   // (past the last plane of an odd count: nothing stored)
    }
}

bool tb2_supported(int precision) { return precision != LBM_FP64; }

namespace {

// Tiles of a lattice along x and y.
template <class Tile>
std::pair<uint32_t, uint32_t> tiles_of(const LatticeArgs& L) {
    return {(L.nx + Tile::TX - 1) / Tile::TX, (L.ny + Tile::TY - 1) / Tile::TY};
}

// Compute units of the current device, asked once per device.
uint32_t compute_units() {
    static std::atomic<int> cus[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cus[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n <= 0)
            n = 256;
        cus[dev].store(n, std::memory_order_relaxed);
    }
    return (uint32_t)n;
}

// Plans are made once per (shape, grouping, CU count) and kept.
template <class Tile>
const Tb2Plan& plan_for(const LatticeArgs& L, uint32_t groups) {
    static std::mutex mu;
    static std::map<std::array<uint32_t, 5>, Tb2Plan> plans;
    const uint32_t cus = compute_units();
    const std::array<uint32_t, 5> key{L.nx, L.ny, L.nz, groups, cus};
    std::lock_guard<std::mutex> lock(mu);
    auto it = plans.find(key);
    if (it == plans.end())
        it = plans.emplace(key, make_plan(L.nx, L.ny, L.nz, tiles_of<Tile>(L).first,
                                          tiles_of<Tile>(L).second, groups, cus, Tile::TX,
                                          Tile::TY)).first;
    return it->second;
}

}  // namespace

template <class Cd, bool kHaloWave>
static hipError_t launch_tile(const LatticeArgs& L, const Tb2Plan& P, hipStream_t s) {
    using Tile = Tb2Tile<kHaloWave>;
    TB2Args A;
    A.L = L;
    A.tiles_x = tiles_of<Tile>(L).first;
    A.tiles_y = tiles_of<Tile>(L).second;
    A.W = P.w;
    const uint64_t nblocks = (uint64_t)P.w.groups * P.per_group;
    if (nblocks == 0 || nblocks > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_step_tb2<Cd, kHaloWave>), dim3((uint32_t)nblocks), dim3(Tile::kThreads),
                       0, s, A);
    return hipGetLastError();
}

template <class Cd>
static hipError_t launch_cd(const LatticeArgs& L, hipStream_t s) {
    // one tile range per XCD whenever a block order is asked for
    const uint32_t groups = L.xcd_remap ? 8u : 1u;
    constexpr uint32_t bytes = sizeof(typename Cd::T);
    const Tb2Plan& narrow = plan_for<Tb2Tile<false>>(L, groups);
    if (wide_possible(L.nx, L.ny, bytes)) {
        const Tb2Plan& wide = plan_for<Tb2Tile<true>>(L, groups);
        if (wide_tile(L.nx, L.ny, bytes, wide.makespan, narrow.makespan))
            return launch_tile<Cd, true>(L, wide, s);
    }
    return launch_tile<Cd, false>(L, narrow, s);
}

hipError_t launch_step_tb2(int precision, const LatticeArgs& L, hipStream_t s) {
    // one 1024-thread workgroup and 115-154 KB of LDS per CU (64 x 8 tiles, two
    // workgroups per CU, measured 25 % slower at 800^3)
    switch (precision) {
        case LBM_FP32: return launch_cd<CdF32>(L, s);
        case LBM_FP16_DEV: return launch_cd<CdF16>(L, s);
        case LBM_BF16_DEV: return launch_cd<CdBF16>(L, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace lbm
