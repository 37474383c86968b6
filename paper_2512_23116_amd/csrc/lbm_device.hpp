// lbm_device.hpp — device-side building blocks shared by the single-lattice
// kernels (lbm_kernels.hip) and the batched serving kernel (lbm_batch.hip):
// storage codecs, index decode with periodic neighbours, the AA / A-B access
// patterns, and the per-cell body force.
#pragma once

#include <math.h>

#include <type_traits>
#include <utility>

#include "d3q19_mrt.hpp"
#include "lbm_internal.hpp"

namespace lbm {

// --------------------------------------------------------------- codecs ---
struct CdF64 { using T = double;   using R = double; };
struct CdF32 { using T = float;    using R = float;  };
struct CdF16 { using T = _Float16; using R = float;  };
struct CdBF16 { using T = uint16_t; using R = float; };

// float -> bf16 with round-to-nearest-even.  gfx950 has a conversion
// instruction for it (v_cvt_pk_bf16_f32, emitted for this cast): one
// instruction where the integer rounding took six, bit-identical to it for
// every finite input (NaN stays NaN).
__device__ __forceinline__ uint16_t bf16_rne(float x) {
    const __bf16 h = (__bf16)x;
    return __builtin_bit_cast(uint16_t, h);
}

// Whether the one-step kernel collides on the stored scale (collide's kScaled),
// so that the 16-bit codecs reduce to conversions instead of a conversion and a
// multiplication each way (FP16: 19 VALU instructions per cell fewer).
template <class Cd>
constexpr bool kScaledCodec = sizeof(typename Cd::T) == 2;

template <class Cd>
__device__ __forceinline__ typename Cd::R dec(typename Cd::T v, typename Cd::R inv_s) {
    if constexpr (std::is_same_v<Cd, CdF16>) return (float)v * inv_s;
    else if constexpr (std::is_same_v<Cd, CdBF16>) return __uint_as_float((uint32_t)v << 16) * inv_s;
    else return v;
}
template <class Cd>
__device__ __forceinline__ typename Cd::T enc(typename Cd::R v, typename Cd::R s) {
    if constexpr (std::is_same_v<Cd, CdF16>) return (_Float16)(v * s);   // v_cvt_f16_f32: RNE
    else if constexpr (std::is_same_v<Cd, CdBF16>) return bf16_rne(v * s);
    else return v;
}

// ---------------------------------------------------------- small tools ---
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Offsets (in cells) from x to x-1, x+1, y-1, ... with periodic wrap.
struct Nbr {
    int32_t xm, xp, ym, yp, zm, zp;
};

struct CellPos {
    uint32_t x, y, z, row;   // row = y + ny z
};

__device__ __forceinline__ CellPos decode(uint32_t cell, const LatticeArgs& L) {
    CellPos p;
    p.row = fast_div(cell, L.mx);
    p.x = cell - p.row * L.nx;
    p.z = fast_div(p.row, L.my);
    p.y = p.row - p.z * L.ny;
    return p;
}

__device__ __forceinline__ Nbr make_nbr(const CellPos& p, const LatticeArgs& L) {
    Nbr n;
    const int32_t nx = (int32_t)L.nx, sy = (int32_t)L.nx, sz = (int32_t)L.nxy;
    n.xm = (p.x == 0) ? nx - 1 : -1;
    n.xp = (p.x == L.nx - 1) ? 1 - nx : 1;
    n.ym = (p.y == 0) ? ((int32_t)L.ny - 1) * sy : -sy;
    n.yp = (p.y == L.ny - 1) ? (1 - (int32_t)L.ny) * sy : sy;
    n.zm = (p.z == 0) ? ((int32_t)L.nz - 1) * sz : -sz;
    n.zp = (p.z == L.nz - 1) ? (1 - (int32_t)L.nz) * sz : sz;
    return n;
}

// Offset of the cell x - c_I.
template <int I>
__device__ __forceinline__ int32_t off_minus(const Nbr& n) {
    constexpr int cx = cx_of(I), cy = cy_of(I), cz = cz_of(I);
    int32_t o = 0;
    if constexpr (cx == 1) o += n.xm; else if constexpr (cx == -1) o += n.xp;
    if constexpr (cy == 1) o += n.ym; else if constexpr (cy == -1) o += n.yp;
    if constexpr (cz == 1) o += n.zm; else if constexpr (cz == -1) o += n.zp;
    return o;
}

// Runtime-direction variant (observation kernels only).
__device__ __forceinline__ int32_t off_minus_rt(int i, const Nbr& n) {
    const int cx = cx_of(i), cy = cy_of(i), cz = cz_of(i);
    int32_t o = 0;
    o += cx == 1 ? n.xm : (cx == -1 ? n.xp : 0);
    o += cy == 1 ? n.ym : (cy == -1 ? n.yp : 0);
    o += cz == 1 ? n.zm : (cz == -1 ? n.zp : 0);
    return o;
}

// Element index (slot * plane + cell) of the canonical f_i(x) for a runtime
// direction and pattern (set-up and observation kernels).
__device__ __forceinline__ uint64_t canon_index(int pat, int i, uint32_t cell, const Nbr& nb,
                                                uint64_t plane) {
    const int slot = (pat == PAT_AA_ODD) ? opp_of(i) : i;
    const uint32_t c = (pat == PAT_AA_EVEN) ? cell : cell + (uint32_t)off_minus_rt(i, nb);
    return (uint64_t)slot * plane + c;
}

// Block of cells of this workgroup in the XCD-aware order of L.xcd_remap, for a launch
// of one block per 256 cells (counted here: gridDim would be one more scalar load).
__device__ __forceinline__ uint32_t block_id(const LatticeArgs& L) {
    return block_order(blockIdx.x, (L.ncell + 255u) / 256u, L.xcd_remap);
}

// Plane addressing.  The 64-bit base of plane `slot` is uniform (SGPRs) and
// the per-lane part is a 32-bit byte offset (plane bytes < 2^32 is enforced at
// create), which maps to global loads and stores with a scalar base.  Two ways
// to get the plane base:
//  * PlaneTable: the 19 bases precomputed on the host, read from the kernel
//    arguments (no scalar arithmetic; used where they need not stay live across
//    a loop);
//  * PlaneStride: array base + slot * plane bytes (a few scalar instructions,
//    no extra SGPRs held; used by the z-marching two-step kernel).
// Both return pointers of the global address space, so that the accesses are
// global_load / global_store with a scalar base also where the compiler cannot see
// where the base comes from (the two-step kernel hides it; a generic pointer there
// costs a flat access and a 64-bit vector addition each).
#if defined(__HIP_DEVICE_COMPILE__)
#define LBM_GLOBAL_SPACE __attribute__((address_space(1)))
#else
#define LBM_GLOBAL_SPACE
#endif
struct PlaneTable {
    char* const* p;
    __device__ __forceinline__ LBM_GLOBAL_SPACE char* operator()(int slot) const {
        return (LBM_GLOBAL_SPACE char*)p[slot];
    }
};
struct PlaneStride {
    char* base;
    uint64_t bytes;
    __device__ __forceinline__ LBM_GLOBAL_SPACE char* operator()(int slot) const {
        return (LBM_GLOBAL_SPACE char*)(base + (uint64_t)slot * bytes);
    }
};

template <typename T, class Planes>
__device__ __forceinline__ LBM_GLOBAL_SPACE T* elem_ptr(const Planes& planes, int slot,
                                                        uint32_t c) {
    return (LBM_GLOBAL_SPACE T*)(planes(slot) + (uint32_t)(c * (uint32_t)sizeof(T)));
}

// Location of the pre-collision f_i(x) for pattern PAT: slot and cell.
//   AA_EVEN: (i, x)   AA_ODD: (opp i, x - c_i)   AB: (i, x - c_i)
template <class Cd, int PAT, bool kNT = false, class Planes>
__device__ __forceinline__ void load_cell(const Planes& planes, uint32_t cell,
                                          const Nbr& nb, typename Cd::R (&g)[19],
                                          typename Cd::R inv_s) {
    static_for<19>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int slot = (PAT == PAT_AA_ODD) ? opp_of(i) : i;
        const uint32_t c = (PAT == PAT_AA_EVEN) ? cell : cell + (uint32_t)off_minus<i>(nb);
        LBM_GLOBAL_SPACE const typename Cd::T* p = elem_ptr<const typename Cd::T>(planes, slot, c);
        if constexpr (kNT) g[i] = dec<Cd>(__builtin_nontemporal_load(p), inv_s);
        else g[i] = dec<Cd>(*p, inv_s);
    });
}

// Where the post-collision f*_i(x) goes for pattern PAT (the pattern the step
// reads with): AA_EVEN -> (opp i, x); AA_ODD -> (i, x + c_i); AB -> (i, x) of dst.
template <class Cd, int PAT, bool kNT = false, class Planes>
__device__ __forceinline__ void store_cell(const Planes& planes, uint32_t cell,
                                           const Nbr& nb, const typename Cd::R (&g)[19],
                                           typename Cd::R s) {
    static_for<19>([&](auto I) {
        constexpr int i = decltype(I)::value;
        constexpr int slot = (PAT == PAT_AA_EVEN) ? opp_of(i) : i;
        const uint32_t c = (PAT == PAT_AA_ODD) ? cell + (uint32_t)off_minus<opp_of(i)>(nb) : cell;
        LBM_GLOBAL_SPACE typename Cd::T* p = elem_ptr<typename Cd::T>(planes, slot, c);
        if constexpr (kNT) __builtin_nontemporal_store(enc<Cd>(g[i], s), p);
        else *p = enc<Cd>(g[i], s);
    });
}

template <typename R>
__device__ __forceinline__ const CollideConst<R>& collide_const(const LatticeArgs& L) {
    if constexpr (std::is_same_v<R, double>) return L.kd;
    else return L.kf;
}
template <typename R>
__device__ __forceinline__ R scale_of(const LatticeArgs& L) {
    if constexpr (std::is_same_v<R, double>) return L.sigma;
    else return L.sigma_f;
}
template <typename R>
__device__ __forceinline__ R inv_scale_of(const LatticeArgs& L) {
    if constexpr (std::is_same_v<R, double>) return L.inv_sigma;
    else return L.inv_sigma_f;
}

// Body force at a cell from the 15 coefficients of its row and the four harmonics of its
// x (s1, c1, s2, c2 = sin, cos of 2 pi x/nx and 4 pi x/nx):
// F = c0 + A1 s1 + B1 c1 + A2 s2 + B2 c2, in the explicit fused multiply-adds that every
// kernel that collides shares (see collide).
template <typename R>
__device__ __forceinline__ void force_sum(const R* rc, R s1, R c1, R s2, R c2, R& Fx, R& Fy,
                                          R& Fz) {
    Fx = mad(c2, rc[12], mad(s2, rc[9], mad(c1, rc[6], mad(s1, rc[3], rc[0]))));
    Fy = mad(c2, rc[13], mad(s2, rc[10], mad(c1, rc[7], mad(s1, rc[4], rc[1]))));
    Fz = mad(c2, rc[14], mad(s2, rc[11], mad(c1, rc[8], mad(s1, rc[5], rc[2]))));
}
template <typename R>
__device__ __forceinline__ void force_at(const LatticeArgs& L, const CellPos& p, R& Fx, R& Fy,
                                         R& Fz) {
    if (L.rowc == nullptr) {
        Fx = Fy = Fz = R(0);
        return;
    }
    const R* xt = (const R*)L.xtab + (uint64_t)p.x * 4;
    force_sum((const R*)L.rowc + (uint64_t)p.row * 16, xt[0], xt[1], xt[2], xt[3], Fx, Fy, Fz);
}

// The collision's constants, read before the populations are waited for, and the planes
// an A/B step stores to, read before the collision.  Left where they are first used,
// their scalar loads come after that wait, or between the collision and the stores, and
// add to the launch: 100^3 FP32 A/B then takes 23.95 us for either instead of 23.70,
// 129x127x130 AA 48.24 instead of 48.14 without the constants.  FP64 has no registers for
// the constants (k_step), and 16-bit storage, which has more conversions to hide behind,
// gains nothing from the planes (256^3 FP16 A/B 245.2 against 244.6).
__device__ __forceinline__ CollideConst<float> early(const CollideConst<float>& c) {
    CollideConst<float> k = c;
    asm volatile("" : "+s"(k.ea_sa), "+s"(k.ea_sd), "+s"(k.ea_r), "+s"(k.ea_u2), "+s"(k.ea_uF),
                      "+s"(k.ed_sa), "+s"(k.ed_sd), "+s"(k.ed_r), "+s"(k.ed_u2), "+s"(k.ed_uF));
    asm volatile("" : "+s"(k.pi_m), "+s"(k.pi_F), "+s"(k.o_s), "+s"(k.o_F),
                      "+s"(k.a_s), "+s"(k.a_F), "+s"(k.a_m), "+s"(k.w_tr), "+s"(k.c_tau),
                      "+s"(k.tau0), "+s"(k.rho0));
    return k;
}
__device__ __forceinline__ PlaneTable early(char* const* planes, char* (&held)[19]) {
#pragma unroll
    for (int i = 0; i < 19; ++i) held[i] = planes[i];
    asm volatile("" : "+s"(held[0]), "+s"(held[1]), "+s"(held[2]), "+s"(held[3]), "+s"(held[4]),
                      "+s"(held[5]), "+s"(held[6]), "+s"(held[7]), "+s"(held[8]), "+s"(held[9]));
    asm volatile("" : "+s"(held[10]), "+s"(held[11]), "+s"(held[12]), "+s"(held[13]),
                      "+s"(held[14]), "+s"(held[15]), "+s"(held[16]), "+s"(held[17]),
                      "+s"(held[18]));
    return PlaneTable{held};
}
__device__ __forceinline__ const CollideConst<double>& early(const CollideConst<double>& c) {
    return c;
}

// One cell of the fused stream-and-collide step (eq. mrt_les_guo): gather the
// 19 pre-collision populations of pattern PAT, collide, scatter.
// NT: bit 0 = non-temporal loads, bit 1 = non-temporal stores.
template <class Cd, int PAT, int NT = 0>
__device__ __forceinline__ void step_cell(const LatticeArgs& L, uint32_t cell) {
    using R = typename Cd::R;
    const CellPos p = decode(cell, L);
    const Nbr nb = make_nbr(p, L);
    constexpr bool kS = kScaledCodec<Cd>;
    const auto& k = early(collide_const<R>(L));
    R g[19];
    load_cell<Cd, PAT, (NT & 1) != 0>(PlaneTable{L.pa}, cell, nb, g,
                                      kS ? R(1) : inv_scale_of<R>(L));
    R Fx, Fy, Fz;
    force_at<R>(L, p, Fx, Fy, Fz);
    if constexpr (kS) {
        const R s = scale_of<R>(L);
        Fx *= s;
        Fy *= s;
        Fz *= s;
    }
    PlaneTable out{PAT == PAT_AB ? L.pb : L.pa};
    char* held[19];
    if constexpr (PAT == PAT_AB && std::is_same_v<Cd, CdF32>) out = early(L.pb, held);
    collide<R, kS>(g, Fx, Fy, Fz, k, inv_scale_of<R>(L));
    // Rebuild the store addresses from here: an empty register barrier on the
    // cell index keeps the compiler from holding 19 precomputed 64-bit store
    // addresses live across the collision (38 VGPRs), so stores use the same
    // scalar-base + 32-bit-offset form as the loads.
    uint32_t cs = cell;
    asm volatile("" : "+v"(cs));
    store_cell<Cd, PAT, (NT & 2) != 0>(out, cs, nb, g, kS ? R(1) : scale_of<R>(L));
}

}  // namespace lbm
