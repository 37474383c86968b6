// lbm_analysis.hip — on-device turbulence diagnostics of the current state:
// the shell-binned kinetic-energy spectrum (Sec. 2.2, eq. integral_length_scale
// with the squared modulus), longitudinal structure functions / flatness
// (Sec. 5.3), and the turbulence scales of Sec. 2.2 (integral scale,
// dissipation, Kolmogorov and Taylor scales, energy balance terms).  All start
// from the velocity with the half-force shift (eq. guo_velocity) that
// lbm_moments returns, computed on the device in FP64.
#include <hipfft/hipfft.h>
#include <string.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <string>
#include <vector>

#include "lbm_device.hpp"
#include "lbm_observe.hpp"

namespace lbm {

constexpr int kAnaBlocks = 1024;

// The binning kernels below sum in a fixed order, so that a spectrum is the
// same bit for bit on every call: each wave of a block takes whole rows (fixed
// ky, kz) of the R2C output c[nz][ny][nx/2+1] in turn, 64 values of kx at a
// time, and adds into a histogram of its own in LDS in program order; the block
// then adds its waves' histograms in wave order (and k_sum_rows its blocks'
// partial sums in block order).  A block has 1 to 4 waves, as many as let their
// histograms fit 64 KB of LDS.

// Per-block partial sums of 1/2 w |c|^2 / n^2 over the shells 0..kmax, |c|^2
// summed over ncomp transforms stored cstride apart (the velocity components);
// w = 2 for the kx > 0 modes that stand for a conjugate pair.  Along a row the shell index
// never decreases with kx, so equal shells are contiguous runs of lanes: a
// segmented scan over the 64 lanes sums each run, and the run's last lane adds
// that sum to the wave's histogram (one lane per shell, no two lanes on one bin).
__global__ __launch_bounds__(256) void k_shell_bin(const hipfftDoubleComplex* c, uint64_t cstride,
                                                   int ncomp, uint32_t nx, uint32_t ny,
                                                   uint32_t nz, int kmax, double inv_n2,
                                                   double* partials) {
    extern __shared__ double hist[];   // [waves][kmax + 1]
    const int nb = kmax + 1, waves = (int)(blockDim.x >> 6);
    for (int k = threadIdx.x; k < waves * nb; k += blockDim.x) hist[k] = 0.0;
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
    double* wh = hist + wave * nb;
    const uint32_t hx = nx / 2 + 1;
    const uint64_t rows = (uint64_t)ny * nz;
    for (uint64_t row = (uint64_t)blockIdx.x * waves + wave; row < rows;
         row += (uint64_t)gridDim.x * waves) {
        const uint32_t iy = (uint32_t)(row % ny), iz = (uint32_t)(row / ny);
        const double ky = iy <= ny / 2 ? (double)iy : (double)iy - ny;
        const double kz = iz <= nz / 2 ? (double)iz : (double)iz - nz;
        const double kyz2 = ky * ky + kz * kz;
        const hipfftDoubleComplex* crow = c + row * hx;
        for (uint32_t x0 = 0; x0 < hx; x0 += 64) {
            const uint32_t ix = x0 + (uint32_t)lane;
            const bool in = ix < hx;
            const double kx = (double)ix;
            const int shell = in ? (int)floor(sqrt(kx * kx + kyz2) + 0.5) : INT_MAX;
            // the row's shells only grow: once lane 0 is past kmax, so is the rest
            if (__shfl(shell, 0, 64) > kmax) break;
            double v = 0.0;
            if (in && shell <= kmax) {
                const double w = (ix == 0 || (nx % 2 == 0 && ix == nx / 2)) ? 1.0 : 2.0;
                double e = 0.0;   // |u_hat|^2 summed over the ncomp components
                for (int q = 0; q < ncomp; ++q) {
                    const hipfftDoubleComplex z = crow[(uint64_t)q * cstride + ix];
                    e += z.x * z.x + z.y * z.y;
                }
                v = 0.5 * w * e * inv_n2;
            }
            for (int d = 1; d < 64; d <<= 1) {   // segmented inclusive scan over the runs
                const double vu = __shfl_up(v, d, 64);
                const int su = __shfl_up(shell, d, 64);
                if (lane >= d && su == shell) v += vu;
            }
            const int next = __shfl_down(shell, 1, 64);
            if (in && shell <= kmax && (lane == 63 || next != shell)) wh[shell] += v;
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nb; k += blockDim.x) {
        double s = hist[k];
        for (int w = 1; w < waves; ++w) s += hist[w * nb + k];
        partials[(uint64_t)blockIdx.x * nb + k] = s;
    }
}

// Per-block partial sums of w |c|^2 / n^2 binned by |k_x|, |k_y| and |k_z|
// separately (0..kmax each): partials[block][axis][k], axis 0, 1, 2 = x, y, z.
// w = 2 for the kx > 0 modes that stand for a conjugate pair (both members
// have the same |k_a|).  In a row every lane has its own |k_x| bin, and the
// whole row shares one |k_y| and one |k_z| bin: lane 0 adds the row's total,
// folded chunk by chunk over a fixed butterfly.  blockIdx.y takes the transform
// blockIdx.y * cstride on, into partials[blockIdx.y] of gridDim.x blocks each.
__global__ __launch_bounds__(256) void k_axis_bin(const hipfftDoubleComplex* c, uint64_t cstride,
                                                  uint32_t nx, uint32_t ny, uint32_t nz, int kmax,
                                                  double inv_n2, double* partials) {
    c += blockIdx.y * cstride;
    extern __shared__ double hist[];   // [waves][3][kmax + 1]
    const int nb = 3 * (kmax + 1), waves = (int)(blockDim.x >> 6);
    for (int k = threadIdx.x; k < waves * nb; k += blockDim.x) hist[k] = 0.0;
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
    double* wh = hist + wave * nb;
    const uint32_t hx = nx / 2 + 1;
    const uint64_t rows = (uint64_t)ny * nz;
    for (uint64_t row = (uint64_t)blockIdx.x * waves + wave; row < rows;
         row += (uint64_t)gridDim.x * waves) {
        const uint32_t iy = (uint32_t)(row % ny), iz = (uint32_t)(row / ny);
        const int ay = (int)(iy <= ny / 2 ? iy : ny - iy);
        const int az = (int)(iz <= nz / 2 ? iz : nz - iz);
        const hipfftDoubleComplex* crow = c + row * hx;
        double total = 0.0;
        for (uint32_t x0 = 0; x0 < hx; x0 += 64) {
            const uint32_t ix = x0 + (uint32_t)lane;
            double p = 0.0;
            if (ix < hx) {
                const double w = (ix == 0 || (nx % 2 == 0 && ix == nx / 2)) ? 1.0 : 2.0;
                const hipfftDoubleComplex z = crow[ix];
                p = w * (z.x * z.x + z.y * z.y) * inv_n2;
                if ((int)ix <= kmax) wh[ix] += p;
            }
            for (int d = 32; d > 0; d >>= 1) p += __shfl_xor(p, d, 64);
            total += p;
        }
        if (lane == 0) {
            if (ay <= kmax) wh[kmax + 1 + ay] += total;
            if (az <= kmax) wh[2 * (kmax + 1) + az] += total;
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nb; k += blockDim.x) {
        double s = hist[k];
        for (int w = 1; w < waves; ++w) s += hist[w * nb + k];
        partials[((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * nb + k] = s;
    }
}

// Threads per block of a binning kernel whose waves each keep `hist_bytes` of
// histogram: up to 4 waves within 64 KB of LDS.
static int bin_threads(size_t hist_bytes) {
    return 64 * (int)std::max<size_t>(1, std::min<size_t>(4, 65536 / hist_bytes));
}

// out[g][j] (+)= scale * sum over rows b of partials[g][b][j], one block per
// (column j, group g): thread t folds rows t, t + 256, ..., then a fixed tree
// over the block, so the order of the sum is the same on every call.
__global__ __launch_bounds__(256) void k_sum_rows(const double* partials, int rows, int cols,
                                                  double scale, int accumulate, double* out) {
    __shared__ double red[256];
    const int j = blockIdx.x;
    const double* p = partials + (uint64_t)blockIdx.y * rows * cols;
    double s = 0.0;
    for (int b = threadIdx.x; b < rows; b += 256) s += p[(uint64_t)b * cols + j];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double* o = out + (uint64_t)blockIdx.y * cols + j;
        *o = accumulate ? *o + red[0] * scale : red[0] * scale;
    }
}

// ------------------------------------------------ structure functions ---
// The velocity component along an axis is cut into tiles of `w` whole lines of that
// axis, held as tile[j][line], j along the axis: the separation r is then a shift by
// r * w elements, periodic over the tile.  A block loads a tile into LDS once and
// takes every separation from it; its 8 waves share out the separations, two to a
// wave, and what is left of the waves splits the elements.
constexpr int kStructRs = 16;          // separations of one launch
constexpr int kStructThreads = 512;
constexpr uint32_t kStructLine = 2048;

// One axis: lines of n elements, w of them to a tile.  Lines along y and z are grouped
// with their neighbours in x, `groups` tiles to a row of nx.
struct StructAxis {
    uint32_t n, w, groups;
};

struct StructArgs {
    const double* u;
    uint32_t nx, ny, nz;
    StructAxis ax[3];
    uint32_t first[4];           // ax[a]'s tiles are first[a] .. first[a + 1] - 1
    int32_t nr, pairs, share;    // separations; wave pairs (power of two); waves per pair
    uint32_t r[kStructRs];
};

__device__ __forceinline__ void struct_sums(double (&acc)[6], double du) {
    const double d2 = du * du, ad = fabs(du), d4 = d2 * d2;
    acc[0] += d2;
    acc[1] = fma(d2, du, acc[1]);
    acc[2] = fma(d2, ad, acc[2]);
    acc[3] += d4;
    acc[4] = fma(d4, ad, acc[4]);
    acc[5] = fma(d4, d2, acc[5]);
}

// Sums of du^2, du^3, |du|^3, du^4, |du|^5, du^6 for each separation over the three
// axes, du = u_a(x + r e_a) - u_a(x), periodic: one row of 6 per wave that shares a
// separation, partials[r][block][share].  Bound by the FP64 unit (9 instructions per
// axis, cell and separation) and, next, by LDS (1.5 reads).  Held to 8 waves, at the price
// of two spilled registers (with 6 the call took 823 us where this took 764).  256^3 with 14
// separations: 0.45 ms, of which 0.12 load the tiles; a thread per cell that read
// u[x + r] from memory for every separation took 1.27.
__global__ __launch_bounds__(kStructThreads)
__attribute__((amdgpu_waves_per_eu(8, 8))) void k_structure(StructArgs A, double* partials) {
    extern __shared__ double tile[];
    const uint32_t lane = threadIdx.x & 63u;
    const int wave = (int)(threadIdx.x >> 6);
    const int pair = wave & (A.pairs - 1), sub = wave / A.pairs;
    const int j0 = 2 * pair, j1 = j0 + 1;
    const bool live = j0 < A.nr;
    const uint32_t r0 = A.r[live ? j0 : 0], r1 = A.r[j1 < A.nr ? j1 : 0];
    double a0[6] = {0, 0, 0, 0, 0, 0}, a1[6] = {0, 0, 0, 0, 0, 0};
    const uint64_t nxy = (uint64_t)A.nx * A.ny, ncell = nxy * A.nz;
    for (uint32_t t = blockIdx.x; t < A.first[3]; t += gridDim.x) {
        const int a = t >= A.first[2] ? 2 : (t >= A.first[1] ? 1 : 0);
        const StructAxis& X = A.ax[a];
        const uint32_t i = t - A.first[a], n = X.n, w = X.w, total = n * w;
        const double* u = A.u + a * ncell;
        // element (j, line) of the tile at u[base + j * sj + line], along x at
        // u[base + line * n + j], line < lines
        uint64_t base, sj;
        uint32_t lines;
        if (a == 0) {
            base = (uint64_t)i * w * A.nx;
            sj = 1;
            const uint64_t left = (uint64_t)A.ny * A.nz - (uint64_t)i * w;
            lines = left < w ? (uint32_t)left : w;
        } else {
            const uint32_t row = i / X.groups, x0 = (i - row * X.groups) * w;
            base = x0 + (uint64_t)row * (a == 1 ? nxy : A.nx);
            sj = a == 1 ? A.nx : nxy;
            lines = A.nx - x0 < w ? A.nx - x0 : w;
        }
        __syncthreads();   // the last tile has been read
        if (a == 0) {
            for (uint32_t l = (uint32_t)wave; l < w; l += kStructThreads / 64)
                for (uint32_t j = lane; j < n; j += 64)
                    tile[j * w + l] = l < lines ? u[base + (uint64_t)l * n + j] : 0.0;
        } else {
            const uint32_t jn = kStructThreads / w, jt = threadIdx.x / w;
            const uint32_t l = threadIdx.x - jt * w;
            for (uint32_t j = jt < jn ? jt : n; j < n; j += jn)
                tile[j * w + l] = l < lines ? u[base + j * sj + l] : 0.0;
        }
        __syncthreads();
        if (!live) continue;
        const uint32_t s0 = r0 % n * w, s1 = r1 % n * w;
        // 4 x 64 elements at a time: a run that does not straddle the wrap is four
        // reads off one address
        for (uint32_t c = (uint32_t)sub * 256u; c < total; c += (uint32_t)A.share * 256u) {
            const uint32_t b0 = c + s0 >= total ? c + s0 - total : c + s0;
            const uint32_t b1 = c + s1 >= total ? c + s1 - total : c + s1;
            if (c + 256 <= total && b0 + 256 <= total && b1 + 256 <= total) {
#pragma unroll 2
                for (uint32_t k = 0; k < 4; ++k) {
                    const double v = tile[c + lane + 64 * k];
                    struct_sums(a0, tile[b0 + lane + 64 * k] - v);
                    struct_sums(a1, tile[b1 + lane + 64 * k] - v);
                }
            } else {
                for (uint32_t k = 0; k < 4; ++k) {
                    const uint32_t o = lane + 64 * k;
                    if (c + o >= total) break;
                    const double v = tile[c + o];
                    struct_sums(a0, tile[b0 + o >= total ? b0 + o - total : b0 + o] - v);
                    struct_sums(a1, tile[b1 + o >= total ? b1 + o - total : b1 + o] - v);
                }
            }
        }
    }
    if (!live) return;
    for (int m = 0; m < 6; ++m) {
        for (int o = 32; o > 0; o >>= 1) {
            a0[m] += __shfl_xor(a0[m], o, 64);
            a1[m] += __shfl_xor(a1[m], o, 64);
        }
    }
    if (lane == 0) {
        const uint64_t rows = (uint64_t)gridDim.x * A.share;
        const uint64_t row = (uint64_t)blockIdx.x * A.share + sub;
        for (int m = 0; m < 6; ++m) partials[((uint64_t)j0 * rows + row) * 6 + m] = a0[m];
        if (j1 < A.nr)
            for (int m = 0; m < 6; ++m) partials[((uint64_t)j1 * rows + row) * 6 + m] = a1[m];
    }
}

// The same sums for the separation r[blockIdx.y], each block a row of
// partials[r][block]: a thread per cell reads its neighbours along the axes from memory.
// For few separations (struct_direct), and for lines too long for LDS.
__global__ __launch_bounds__(256) void k_structure_direct(StructArgs A, DivMagic mx, DivMagic my,
                                                          double* partials) {
    __shared__ double red[4][6];
    const uint32_t r = A.r[blockIdx.y], rx = r % A.nx, ry = r % A.ny, rz = r % A.nz;
    const uint32_t nxy = A.nx * A.ny, ncell = nxy * A.nz;
    const double *ux = A.u, *uy = ux + ncell, *uz = uy + ncell;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (uint32_t c = blockIdx.x * 256u + threadIdx.x; c < ncell; c += gridDim.x * 256u) {
        const uint32_t row = fast_div(c, mx), z = fast_div(row, my);
        const uint32_t x = c - row * A.nx, y = row - z * A.ny;
        const uint32_t cx = x + rx >= A.nx ? c + rx - A.nx : c + rx;
        const uint32_t cy = y + ry >= A.ny ? c + ry * A.nx - nxy : c + ry * A.nx;
        const uint32_t cz = z + rz >= A.nz ? c + rz * nxy - ncell : c + rz * nxy;
        struct_sums(acc, ux[cx] - ux[c]);
        struct_sums(acc, uy[cy] - uy[c]);
        struct_sums(acc, uz[cz] - uz[c]);
    }
    for (int m = 0; m < 6; ++m) {
        for (int o = 32; o > 0; o >>= 1) acc[m] += __shfl_xor(acc[m], o, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][m] = acc[m];
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int m = (int)threadIdx.x;
        partials[((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * 6 + m] =
            red[0][m] + red[1][m] + red[2][m] + red[3][m];
    }
}

// The tiles of a lattice's three axes; returns the bytes of LDS they take.  A tile is 32
// KB (4 blocks to a CU) where that holds 128 bytes of every row (n <= 256), then up to
// 64 KB, in fewer lines from n = 512.  Lines of more than kStructLine elements take
// k_structure_direct: four of them would not fit.  Tiles along x hold an odd number of lines, so that the
// store that transposes them spreads over the LDS banks; along y and z a row is cut
// into equal tiles.
static size_t struct_plan(StructArgs& A) {
    const uint32_t len[3] = {A.nx, A.ny, A.nz};
    uint32_t most = 0;
    A.first[0] = 0;
    for (int a = 0; a < 3; ++a) {
        StructAxis& X = A.ax[a];
        X.n = len[a];
        uint32_t w = X.n <= 256 ? 4096 / X.n : (X.n <= 512 ? 16 : (X.n <= 1024 ? 8 : 4));
        w = std::min<uint32_t>(w, kStructThreads);
        // two blocks per CU at least, while a row of the tile keeps 64 bytes
        while (w > 8 && 3ull * A.nx * A.ny * A.nz < 512ull * X.n * w) w /= 2;
        if (a == 0) {
            X.w = w - (w % 2 == 0);
            X.groups = 1;
            A.first[1] = (uint32_t)(((uint64_t)A.ny * A.nz + X.w - 1) / X.w);
        } else {
            X.groups = (A.nx + w - 1) / w;
            X.w = (A.nx + X.groups - 1) / X.groups;
            A.first[a + 1] = A.first[a] + X.groups * (a == 1 ? A.nz : A.ny);
        }
        most = std::max(most, X.n * X.w);
    }
    return most * sizeof(double);
}

// Whether a launch of few separations reads the velocity from memory for each instead
// of going through LDS: a first separation takes 8 to 38 us less that way, and each
// further one adds its reads.  us per call at n^3, memory / LDS:
//   32^3  16 separations: 40.5/42.0       64^3   4: 49/52   5: 52/48
//   100^3  4: 69/70   5: 73/68            128^3  3: 86/89   4: 95/89
//   160^3  2: 138/144  3: 160/148         200^3  1: 216/240  2: 256/241
// Rows of at most 128 bytes fill the tiles of the other axes badly (nx = 4, ny = nz = 512,
// 8 separations: 78/92; nx = 8, 4 separations: 95/109).
static bool struct_direct(const StructArgs& A) {
    const uint64_t cells = (uint64_t)A.nx * A.ny * A.nz;
    if (A.nr == 1 || cells <= 40000) return true;
    if (A.nx < 16) return A.nr <= (A.nx < 8 ? 8 : 5);
    return A.nr <= 4 && (A.nr - 1) * cells <= 5000000;
}

}  // namespace lbm

using namespace lbm;

namespace {

const char* fft_error(hipfftResult r) {
    switch (r) {
        case HIPFFT_SUCCESS: return "success";
        case HIPFFT_ALLOC_FAILED: return "allocation failed";
        case HIPFFT_INVALID_VALUE: return "invalid value";
        case HIPFFT_INVALID_SIZE: return "invalid size";
        default: return "hipFFT error";
    }
}

lbm_status set_err(lbm_handle* h, lbm_status st, const std::string& m) {
    h->err = m;
    return st;
}

lbm_status hip_err(lbm_handle* h, hipError_t e, const char* what) {
    return set_err(h, e == hipErrorOutOfMemory ? LBM_ERR_OUT_OF_MEMORY : LBM_ERR_DEVICE,
                   std::string(what) + ": " + hipGetErrorString(e));
}

}  // namespace

namespace lbm {

struct AnalysisCache {
    unsigned long long* hist = nullptr;   // theta histogram counts
    size_t hist_elems = 0;
    double* u = nullptr;                  // [3][ncell] velocity, FP64
    hipfftDoubleComplex* c = nullptr;     // [nz][ny][nx/2+1] transform of one component
    size_t c_elems = 0;
    double* part = nullptr;               // per-block partial sums
    size_t part_elems = 0;
    double* out = nullptr;                // reduced results
    size_t out_elems = 0;
    hipfftHandle plan = nullptr;
    bool has_plan = false;
    hipfftHandle plan3 = nullptr;         // the three components in one batched call
    bool has_plan3 = false;
    // snapshot (lbm_snapshot_begin / _end): completion event, the device K_t
    // plane and the page-locked results
    hipEvent_t ev_snap = nullptr;
    float* d_plane = nullptr;
    double* h_sums = nullptr;        // kStatSums reduced sums
    double* h_E = nullptr;           // spectrum, h_E_elems
    size_t h_E_elems = 0;
    float* h_plane = nullptr;        // nx * ny
    bool snap_pending = false;
    int snap_kmax = 0;
    int64_t snap_steps = 0;
};

void release_analysis(AnalysisCache* a) {
    if (!a) return;
    if (a->ev_snap) {
        (void)hipEventSynchronize(a->ev_snap);
        (void)hipEventDestroy(a->ev_snap);
    }
    if (a->d_plane) (void)hipFree(a->d_plane);
    if (a->h_sums) (void)hipHostFree(a->h_sums);
    if (a->h_E) (void)hipHostFree(a->h_E);
    if (a->h_plane) (void)hipHostFree(a->h_plane);
    if (a->has_plan) (void)hipfftDestroy(a->plan);
    if (a->has_plan3) (void)hipfftDestroy(a->plan3);
    if (a->hist) (void)hipFree(a->hist);
    if (a->u) (void)hipFree(a->u);
    if (a->c) (void)hipFree(a->c);
    if (a->part) (void)hipFree(a->part);
    if (a->out) (void)hipFree(a->out);
    delete a;
}

}  // namespace lbm

namespace {

AnalysisCache& cache(lbm_handle* h) {
    if (!h->ana) h->ana = new AnalysisCache();
    return *h->ana;
}

// Grow a cached device buffer to at least n elements of T.
template <typename T>
hipError_t ensure(T*& p, size_t& have, size_t n) {
    if (p && have >= n) return hipSuccess;
    if (p) (void)hipFree(p);
    p = nullptr;
    have = 0;
    hipError_t e = hipMalloc((void**)&p, n * sizeof(T));
    if (e == hipSuccess) have = n;
    return e;
}

// Velocity (FP64, [3][ncell]) of the current state into the cached buffer.
lbm_status velocity(lbm_handle* h, const double** u) {
    AnalysisCache& a = cache(h);
    if (a.snap_pending)
        return set_err(h, LBM_ERR_STATE, "a snapshot is pending (lbm_snapshot_end first)");
    const size_t nc = h->args.ncell;
    if (!a.u) {
        hipError_t e = hipMalloc((void**)&a.u, 3 * nc * sizeof(double));
        if (e != hipSuccess) {
            a.u = nullptr;
            return hip_err(h, e, "hipMalloc(velocity)");
        }
    }
    hipError_t e = launch_moments(h->cfg.precision, current_pattern(h), current_args(h), nullptr,
                                  a.u, h->stream);
    if (e != hipSuccess) return hip_err(h, e, "moments kernel");
    *u = a.u;
    return LBM_OK;
}

// The handle's D2Z plan of its lattice (created on first use), bound to `stream`
// (the handle's stream by default).
lbm_status fft_plan(lbm_handle* h, AnalysisCache& a, hipStream_t stream) {
    if (!a.has_plan) {
        hipfftResult fr = hipfftPlan3d(&a.plan, (int)h->args.nz, (int)h->args.ny,
                                       (int)h->args.nx, HIPFFT_D2Z);
        if (fr != HIPFFT_SUCCESS)
            return set_err(h, LBM_ERR_DEVICE, std::string("hipfftPlan3d: ") + fft_error(fr));
        a.has_plan = true;
    }
    hipfftResult fr = hipfftSetStream(a.plan, stream);
    if (fr != HIPFFT_SUCCESS)
        return set_err(h, LBM_ERR_DEVICE, std::string("hipfftSetStream: ") + fft_error(fr));
    return LBM_OK;
}

// Lattices of up to 2^24 cells (256^3) transform the three velocity components in
// one batched call: at those sizes each transform's kernels are short and
// latency-bound, and batching them costs 16 bytes per cell more for the
// three-component transform buffer.  Larger lattices transform one component
// at a time into a one-component buffer, where the kernels are bandwidth-bound
// and the memory counts.
bool batched_fft(const lbm_handle* h) { return h->args.ncell <= (size_t(1) << 24); }

lbm_status fft_plan3(lbm_handle* h, AnalysisCache& a, hipStream_t stream) {
    if (!a.has_plan3) {
        const int nx = (int)h->args.nx, ny = (int)h->args.ny, nz = (int)h->args.nz;
        int n[3] = {nz, ny, nx}, inembed[3] = {nz, ny, nx}, onembed[3] = {nz, ny, nx / 2 + 1};
        const int idist = nz * ny * nx, odist = nz * ny * (nx / 2 + 1);
        hipfftResult fr = hipfftPlanMany(&a.plan3, 3, n, inembed, 1, idist, onembed, 1, odist,
                                         HIPFFT_D2Z, 3);
        if (fr != HIPFFT_SUCCESS)
            return set_err(h, LBM_ERR_DEVICE, std::string("hipfftPlanMany: ") + fft_error(fr));
        a.has_plan3 = true;
    }
    hipfftResult fr = hipfftSetStream(a.plan3, stream);
    if (fr != HIPFFT_SUCCESS)
        return set_err(h, LBM_ERR_DEVICE, std::string("hipfftSetStream: ") + fft_error(fr));
    return LBM_OK;
}

// Enqueue on `stream` the shell spectrum E[0..kmax] of the velocity u ([3][ncell])
// into a.out: the transforms, the per-block shell sums of each component and
// their fixed-order reduction.  a.c, a.part and a.out must be allocated
// (spectrum_buffers).
lbm_status enqueue_spectrum(lbm_handle* h, AnalysisCache& a, const double* u, int kmax,
                            hipStream_t stream) {
    const uint32_t nx = h->args.nx, ny = h->args.ny, nz = h->args.nz;
    const size_t nc = h->args.ncell, nmodes = (nx / 2 + 1) * (size_t)ny * nz;
    const bool batched = batched_fft(h);
    lbm_status st = batched ? fft_plan3(h, a, stream) : fft_plan(h, a, stream);
    if (st != LBM_OK) return st;
    const double inv_n2 = 1.0 / ((double)nc * (double)nc);
    const size_t shm = (size_t)(kmax + 1) * sizeof(double);
    const int bt = bin_threads(shm);
    hipfftResult fr = HIPFFT_SUCCESS;
    // batched: one binning pass sums the three components mode by mode;
    // otherwise each component's transform is binned and added in turn
    const int passes = batched ? 1 : 3, ncomp = batched ? 3 : 1;
    if (batched) fr = hipfftExecD2Z(a.plan3, (hipfftDoubleReal*)u, a.c);
    for (int c = 0; c < passes && fr == HIPFFT_SUCCESS; ++c) {
        if (!batched) {
            fr = hipfftExecD2Z(a.plan, (hipfftDoubleReal*)(u + (size_t)c * nc), a.c);
            if (fr != HIPFFT_SUCCESS) break;
        }
        hipLaunchKernelGGL(k_shell_bin, dim3(kAnaBlocks), dim3(bt), shm * (bt / 64), stream,
                           (const hipfftDoubleComplex*)a.c, (uint64_t)nmodes, ncomp, nx, ny, nz,
                           (int)kmax, inv_n2, a.part);
        hipLaunchKernelGGL(k_sum_rows, dim3(kmax + 1), dim3(256), 0, stream,
                           (const double*)a.part, kAnaBlocks, (int)(kmax + 1), 1.0, c > 0, a.out);
    }
    if (fr != HIPFFT_SUCCESS) return set_err(h, LBM_ERR_DEVICE, std::string("hipFFT: ") + fft_error(fr));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_err(h, e, "spectrum kernels");
    return LBM_OK;
}

// The transform buffer and the partial and reduced sums of a spectrum to kmax.
hipError_t spectrum_buffers(lbm_handle* h, AnalysisCache& a, int kmax) {
    const size_t nmodes = (h->args.nx / 2 + 1) * (size_t)h->args.ny * h->args.nz;
    hipError_t e = ensure(a.c, a.c_elems, batched_fft(h) ? 3 * nmodes : nmodes);
    if (e == hipSuccess) e = ensure(a.part, a.part_elems, (size_t)kAnaBlocks * (kmax + 1));
    if (e == hipSuccess) e = ensure(a.out, a.out_elems, (size_t)(kmax + 1));
    return e;
}

}  // namespace

extern "C" {

lbm_status lbm_spectrum(lbm_handle* h, int32_t kmax, double* E) {
    if (!h) return LBM_ERR_INVALID_ARG;
    if (!E || kmax < 0 || kmax > 4096) return set_err(h, LBM_ERR_INVALID_ARG, "kmax must be 0..4096");
    if (!h->initialized) return set_err(h, LBM_ERR_STATE, "state not initialised");
    const double* u = nullptr;
    lbm_status st = velocity(h, &u);
    if (st != LBM_OK) return st;
    AnalysisCache& a = cache(h);
    hipError_t e = spectrum_buffers(h, a, kmax);
    if (e != hipSuccess) return hip_err(h, e, "hipMalloc(spectrum)");
    st = enqueue_spectrum(h, a, u, kmax, h->stream);
    if (st != LBM_OK) return st;
    const size_t shm = (size_t)(kmax + 1) * sizeof(double);
    e = hipMemcpyAsync(E, a.out, shm, hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_err(h, e, "spectrum");
    return LBM_OK;
}

lbm_status lbm_snapshot_begin(lbm_handle* h, int32_t kmax, int32_t z) {
    if (!h) return LBM_ERR_INVALID_ARG;
    if (kmax < 0 || kmax > 4096) return set_err(h, LBM_ERR_INVALID_ARG, "kmax must be 0..4096");
    if (z < 0 || (uint32_t)z >= h->args.nz) return set_err(h, LBM_ERR_INVALID_ARG, "z outside 0..nz-1");
    if (!h->initialized) return set_err(h, LBM_ERR_STATE, "state not initialised");
    AnalysisCache& a = cache(h);
    if (a.snap_pending) return set_err(h, LBM_ERR_STATE, "a snapshot is already pending");
    const size_t nc = h->args.ncell, nxy = h->args.nxy;
    // buffers, created on first use and kept until lbm_destroy
    hipError_t e = hipSuccess;
    if (!a.u) e = hipMalloc((void**)&a.u, 3 * nc * sizeof(double));
    if (e == hipSuccess) e = spectrum_buffers(h, a, kmax);
    if (e == hipSuccess && !a.d_plane) e = hipMalloc((void**)&a.d_plane, nxy * sizeof(float));
    if (e == hipSuccess && !a.h_sums) e = hipHostMalloc((void**)&a.h_sums, kDiagSlots * sizeof(double), hipHostMallocDefault);
    if (e == hipSuccess && !a.h_plane) e = hipHostMalloc((void**)&a.h_plane, nxy * sizeof(float), hipHostMallocDefault);
    if (e == hipSuccess && a.h_E_elems < (size_t)kmax + 1) {
        if (a.h_E) (void)hipHostFree(a.h_E);
        a.h_E = nullptr;
        a.h_E_elems = 0;
        e = hipHostMalloc((void**)&a.h_E, ((size_t)kmax + 1) * sizeof(double), hipHostMallocDefault);
        if (e == hipSuccess) a.h_E_elems = (size_t)kmax + 1;
    }
    if (e == hipSuccess && !a.ev_snap) e = hipEventCreateWithFlags(&a.ev_snap, hipEventDisableTiming);
    if (e != hipSuccess) return hip_err(h, e, "snapshot buffers");
    // everything on the handle's stream, in order with the steps: the state reads,
    // the transforms of the velocity and the copies to page-locked memory
    double* sums = nullptr;
    e = launch_stats(h, &sums);
    const int pat = current_pattern(h);
    const LatticeArgs args = current_args(h);
    if (e == hipSuccess) e = launch_ktslice(h->cfg.precision, pat, args, (uint32_t)z, a.d_plane, h->stream);
    if (e == hipSuccess) e = launch_moments(h->cfg.precision, pat, args, nullptr, a.u, h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(a.h_sums, sums, kStatSums * sizeof(double), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(a.h_plane, a.d_plane, nxy * sizeof(float), hipMemcpyDeviceToHost, h->stream);
    if (e != hipSuccess) return hip_err(h, e, "snapshot (state reads)");
    lbm_status st = enqueue_spectrum(h, a, a.u, kmax, h->stream);
    if (st != LBM_OK) return st;
    const size_t shm = (size_t)(kmax + 1) * sizeof(double);
    e = hipMemcpyAsync(a.h_E, a.out, shm, hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipEventRecord(a.ev_snap, h->stream);
    if (e != hipSuccess) return hip_err(h, e, "snapshot (spectrum)");
    a.snap_pending = true;
    a.snap_kmax = kmax;
    a.snap_steps = h->steps;
    return LBM_OK;
}

lbm_status lbm_snapshot_end(lbm_handle* h, lbm_stats* stats, double* E, float* kt_plane) {
    if (!h) return LBM_ERR_INVALID_ARG;
    AnalysisCache* a = h->ana;
    if (!a || !a->snap_pending) return set_err(h, LBM_ERR_STATE, "no snapshot is pending");
    a->snap_pending = false;
    const hipError_t e = hipEventSynchronize(a->ev_snap);
    if (e != hipSuccess) return hip_err(h, e, "snapshot");
    if (E) memcpy(E, a->h_E, ((size_t)a->snap_kmax + 1) * sizeof(double));
    if (kt_plane) memcpy(kt_plane, a->h_plane, h->args.nxy * sizeof(float));
    if (stats) {
        fill_stats(h, a->h_sums, a->snap_steps, stats);
        if (stats->n_nonfinite > 0)
            return set_err(h, LBM_ERR_UNSTABLE, std::to_string(stats->n_nonfinite) + " non-finite cells");
    }
    return LBM_OK;
}

lbm_status lbm_theta_histogram(lbm_handle* h, double lo, double hi, int32_t nbins,
                               int64_t* counts) {
    if (!h) return LBM_ERR_INVALID_ARG;
    if (!counts || nbins < 1 || nbins > 4096)
        return set_err(h, LBM_ERR_INVALID_ARG, "nbins must be 1..4096 and counts non-NULL");
    if (!(std::isfinite(lo) && std::isfinite(hi) && hi > lo))
        return set_err(h, LBM_ERR_INVALID_ARG, "need finite lo < hi");
    if (!h->initialized) return set_err(h, LBM_ERR_STATE, "state not initialised");
    AnalysisCache& a = cache(h);
    const size_t n = (size_t)nbins + 3;
    hipError_t e = ensure(a.hist, a.hist_elems, n);
    if (e == hipSuccess) e = hipMemsetAsync(a.hist, 0, n * sizeof(unsigned long long), h->stream);
    if (e == hipSuccess)
        e = launch_theta_hist(h->cfg.precision, current_pattern(h), current_args(h), lo,
                              (double)nbins / (hi - lo), (int)nbins, a.hist, h->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(counts, a.hist, n * sizeof(int64_t), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_err(h, e, "theta histogram");
    return LBM_OK;
}

lbm_status lbm_spectra_1d(lbm_handle* h, int32_t kmax, double* E, double* ic) {
    if (!h) return LBM_ERR_INVALID_ARG;
    if (!E || kmax < 0 || kmax > 2048) return set_err(h, LBM_ERR_INVALID_ARG, "kmax must be 0..2048");
    if (!h->initialized) return set_err(h, LBM_ERR_STATE, "state not initialised");
    const uint32_t nx = h->args.nx, ny = h->args.ny, nz = h->args.nz;
    if (ic && (ny != nx || nz != nx))
        return set_err(h, LBM_ERR_INVALID_ARG, "the isotropy coefficient needs a cubic lattice");
    const size_t nc = h->args.ncell, nmodes = (nx / 2 + 1) * (size_t)ny * nz;
    const int cols = 3 * (kmax + 1);
    const double* u = nullptr;
    lbm_status st = velocity(h, &u);
    if (st != LBM_OK) return st;
    AnalysisCache& a = cache(h);
    // one call for the three transforms and one for each sum over them (32^3 111 ->
    // 45 us, 128^3 222 -> 153, 240^3 885 -> 857); from 2^24 cells a component at a time,
    // whose sums fold what is still in the cache (256^3 1110 us, batched 1130).  The
    // handle keeps the partial sums: past 16 MB for the three (kmax 226) the components'
    // sums take turns in one component's
    const bool batched = h->args.ncell < (size_t(1) << 24);
    const size_t part = (size_t)kAnaBlocks * cols;
    const int together = batched && 3 * part * sizeof(double) <= (size_t(16) << 20) ? 3 : 1;
    hipError_t e = ensure(a.c, a.c_elems, (batched ? 3 : 1) * nmodes);
    if (e == hipSuccess) e = ensure(a.part, a.part_elems, together * part);
    if (e == hipSuccess) e = ensure(a.out, a.out_elems, (size_t)3 * cols);
    if (e != hipSuccess) return hip_err(h, e, "hipMalloc(one-dimensional spectra)");
    st = batched ? fft_plan3(h, a, h->stream) : fft_plan(h, a, h->stream);
    if (st != LBM_OK) return st;
    const double inv_n2 = 1.0 / ((double)nc * (double)nc);
    const size_t hb = (size_t)cols * sizeof(double);
    const int bt = bin_threads(hb);
    hipfftResult fr = HIPFFT_SUCCESS;
    for (int c = 0; c < 3 && fr == HIPFFT_SUCCESS; c += together) {
        if (!batched)
            fr = hipfftExecD2Z(a.plan, (hipfftDoubleReal*)(u + (size_t)c * nc), a.c);
        else if (c == 0)
            fr = hipfftExecD2Z(a.plan3, (hipfftDoubleReal*)u, a.c);
        if (fr != HIPFFT_SUCCESS) break;
        hipLaunchKernelGGL(k_axis_bin, dim3(kAnaBlocks, together), dim3(bt), hb * (bt / 64), h->stream,
                           (const hipfftDoubleComplex*)a.c + (batched ? c * nmodes : 0),
                           (uint64_t)nmodes, nx, ny, nz, (int)kmax, inv_n2, a.part);
        hipLaunchKernelGGL(k_sum_rows, dim3(cols, together), dim3(256), 0, h->stream,
                           (const double*)a.part, kAnaBlocks, cols, 1.0, 0,
                           a.out + (size_t)c * cols);
    }
    if (fr != HIPFFT_SUCCESS) return set_err(h, LBM_ERR_DEVICE, std::string("hipFFT: ") + fft_error(fr));
    e = hipGetLastError();
    if (e == hipSuccess)
        e = hipMemcpyAsync(E, a.out, (size_t)3 * cols * sizeof(double), hipMemcpyDeviceToHost,
                           h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_err(h, e, "one-dimensional spectra");
    if (ic) {
        // App. spectral isotropy, with the isotropic relation between the
        // longitudinal and transverse spectra: IC = (E_L - k dE_L/dk) / (2 E_T),
        // E_L / E_T the means of the 3 longitudinal / 6 transverse spectra, the
        // slope k dE_L/dk = E_L dln E_L / dln k by a central difference in
        // log-log space; NaN where it is undefined.
        std::vector<double> EL(kmax + 1), ET(kmax + 1);
        const size_t K = (size_t)kmax + 1;
        for (size_t k = 0; k < K; ++k) {
            // E[c][a][k] at E[(3 c + a) K + k]
            EL[k] = (E[0 * K + k] + E[4 * K + k] + E[8 * K + k]) / 3.0;
            ET[k] = (E[3 * K + k] + E[6 * K + k] + E[1 * K + k] + E[7 * K + k] + E[2 * K + k] +
                     E[5 * K + k]) / 6.0;
        }
        for (size_t k = 0; k < K; ++k) {
            ic[k] = NAN;
            if (k >= 2 && k + 1 < K && EL[k + 1] > 0.0 && EL[k - 1] > 0.0 && ET[k] > 0.0) {
                const double slope = (log(EL[k + 1]) - log(EL[k - 1])) /
                                     (log((double)k + 1.0) - log((double)k - 1.0));
                ic[k] = (EL[k] - EL[k] * slope) / (2.0 * ET[k]);
            }
        }
    }
    return LBM_OK;
}

lbm_status lbm_structure_functions(lbm_handle* h, const int32_t* rs, int32_t nr, double* out) {
    if (!h) return LBM_ERR_INVALID_ARG;
    if (nr < 1 || nr > 65535 || !rs || !out) return set_err(h, LBM_ERR_INVALID_ARG, "bad rs/nr/out");
    for (int j = 0; j < nr; ++j)
        if (rs[j] < 1) return set_err(h, LBM_ERR_INVALID_ARG, "separations must be >= 1");
    if (!h->initialized) return set_err(h, LBM_ERR_STATE, "state not initialised");
    const double* u = nullptr;
    lbm_status st = velocity(h, &u);
    if (st != LBM_OK) return st;
    StructArgs A{};
    A.u = u;
    A.nx = h->args.nx;
    A.ny = h->args.ny;
    A.nz = h->args.nz;
    const bool tiled = std::max(A.nx, std::max(A.ny, A.nz)) <= kStructLine;
    const size_t shm = tiled ? struct_plan(A) : 0;
    constexpr int kWaves = kStructThreads / 64;
    AnalysisCache& a = cache(h);
    hipError_t e = ensure(a.part, a.part_elems, (size_t)kAnaBlocks * kWaves * 2 * 6);
    if (e == hipSuccess) e = ensure(a.out, a.out_elems, (size_t)nr * 6);
    if (e != hipSuccess) return hip_err(h, e, "hipMalloc(structure functions)");
    for (int j = 0; j < nr && e == hipSuccess; j += kStructRs) {
        A.nr = std::min(nr - j, kStructRs);
        A.pairs = 1;
        while (2 * A.pairs < A.nr) A.pairs *= 2;
        A.share = kWaves / A.pairs;
        for (int k = 0; k < A.nr; ++k) A.r[k] = (uint32_t)rs[j + k];
        int rows;
        if (tiled && !struct_direct(A)) {
            const int nb = (int)std::min<uint32_t>(kAnaBlocks, A.first[3]);
            rows = nb * A.share;
            hipLaunchKernelGGL(k_structure, dim3(nb), dim3(kStructThreads), shm, h->stream, A,
                               a.part);
        } else {
            rows = (int)std::min<uint32_t>(kAnaBlocks, (h->args.ncell + 255) / 256);
            hipLaunchKernelGGL(k_structure_direct, dim3(rows, A.nr), dim3(256), 0, h->stream, A,
                               h->args.mx, h->args.my, a.part);
        }
        // rows of 6 sums per (r, row): reduce the rows of each r in a fixed order
        hipLaunchKernelGGL(k_sum_rows, dim3(6, A.nr), dim3(256), 0, h->stream,
                           (const double*)a.part, rows, 6, 1.0 / (3.0 * h->args.ncell), 0,
                           a.out + (size_t)j * 6);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(out, a.out, (size_t)nr * 6 * sizeof(double),
                                            hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_err(h, e, "structure functions");
    return LBM_OK;
}

lbm_status lbm_turbulence(lbm_handle* h, int32_t kmax, lbm_turbulence_stats* out) {
    if (!h) return LBM_ERR_INVALID_ARG;
    if (!out) return set_err(h, LBM_ERR_INVALID_ARG, "out is NULL");
    const uint32_t N = h->args.nx;
    if (h->args.ny != N || h->args.nz != N)
        return set_err(h, LBM_ERR_INVALID_ARG, "turbulence scales need a cubic lattice");
    const int32_t kall = (int32_t)(0.5 * sqrt(3.0) * N + 1.0);   // every shell present
    if (kmax <= 0 || kmax > kall) kmax = kall;
    if (kmax > 4096) return set_err(h, LBM_ERR_INVALID_ARG, "lattice too large for the spectrum");
    std::vector<double> E((size_t)kmax + 1);
    lbm_status st = lbm_spectrum(h, kmax, E.data());
    if (st != LBM_OK) return st;
    lbm_stats s;
    st = lbm_kt_stats(h, &s);
    if (st != LBM_OK) return st;
    // Sec. 2.2 with the shell index k of the N-cell box as the wavenumber
    // kappa = 2 pi k / N in lattice units; the mean flow (k = 0) is excluded.
    const double nu0 = (h->cfg.tau0 - 0.5) / 3.0;
    double e = 0.0, e_over_k = 0.0, k2e = 0.0;
    for (int32_t k = 1; k <= kmax; ++k) {
        const double kap = 2.0 * M_PI * k / N;
        e += E[k];
        e_over_k += E[k] / kap;
        k2e += kap * kap * E[k];
    }
    memset(out, 0, sizeof *out);
    out->kmax = kmax;
    out->energy = s.energy;
    out->energy_spec = e;
    out->u_rms = sqrt(2.0 * e / 3.0);                        // eq. rms_velocity
    out->integral_scale = e > 0.0 ? 0.75 * M_PI * e_over_k / e : NAN;   // eq. integral_length_scale
    out->eps_spec = 2.0 * nu0 * k2e;                          // eq. dissipation_rate
    out->eps_strain = nu0 * s.strain2;                        // 2 nu0 <S:S>
    out->eps_sgs = s.nut_strain2;
    out->injection = s.injection;                             // <F.u>
    const double eps = out->eps_spec;
    out->eta = eps > 0.0 ? pow(nu0 * nu0 * nu0 / eps, 0.25) : NAN;          // eq. kolmogorov_scale
    out->taylor = eps > 0.0 ? sqrt(15.0 * nu0 * out->u_rms * out->u_rms / eps) : NAN;  // eq. taylor_microscale
    out->re_lambda = out->u_rms * out->taylor / nu0;
    // isotropy: Reynolds stresses of the fluctuations about the mean velocity
    const double* m = s.u_mean;
    const double R[3][3] = {
        {s.uu[0] - m[0] * m[0], s.uu[3] - m[0] * m[1], s.uu[4] - m[0] * m[2]},
        {s.uu[3] - m[0] * m[1], s.uu[1] - m[1] * m[1], s.uu[5] - m[1] * m[2]},
        {s.uu[4] - m[0] * m[2], s.uu[5] - m[1] * m[2], s.uu[2] - m[2] * m[2]}};
    const double tr = R[0][0] + R[1][1] + R[2][2];
    double b[3][3];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) b[i][j] = tr > 0.0 ? R[i][j] / tr - (i == j ? 1.0 / 3.0 : 0.0) : NAN;
    double b2 = 0.0, b3 = 0.0;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            b2 += b[i][j] * b[j][i];
            for (int k = 0; k < 3; ++k) b3 += b[i][j] * b[j][k] * b[k][i];
        }
    for (int i = 0; i < 3; ++i) out->energy_frac[i] = tr > 0.0 ? R[i][i] / tr : NAN;
    out->b[0] = b[0][0]; out->b[1] = b[1][1]; out->b[2] = b[2][2];
    out->b[3] = b[0][1]; out->b[4] = b[0][2]; out->b[5] = b[1][2];
    out->II_b = -0.5 * b2;
    out->III_b = b3 / 3.0;
    out->lumley_xi = cbrt(0.5 * out->III_b);
    out->lumley_eta = sqrt(fmax(0.0, -out->II_b / 3.0));
    return LBM_OK;
}

}  // extern "C"
