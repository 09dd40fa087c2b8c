// bgk_kernels.hip -- the BGK lattice Boltzmann comparison scheme on gfx950
// (Eq. pdf): collide the 20 populations of S, E, I, R with f^eq = w_i rho and
// the source w_i Psi dt, and stream each one to x + c_i (periodic wrap, or
// half-way bounce-back at a no-flux wall). Large grids take several steps per
// pass over HBM (bgk_march.h); single steps and small grids the kernel below:
// one thread per node reads its populations, collides and pushes. Rows of the
// grid lie on blockIdx.y (grids taller than the 65535 rows a launch can span
// take rows y, y + 65535, ... in one workgroup), so every population plane is
// read and written in coalesced 256-node row segments (the pushed ones shifted
// by one node). Stores keep the default cache policy: the pushed rows are
// shifted by one node, and L2 merges the partial lines (non-temporal stores
// measured 5% slower).
#include <hip/hip_runtime.h>

#include "bgk_march.h"

namespace sslbm {

constexpr int BGK_THREADS = 256;

// Most rows a launch spans (the grid's y dimension).
constexpr int BGK_MAX_GRID_ROWS = 65535;

// One node (x, y): collide and push.
template <typename T>
__device__ __forceinline__ void bgk_node(const T *__restrict__ f_in, const T *__restrict__ d_in,
                                         T *__restrict__ f_out, T *__restrict__ d_out,
                                         const GridDesc &g, const BgkCoef<T> &k, int x, int y) {
    const long long plane = g.plane;
    const long long cell = (long long)y * g.nx + x;

    T f[4][5], rho[4], src[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 5; ++i)
            f[c][i] = f_in[(c * 5 + i) * plane + cell];
    const T dead = d_in[cell];
    bgk_sources(f, k, rho, src);

    // destinations of the five links; at a no-flux wall the population
    // returns to this node in the opposite direction
    constexpr int CX[5] = {0, 1, 0, -1, 0};
    constexpr int CY[5] = {0, 0, 1, 0, -1};
    constexpr int OPP[5] = {0, 3, 4, 1, 2};
    long long dest[5];
    int dir[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        int xd = x + CX[i], yd = y + CY[i];
        dir[i] = i;
        const bool outside = xd < 0 || xd >= g.nx || yd < 0 || yd >= g.ny;
        if (outside && g.bc == SSLBM_NOFLUX) {
            xd = x;
            yd = y;
            dir[i] = OPP[i];
        } else if (outside) {
            xd = xd < 0 ? xd + g.nx : (xd >= g.nx ? xd - g.nx : xd);
            yd = yd < 0 ? yd + g.ny : (yd >= g.ny ? yd - g.ny : yd);
        }
        dest[i] = (long long)yd * g.nx + xd;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int i = 0; i < 5; ++i)
            f_out[(c * 5 + dir[i]) * plane + dest[i]] =
                bgk_collided(f[c][i], rho[c], src[c], k, c, i);
    }
    d_out[cell] = fma(k.k.kD, rho[2], dead);
}

template <typename T>
__global__ __launch_bounds__(BGK_THREADS) void bgk_step_kernel(const T *__restrict__ f_in,
                                                               const T *__restrict__ d_in,
                                                               T *__restrict__ f_out,
                                                               T *__restrict__ d_out, GridDesc g,
                                                               BgkCoef<T> k) {
    const int x = blockIdx.x * BGK_THREADS + threadIdx.x;
    if (x >= g.nx)
        return;
    for (int y = blockIdx.y; y < g.ny; y += gridDim.y)
        bgk_node(f_in, d_in, f_out, d_out, g, k, x, y);
}

template <typename T>
__global__ __launch_bounds__(BGK_THREADS) void bgk_init_kernel(const T *__restrict__ rho,
                                                               T *__restrict__ f,
                                                               T *__restrict__ rhoD, GridDesc g) {
    const long long plane = g.plane;
    const long long stride = (long long)gridDim.x * BGK_THREADS;
    for (long long cell = (long long)blockIdx.x * BGK_THREADS + threadIdx.x; cell < plane;
         cell += stride) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const T r = rho[c * plane + cell];
#pragma unroll
            for (int i = 0; i < 5; ++i)
                f[(c * 5 + i) * plane + cell] = weight<T>(i) * r;
        }
        rhoD[cell] = rho[4 * plane + cell];
    }
}

template <typename T>
__global__ __launch_bounds__(BGK_THREADS) void bgk_density_kernel(const T *__restrict__ f,
                                                                  const T *__restrict__ rhoD,
                                                                  T *__restrict__ rho, GridDesc g) {
    const long long plane = g.plane;
    const long long stride = (long long)gridDim.x * BGK_THREADS;
    for (long long cell = (long long)blockIdx.x * BGK_THREADS + threadIdx.x; cell < plane;
         cell += stride) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            T s = T(0);
#pragma unroll
            for (int i = 0; i < 5; ++i)
                s += f[(c * 5 + i) * plane + cell];
            rho[c * plane + cell] = s;
        }
        rho[4 * plane + cell] = rhoD[cell];
    }
}

template <typename T>
static BgkCoef<T> bgk_coef(const StepCoef &s) {
    BgkCoef<T> b;
    for (int c = 0; c < 5; ++c)
        b.k.dl[c] = (T)s.dl[c];
    b.k.bdt = (T)s.bdt;
    b.k.kE = (T)s.kE;
    b.k.kI = (T)s.kI;
    b.k.kR = (T)s.kR;
    b.k.kD = (T)s.kD;
    for (int c = 0; c < 4; ++c)
        b.omega[c] = (T)s.omega[c];
    return b;
}

// One thread per cell, at most 2^22 workgroups (2^30 work-items, within a
// launch's 32-bit work-item count); larger planes loop.
static dim3 plane_grid(const GridDesc &g) {
    const long long blocks = (g.plane + BGK_THREADS - 1) / BGK_THREADS;
    return dim3((unsigned)(blocks < (1ll << 22) ? blocks : (1ll << 22)));
}

hipError_t launch_bgk_step(int dtype, const void *f_in, const void *rhoD_in, void *f_out,
                           void *rhoD_out, const GridDesc &g, const StepCoef &k, hipStream_t s) {
    const dim3 grid((g.nx + BGK_THREADS - 1) / BGK_THREADS,
                    g.ny < BGK_MAX_GRID_ROWS ? g.ny : BGK_MAX_GRID_ROWS);
    if (dtype == SSLBM_F32)
        hipLaunchKernelGGL(bgk_step_kernel<float>, grid, dim3(BGK_THREADS), 0, s,
                           (const float *)f_in, (const float *)rhoD_in, (float *)f_out,
                           (float *)rhoD_out, g, bgk_coef<float>(k));
    else
        hipLaunchKernelGGL(bgk_step_kernel<double>, grid, dim3(BGK_THREADS), 0, s,
                           (const double *)f_in, (const double *)rhoD_in, (double *)f_out,
                           (double *)rhoD_out, g, bgk_coef<double>(k));
    return hipGetLastError();
}

// Deepest pass that fits 256 VGPRs without scratch (two wavefronts per SIMD).
template <typename T>
constexpr int BGK_MAX_DEPTH = sizeof(T) == 4 ? 7 : 3;

// Steps per pass. A pass of several steps needs a wavefront per SIMD and a
// few rows each to pay for its halo: from 384^2 on it is ahead (FP32 5.5 us a
// step against 5.8, FP64 7.9 against 9.7), at 256^2 behind (FP32 5.6 against
// 4.0, FP64 7.5 against 5.9), and a strip narrower than half a wavefront
// would compute mostly halo, as a single row would (150000 x 1, 42 steps: FP32
// 348 us against 231 of single steps, FP64 486 against 379; two rows are even).
// FP32 takes seven steps on grids large enough that HBM decides (1536^2: 22.0 us
// a step against 23.5 at five) and five below, where the halo does (1024^2: 12.9
// against 13.4).
int bgk_depth(int dtype, const GridDesc &g) {
    if (g.plane < 140000 || g.nx < 32 || g.ny < 2)
        return 1;
    if (dtype == SSLBM_F64)
        return BGK_MAX_DEPTH<double>;
    return g.plane < 1500000 ? 5 : BGK_MAX_DEPTH<float>;
}

// Rows per wavefront: one wavefront per SIMD on grids where that leaves
// chunks of at most 16 rows (512^2 at five steps: 6 rows 6.2 us a step, 3
// rows 8.5; 768^2: 12 rows 8.4, 6 rows 10.1), at least 6 of them; taller
// grids give every SIMD its two wavefronts (2048^2 at seven steps: 42 rows
// 33 us, 64 rows 43).
static int bgk_rows_per_wave(const GridDesc &g, int strips) {
    const int cus = compute_units();
    auto rows = [&](int waves) {
        const int chunks = waves / strips > 1 ? waves / strips : 1;
        return (g.ny + chunks - 1) / chunks;
    };
    const int one = rows(4 * cus);
    if (one <= 16)
        return one < 6 ? 6 : one;
    return rows(8 * cus);
}

template <typename T, int K>
static hipError_t launch_march_k(const void *f_in, const void *d_in, void *f_out, void *d_out,
                                 const GridDesc &g, const StepCoef &k, hipStream_t s) {
    constexpr int W = 64 - 2 * K;
    const int strips = (g.nx + W - 1) / W;
    const int rows = bgk_rows_per_wave(g, strips);
    const long long waves = (long long)strips * ((g.ny + rows - 1) / rows);
    if (waves > 0x7fffffffll - WAVES_PER_BLOCK)
        return hipErrorInvalidConfiguration;
    const unsigned blocks = (unsigned)((waves + WAVES_PER_BLOCK - 1) / WAVES_PER_BLOCK);
    hipLaunchKernelGGL((bgk_march_kernel<T, K>), dim3(blocks), dim3(BLOCK_THREADS), 0, s,
                       (const T *)f_in, (const T *)d_in, (T *)f_out, (T *)d_out, g,
                       bgk_coef<T>(k), rows, strips, (int)waves);
    return hipGetLastError();
}

// K steps, in -> out; K = 1 is the one-step kernel.
hipError_t launch_bgk_pass(int dtype, const void *f_in, const void *rhoD_in, void *f_out,
                           void *rhoD_out, const GridDesc &g, const StepCoef &k, int K,
                           hipStream_t s) {
    if (K == 1)
        return launch_bgk_step(dtype, f_in, rhoD_in, f_out, rhoD_out, g, k, s);
    if (dtype == SSLBM_F64) {
        switch (K) {
        case 2: return launch_march_k<double, 2>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
        case 3: return launch_march_k<double, 3>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
        default: return hipErrorInvalidValue;
        }
    }
    switch (K) {
    case 2: return launch_march_k<float, 2>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
    case 3: return launch_march_k<float, 3>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
    case 4: return launch_march_k<float, 4>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
    case 5: return launch_march_k<float, 5>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
    case 6: return launch_march_k<float, 6>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
    case 7: return launch_march_k<float, 7>(f_in, rhoD_in, f_out, rhoD_out, g, k, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_bgk_init(int dtype, const void *rho, void *f, void *rhoD, const GridDesc &g,
                           hipStream_t s) {
    if (dtype == SSLBM_F32)
        hipLaunchKernelGGL(bgk_init_kernel<float>, plane_grid(g), dim3(BGK_THREADS), 0, s,
                           (const float *)rho, (float *)f, (float *)rhoD, g);
    else
        hipLaunchKernelGGL(bgk_init_kernel<double>, plane_grid(g), dim3(BGK_THREADS), 0, s,
                           (const double *)rho, (double *)f, (double *)rhoD, g);
    return hipGetLastError();
}

hipError_t launch_bgk_density(int dtype, const void *f, const void *rhoD, void *rho,
                              const GridDesc &g, hipStream_t s) {
    if (dtype == SSLBM_F32)
        hipLaunchKernelGGL(bgk_density_kernel<float>, plane_grid(g), dim3(BGK_THREADS), 0, s,
                           (const float *)f, (const float *)rhoD, (float *)rho, g);
    else
        hipLaunchKernelGGL(bgk_density_kernel<double>, plane_grid(g), dim3(BGK_THREADS), 0, s,
                           (const double *)f, (const double *)rhoD, (double *)rho, g);
    return hipGetLastError();
}

}  // namespace sslbm
