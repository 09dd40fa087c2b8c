// tile_kernels.hip -- the register-tile pass (tile_core.h) on one grid, and the
// choice of its tile height and steps per pass.
#include <hip/hip_runtime.h>

#include "tile_core.h"

namespace sslbm {

template <typename T, int R, bool DD>
__global__ __launch_bounds__(64 * TILE_WAVES) void sslbm_tile_kernel(const T *__restrict__ in,
                                                                     T *__restrict__ out,
                                                                     GridDesc g, Coef<T> k, int K,
                                                                     int tiles_x) {
    __shared__ TileEdges<T, DD> edges;
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    tile_pass<T, R, DD>(in, out, g, k, K, t % tiles_x * (64 - 2 * K),
                        t / tiles_x * (TILE_WAVES * R - 2 * K), edges);
}

// Tiles of an nx x ny grid at R rows a lane and K steps.
long long tile_count(int nx, int ny, int R, int K) {
    const int w = 64 - 2 * K, h = TILE_WAVES * R - 2 * K;
    return (long long)((nx + w - 1) / w) * ((ny + h - 1) / h);
}

namespace {

int compute_units() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1) {
        (void)hipGetLastError();
        cus = 256;
    }
    return cus;
}

// Time of one pass in us, from a fit to 1000 measured passes (48^2 to 1024^2,
// every R below, 1 to 17 steps; 6% rms in FP32, 12% in FP64): the launch, a
// step's barrier, a step's vector work (rows of the wavefronts that still have
// exact rows, per SIMD) and the loads and stores, the last two once for every
// round of tiles. The shape it prefers was the fastest measured one, or within
// 1% of it, at every size in the range.
// `rows` is the sum over the steps.
double pass_us(int dtype, int R, int K, int rows, long long tiles, int cus) {
    const bool f32 = dtype == SSLBM_F32;
    const double rounds = (double)((tiles + cus - 1) / cus);
    return f32 ? 1.38 + 0.310 * K + rounds * (0.0604 * rows + 0.768 * R)
               : 1.46 + 0.213 * K + rounds * (0.1274 * rows + 1.463 * R);
}

}  // namespace

TilePlan tile_plan(int dtype, const GridSize *sizes, int n, long long nsteps, bool fewest) {
    TilePlan best;
    // Up to where the march has enough rows for every SIMD, it waits for
    // memory (FP32 1152^2: 3.64 against 3.83 us a step, 1280^2 4.27 against
    // 4.2; FP64 640^2: 2.55 against 2.80, 704^2 3.58 against 3.21).
    const long long most = dtype == SSLBM_F32 ? 1400000 : 450000;
    long long cells = 0;
    for (int i = 0; i < n; ++i)
        cells += (long long)sizes[i].nx * sizes[i].ny * sizes[i].count;
    if (cells > most || nsteps <= 0)
        return best;
    const int cus = compute_units();
    constexpr int F32_ROWS[] = {2, 3, 4, 5, 7}, F64_ROWS[] = {1, 2, 3};
    const int *rows = dtype == SSLBM_F32 ? F32_ROWS : F64_ROWS;
    const int heights = dtype == SSLBM_F32 ? 5 : 3;
    double best_us = 0.0;
    // a pass takes no more steps than the run has
    const int deepest = nsteps < TILE_MAX_DEPTH ? (int)nsteps : TILE_MAX_DEPTH;
    for (int j = 0; j < heights; ++j) {
        const int R = rows[j];
        int busy[TILE_MAX_DEPTH + 1] = {};  // rows per SIMD of a pass of so many steps
        for (int s = 1; s <= deepest; ++s)
            busy[s] = busy[s - 1] + (TILE_WAVES - 2 * (s / R)) * R / 4;
        for (int K = 1; K <= deepest && 2 * K < TILE_WAVES * R; ++K) {
            long long tiles = 0;
            for (int i = 0; i < n; ++i)
                tiles += tile_count(sizes[i].nx, sizes[i].ny, R, K) * sizes[i].count;
            if (tiles > 0x7fffffffll)
                continue;
            const PassPlan p = fewest ? fewest_passes(nsteps, K) : plan_passes(nsteps, K);
            const int k = p.steps(0);
            const double us = (double)p.count * pass_us(dtype, R, k, busy[k], tiles, cus);
            if (best.rows == 0 || us < best_us) {
                best_us = us;
                best.rows = R;
                best.depth = K;
            }
        }
    }
    return best;
}

template <typename T, int R, bool DD>
static hipError_t launch_r(const void *in, void *out, const GridDesc &g, const StepCoef &s, int K,
                           hipStream_t st) {
    const long long tiles = tile_count(g.nx, g.ny, R, K);
    if (K < 1 || K > TILE_MAX_DEPTH || 2 * K >= TILE_WAVES * R || tiles > 0x7fffffffll)
        return hipErrorInvalidValue;
    const int w = 64 - 2 * K;
    hipLaunchKernelGGL((sslbm_tile_kernel<T, R, DD>), dim3((unsigned)tiles), dim3(64 * TILE_WAVES),
                       0, st, static_cast<const T *>(in), static_cast<T *>(out), g,
                       cast_coef<T>(s), K, (g.nx + w - 1) / w);
    return hipGetLastError();
}

template <bool DD>
static hipError_t launch_d(int dtype, const void *in, void *out, const GridDesc &g,
                           const StepCoef &k, int K, int R, hipStream_t s) {
    if (dtype == SSLBM_F32) {
        switch (R) {
        case 2: return launch_r<float, 2, DD>(in, out, g, k, K, s);
        case 3: return launch_r<float, 3, DD>(in, out, g, k, K, s);
        case 4: return launch_r<float, 4, DD>(in, out, g, k, K, s);
        case 5: return launch_r<float, 5, DD>(in, out, g, k, K, s);
        case 7: return launch_r<float, 7, DD>(in, out, g, k, K, s);
        default: return hipErrorInvalidValue;
        }
    }
    switch (R) {
    case 1: return launch_r<double, 1, DD>(in, out, g, k, K, s);
    case 2: return launch_r<double, 2, DD>(in, out, g, k, K, s);
    case 3: return launch_r<double, 3, DD>(in, out, g, k, K, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_tile(int dtype, const void *in, void *out, const GridDesc &g, const StepCoef &k,
                       int K, int R, hipStream_t s) {
    return k.diffuse_d ? launch_d<true>(dtype, in, out, g, k, K, R, s)
                       : launch_d<false>(dtype, in, out, g, k, K, R, s);
}

}  // namespace sslbm
