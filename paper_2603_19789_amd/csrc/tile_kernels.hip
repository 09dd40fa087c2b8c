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

// Time of one pass in us, from a fit to 3000 measured passes (48^2 to 1180^2
// and grids 1 to 200 cells wide or high, every R below, 1 to 15 steps; 8% rms):
// the launch, a step's barrier, for every round of tiles its start and a step's
// vector work (`rows`: rows of the wavefronts that still have exact rows, per
// SIMD, summed over the steps), and the loads and stores of the tiles that run
// at once. Over those sizes the shape it prefers is within 2% of the fastest
// measured one on the mean.
static double pass_us(int dtype, int R, int K, int rows, long long tiles, int cus) {
    const double rounds = (double)((tiles + cus - 1) / cus);
    const double filled = tiles < cus ? (double)tiles / cus : 1.0;
    return dtype == SSLBM_F32
               ? 3.06 + 0.126 * K + rounds * (0.643 + 0.0720 * rows) + 0.429 * filled * R
               : 1.58 + 0.0644 * K + rounds * (2.01 + 0.1556 * rows) + 0.494 * filled * R;
}

// From a fit to 640 measured passes (grids and ensembles of up to 4 million
// cells, 1 to 10 wavefronts a SIMD; FP32 5% rms with one column a lane and 4%
// with two, FP64 7%): a wavefront computes H rows of every level and half of
// 2K more while they fill; the wavefronts of a SIMD share its issue slots, and
// the third and later ones start when others end, or crowd the caches.
double march_us(int dtype, int K, int cols_per_lane, int H, long long waves) {
    const int simds = 4 * compute_units();
    const double rows = (double)H * K + (double)K * K;
    const double share = (double)((waves + simds - 1) / simds);
    const double more = share > 2.0 ? share - 2.0 : 0.0;
    if (dtype == SSLBM_F64)
        return 1.98 + rows * (0.0889 + 0.0916 * share + 0.0570 * more);
    return cols_per_lane == 2 ? 4.38 + rows * (0.1135 + 0.0753 * share + 0.0516 * more)
                              : 2.35 + rows * (0.0768 + 0.0452 * share + 0.0116 * more);
}

TilePlan tile_plan(int dtype, const GridSize *sizes, int n, long long nsteps, bool fewest) {
    TilePlan best;
    // Beyond this many cells the march has enough rows for every SIMD (FP32
    // 1180^2: tiles 3.64 us a step, march 4.42, 1280^2 4.27 against 4.2; FP64
    // 670^2: 2.8 against 2.95, 704^2 3.58 against 3.21).
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
            if (best.rows == 0 || us < best.us) {
                best.rows = R;
                best.depth = K;
                best.us = us;
                best.few = tiles <= cus / 2;
            }
        }
    }
    return best;
}

// Runs of a few steps move the state at least twice for little work, so they
// have a fit of their own, with the cells read and written (in millions): 27
// grids of 64^2 to 1.4 million cells and at least 64 each way, 2 to 24 steps,
// 6% rms. With the faster of the two by these estimates, such runs are within
// 0.4% of the faster kind on the mean and 12% at most; with tiles wherever a
// long run takes them it was 7% and 45% (5 steps, FP32: 1500 x 901 30.1 us of
// tiles, 23.2 of marches; 1024^2 23.9 and 20.8; 768^2 16.2 and 14.7).
// Thin grids in FP64: 20 of them, 9% rms, with the cells that tiles and marches
// load; 1.3% on the mean and 26% at most, 7% and 67% by the long run (3 steps of
// 20000 x 13: 29.3 us of tiles, 18.7 of marches). In FP32 such a fit would send as
// many thin grids to the slower kind as it takes from it.
double short_tiles_us(int dtype, const GridSize *sizes, int n, int R, const PassPlan &plan,
                      bool thin) {
    const int cus = compute_units();
    long long cells = 0;
    for (int i = 0; i < n; ++i)
        cells += (long long)sizes[i].nx * sizes[i].ny * sizes[i].count;
    const double mega = 1e-6 * (double)cells;
    auto pass = [&](int k) {
        long long tiles = 0;
        for (int i = 0; i < n; ++i)
            tiles += tile_count(sizes[i].nx, sizes[i].ny, R, k) * sizes[i].count;
        int rows = 0;
        for (int s = 1; s <= k; ++s)
            rows += (TILE_WAVES - 2 * (s / R)) * R / 4;
        const double rounds = (double)((tiles + cus - 1) / cus);
        if (thin)
            return 0.22 + 0.46 * k + rounds * (1.64 + 0.133 * rows) +
                   1.36e-6 * (double)(tiles * 64 * TILE_WAVES * R) + 7.13 * mega;
        return dtype == SSLBM_F32 ? 2.46 + 0.289 * k + 0.075 * rounds * rows + 4.76 * mega
                                  : 0.295 * k + rounds * (3.0 + 0.139 * rows) + 8.31 * mega;
    };
    // (no pass is deeper than the tile allows)
    return (plan.longer ? (double)plan.longer * pass(plan.base + 1) : 0.0) +
           (double)(plan.count - plan.longer) * pass(plan.base);
}

double short_march_us(int dtype, int K, int cols_per_lane, int H, long long waves,
                      long long cells, bool thin) {
    const int simds = 4 * compute_units();
    const double rows = (double)H * K + (double)K * K, mega = 1e-6 * (double)cells;
    const double share = (double)((waves + simds - 1) / simds);
    if (thin)
        return 3.35 + rows * (0.053 + 0.074 * share + (share > 2.0 ? 0.072 * (share - 2.0) : 0.0)) +
               (double)waves * (0.72e-4 + 0.51e-6 * 64 * (H + 2 * K)) + 7.96 * mega;
    if (dtype == SSLBM_F64)
        return 2.94 + rows * (0.047 + 0.074 * share) + 7.97 * mega;
    return cols_per_lane == 2 ? 2.51 + rows * (0.137 + 0.007 * share) + 4.51 * mega
                              : 2.45 + rows * (0.060 + 0.039 * share) + 3.72 * mega;
}

bool tiles_pay(int dtype, const GridSize *sizes, int n, double march_us) {
    constexpr int LONG = 1000;
    return tile_plan(dtype, sizes, n, LONG).us <= 1.05 * LONG * march_us;
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
