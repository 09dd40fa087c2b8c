// fd4_kernels.hip -- the finite-difference reference solver of Sec. III on
// gfx950: fourth-order centred differences in space, the classic RK4 method
// in time, and the SEIRD reactions (Eqs. (EqSEIRD_S)-(EqSEIRD_D)) evaluated
// at every stage. It serves to validate the SSLBM on large grids and to
// time the comparison the paper makes; it is not on the SSLBM's path.
//
// With F the right-hand side and G = dt F, one step is
//   k1 = G(u), k2 = G(u + k1/2), k3 = G(u + k2/2), k4 = G(u + k3),
//   u' = u + (k1 + 2 k2 + 2 k3 + k4) / 6,
// G_C = (dl_C / 12) lap(rho_C) + Psi_C dt with dl = d dt / dx^2 and
// lap u = sum over the axes of -u(-2) + 16 u(-1) - 30 u + 16 u(+1) - u(+2).
// The stage inputs y2 = u + k1/2, y3 = u + k2/2, y4 = u + k3 hold the k's, so
// u' = (y2 + 2 y3 + y4 - u) / 3 + k4 / 6.
//
// One launch takes a whole step: a state is read once and written once, where
// a launch per stage moved 13 state-sized arrays. A workgroup of W wavefronts
// owns 64 columns x R W rows in registers, R rows a lane, of which the four
// stages use up a halo of 8 on every side (recomputed by the neighbouring
// tiles). East and west neighbours come through DPP wave shifts, north and
// south ones from the lane's own rows; only the two first and two last rows
// of each wavefront go through LDS, once a stage. Ghost cells are folded by
// the boundary's index map on loading: periodic wrap, or the even reflection
// about the wall of a no-flux boundary, which stays a reflection under a step.
//
// What bounds it: vector issue on the halo (a 48-row tile stores half of the
// cells it computes) rather than HBM (2048^2: 1.2-1.4 TB/s). Against one
// launch per stage, per step: 200^2 FP64 40.9 -> 8.8 us, FP32 36.0 -> 6.5;
// 2048^2 FP64 594 -> 245 us, FP32 225 -> 120 us. Taller tiles (60 to 96 rows,
// by more rows a lane or more wavefronts) were 4-15% slower in FP32: fewer
// wavefronts fit, and their barriers and loads no longer overlap.
#include <hip/hip_runtime.h>

#include "fd4_internal.h"
#include "seird_device.h"

namespace sslbm {

namespace {

constexpr int FD4_HALO = 8;  // four stages of a stencil that reaches two cells
constexpr int FD4_COLS = 64 - 2 * FD4_HALO;

// One field of a stage's input around a node: rows -2 .. 2 of its column.
template <typename T>
struct Column5 {
    T m2, m1, c, p1, p2;
};

template <typename T>
__device__ __forceinline__ T fd4_laplacian(const Column5<T> &v) {
    const T l1 = lane_from_left(v.c), r1 = lane_from_right(v.c);
    const T l2 = lane_from_left(l1), r2 = lane_from_right(r1);
    const T along_x = (T(16) * (l1 + r1) - (l2 + r2)) - T(30) * v.c;
    const T along_y = (T(16) * (v.m1 + v.p1) - (v.m2 + v.p2)) - T(30) * v.c;
    return along_x + along_y;
}

// The state of one lane: R rows of a column. y is the stage's input, u the
// state the step started from, acc = y2 + 2 y3 once both are known.
template <typename T, int R>
struct Fd4Lane {
    T u[5][R], y[5][R], acc[5][R];
};

// Rows a wavefront passes to its neighbours: its first two and last two rows
// of the diffusing fields.
template <typename T, int W, int F>
struct Fd4Edges {
    T row[W][4][F][64];
};

template <typename T, int R, int W, bool DD, int STAGE>
__device__ __forceinline__ void fd4_stage(Fd4Lane<T, R> &s, Fd4Edges<T, W, DD ? 5 : 4> &e,
                                          const Coef<T> &k, const T (&dl12)[5], int wave,
                                          int lane) {
    constexpr int F = DD ? 5 : 4;
    constexpr int RT = R * W;
    if constexpr (STAGE > 1)
        __syncthreads();  // the stage before has read its edges
#pragma unroll
    for (int c = 0; c < F; ++c) {
        e.row[wave][0][c][lane] = s.y[c][0];
        e.row[wave][1][c][lane] = s.y[c][1];
        e.row[wave][2][c][lane] = s.y[c][R - 2];
        e.row[wave][3][c][lane] = s.y[c][R - 1];
    }
    __syncthreads();
    // rows of this wavefront whose stage output is exact: [2 STAGE, RT - 2 STAGE)
    const int first = wave * R;
    if (first + R <= 2 * STAGE || first >= RT - 2 * STAGE)
        return;
    T above[F][2], below[F][2];
    const int up = wave > 0 ? wave - 1 : 0, down = wave < W - 1 ? wave + 1 : W - 1;
#pragma unroll
    for (int c = 0; c < F; ++c) {
        above[c][0] = e.row[up][2][c][lane];
        above[c][1] = e.row[up][3][c][lane];
        below[c][0] = e.row[down][0][c][lane];
        below[c][1] = e.row[down][1][c][lane];
    }
    // the two rows before the current one, as the stage's input had them
    T m2[F], m1[F];
#pragma unroll
    for (int c = 0; c < F; ++c) {
        m2[c] = above[c][0];
        m1[c] = above[c][1];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        T cen[5];
#pragma unroll
        for (int c = 0; c < 5; ++c)
            cen[c] = s.y[c][r];
        T fdt, rE, rI;
        seird_increments(cen[0], cen[1], cen[2], cen[3], k, fdt, rE, rI);
        const T src[5] = {-fdt, fdt - rE, rE - rI, k.kR * cen[2], k.kD * cen[2]};
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            T kc = src[c];
            if (c < F) {
                Column5<T> v;
                v.m2 = m2[c];
                v.m1 = m1[c];
                v.c = cen[c];
                v.p1 = r + 1 < R ? s.y[c][r + 1 < R ? r + 1 : 0] : below[c][0];
                v.p2 = r + 2 < R ? s.y[c][r + 2 < R ? r + 2 : 0] : below[c][r + 2 - R > 0];
                kc = fma(dl12[c], fd4_laplacian(v), src[c]);
                m2[c] = m1[c];
                m1[c] = cen[c];
            }
            if constexpr (STAGE == 1) {
                s.y[c][r] = fma(kc, T(0.5), cen[c]);
            } else if constexpr (STAGE == 2) {
                const T y3 = fma(kc, T(0.5), s.u[c][r]);
                s.acc[c][r] = cen[c] + T(2) * y3;
                s.y[c][r] = y3;
            } else if constexpr (STAGE == 3) {
                s.y[c][r] = kc + s.u[c][r];
            } else {
                const T sum = (s.acc[c][r] + cen[c]) - s.u[c][r];
                s.y[c][r] = fma(kc, T(1) / T(6), sum / T(3));
            }
        }
    }
}

template <typename T, int R, int W, bool DD>
__global__ __launch_bounds__(64 * W) void fd4_step_kernel(const T *__restrict__ in,
                                                          T *__restrict__ out, GridDesc g,
                                                          Coef<T> k, int tiles_x) {
    constexpr int RT = R * W, OUT = RT - 2 * FD4_HALO;
    __shared__ Fd4Edges<T, W, DD ? 5 : 4> edges;
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int tx = t % tiles_x, ty = t / tiles_x;
    const int x = tx * FD4_COLS + lane - FD4_HALO;
    const int y0 = ty * OUT - FD4_HALO + wave * R;
    const T dl12[5] = {k.dl[0] / T(12), k.dl[1] / T(12), k.dl[2] / T(12), k.dl[3] / T(12),
                       k.dl[4] / T(12)};
    Fd4Lane<T, R> s;
    const int xm = map_index(x, g.nx, g.bc);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const long long row = (long long)map_index(y0 + r, g.ny, g.bc) * g.nx;
#pragma unroll
        for (int c = 0; c < 5; ++c)
            s.u[c][r] = s.y[c][r] = in[c * g.plane + row + xm];
    }
    fd4_stage<T, R, W, DD, 1>(s, edges, k, dl12, wave, lane);
    fd4_stage<T, R, W, DD, 2>(s, edges, k, dl12, wave, lane);
    fd4_stage<T, R, W, DD, 3>(s, edges, k, dl12, wave, lane);
    fd4_stage<T, R, W, DD, 4>(s, edges, k, dl12, wave, lane);
    if (lane < FD4_HALO || lane >= 64 - FD4_HALO || x >= g.nx)
        return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int ry = wave * R + r;
        if (ry >= FD4_HALO && ry < RT - FD4_HALO && y0 + r < g.ny) {
            const long long cell = (long long)(y0 + r) * g.nx + x;
#pragma unroll
            for (int c = 0; c < 5; ++c)
                out[c * g.plane + cell] = s.y[c][r];
        }
    }
}


template <typename T, int R, int W, bool DD>
hipError_t launch_shape(const void *in, void *out, const GridDesc &g, const Coef<T> &k,
                        hipStream_t st) {
    constexpr int OUT = R * W - 2 * FD4_HALO;
    const int tiles_x = (g.nx + FD4_COLS - 1) / FD4_COLS;
    const long long tiles = (long long)tiles_x * ((g.ny + OUT - 1) / OUT);
    if (tiles > 0x7fffffffll)
        return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((fd4_step_kernel<T, R, W, DD>), dim3((unsigned)tiles), dim3(64 * W), 0, st,
                       static_cast<const T *>(in), static_cast<T *>(out), g, k, tiles_x);
    return hipGetLastError();
}

// Tile height: the lowest tile that still gives every CU no more than one
// (4 output rows; 200^2 FP64 8.8 us a step, 10.2 with 8 rows, 18.2 with 32),
// or two (8 rows; 400^2 FP64 19.1 us, 27.1 with 4 rows, 19.5 with 32); larger
// grids the tallest, which wastes least (2048^2 FP64: 245 us, 370 with 8). Grids
// of up to 4 and 16 rows take the lowest tile that holds them or half of them: a
// tile costs what its rows with the halo do (65536 columns, FP32 and FP64: 21 and
// 36 us a step for 4 output rows, 25 and 44 for 8, 61 and 95 for 32).
template <typename T, bool DD>
hipError_t launch_step(const void *in, void *out, const GridDesc &g, const Coef<T> &k, int cus,
                       hipStream_t st) {
    const long long strips = (g.nx + FD4_COLS - 1) / FD4_COLS;
    if (g.ny <= 4 || strips * ((g.ny + 3) / 4) <= cus)
        return launch_shape<T, 2, 10, DD>(in, out, g, k, st);
    if (g.ny <= 16 || strips * ((g.ny + 7) / 8) <= 2 * cus)
        return launch_shape<T, 3, 8, DD>(in, out, g, k, st);
    return launch_shape<T, 6, 8, DD>(in, out, g, k, st);
}

template <typename T>
hipError_t launch_t(void *rho, void *work, const GridDesc &g, const StepCoef &s, long long n,
                    hipStream_t st) {
    Coef<T> k;
    for (int c = 0; c < 5; ++c)
        k.dl[c] = (T)s.dl[c];
    k.bdt = (T)s.bdt;
    k.kE = (T)s.kE;
    k.kI = (T)s.kI;
    k.kR = (T)s.kR;
    k.kD = (T)s.kD;
    const int cus = compute_units();
    T *u = static_cast<T *>(rho), *w0 = static_cast<T *>(work), *w1 = w0 + 5 * g.plane;
    auto step = [&](const T *in, T *out) {
        return s.diffuse_d ? launch_step<T, true>(in, out, g, k, cus, st)
                           : launch_step<T, false>(in, out, g, k, cus, st);
    };
    // steps alternate between u and w0; an odd count takes three of them
    // around u, w0 and w1, so that the result ends in u (one step is copied)
    long long left = n;
    hipError_t e = hipSuccess;
    if (left % 2 == 1 && left >= 3) {
        e = step(u, w0);
        if (e == hipSuccess)
            e = step(w0, w1);
        if (e == hipSuccess)
            e = step(w1, u);
        left -= 3;
    }
    for (; left >= 2 && e == hipSuccess; left -= 2) {
        e = step(u, w0);
        if (e == hipSuccess)
            e = step(w0, u);
    }
    if (left == 1 && e == hipSuccess) {
        e = step(u, w0);
        if (e == hipSuccess)
            e = hipMemcpyAsync(u, w0, sizeof(T) * 5 * g.plane, hipMemcpyDeviceToDevice, st);
    }
    return e;
}

}  // namespace

hipError_t launch_fd4(int dtype, void *rho, void *work, const GridDesc &g, const StepCoef &k,
                      long long nsteps, hipStream_t s) {
    return dtype == SSLBM_F32 ? launch_t<float>(rho, work, g, k, nsteps, s)
                              : launch_t<double>(rho, work, g, k, nsteps, s);
}

}  // namespace sslbm
