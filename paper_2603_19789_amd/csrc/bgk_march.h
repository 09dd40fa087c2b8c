// bgk_march.h -- K steps of the BGK scheme per pass over HBM.
//
// One wavefront owns 64 consecutive columns and walks a chunk of rows, as the
// SSLBM pass does (march_core.h). A row that arrives at level l (the state
// after l steps) collides at once; its post-collision populations are what
// the level keeps: the resting and the two x-moving ones, already shifted to
// the column they stream to (DPP wave shifts), and the y-moving ones that
// travel with the march, for two rows. The next row's populations that travel
// against the march complete the row before it at level l + 1. So a level
// holds 21 values per column (12 + 8 + rho^D), not three rows of 20.
//
// Walls are bounce-back, written where a population would have come from
// outside, so no ghost is ever collided: at the first and last column a lane
// takes its own reversed population, and at the first and last row the value
// is put in place of the one that streams in. Rows and columns beyond a wall
// are carried along with in-range data and never reach an output.
//
// Every population is formed by the same expressions as in the one-step
// kernel (bgk_sources, bgk_collided), so every depth gives the same bits.
//
// What bounds it: the 42 planes a pass streams. At 2048^2 a pass takes
// 195-235 us in FP32 (705 MB algorithmic) at two to seven steps, against
// 143 us for the one-step kernel, so the steps per pass decide: 143 us a step
// at one, 43 at five, 33 at seven. Eight steps spill (34 us with 140 B of
// scratch per lane). FP64 holds three steps in 256 VGPRs: 277 -> 120 us a
// step; four spill (184). Non-temporal stores cost 5-15%, non-temporal loads
// another 15%; a row pitch off the power of two changes nothing.
#pragma once

#include <hip/hip_runtime.h>

#include "march_core.h"

namespace sslbm {

template <typename T>
struct BgkCoef {
    Coef<T> k;
    T omega[4];  // 1 / tau for S, E, I, R
};

// D2Q5 weights, Sec. II.B
template <typename T>
__device__ __forceinline__ T weight(int i) {
    return i == 0 ? T(1) / T(3) : T(1) / T(6);
}

// Sources w_i multiplies of one node, and its densities, from its populations.
template <typename T>
__device__ __forceinline__ void bgk_sources(const T (&f)[4][5], const BgkCoef<T> &k, T (&rho)[4],
                                            T (&src)[4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        T s = f[c][0];
#pragma unroll
        for (int i = 1; i < 5; ++i)
            s += f[c][i];
        rho[c] = s;
    }
    T fdt, rE, rI;
    seird_increments(rho[0], rho[1], rho[2], rho[3], k.k, fdt, rE, rI);
    src[0] = -fdt;
    src[1] = fdt - rE;
    src[2] = rE - rI;
    src[3] = k.k.kR * rho[2];
}

// Collided population i of compartment c (Eq. pdf),
//   f + (w rho - f) / tau + w src.
// FP64 rounds every product. FP32 fuses the two additions (76 instead of 96
// vector instructions a node: 38.7 -> 33.2 us a step at 2048^2, seven steps
// per pass); its distance from FP64 is the same (mean over three inputs of
// the relative L2 error of the populations: 4.76e-7 before and after at
// 2048^2 x 40 steps, 1.05e-5 both at 600 x 500 x 300). w rho is rounded before
// f is taken off in both: near equilibrium the difference is then exact, while
// an fma would feed the error of the rounded weights into every step (4.9e-7).
__device__ __forceinline__ double bgk_collided(double f, double rho, double src,
                                               const BgkCoef<double> &k, int c, int i) {
    const double w = weight<double>(i);
    return f + (w * rho - f) * k.omega[c] + w * src;
}
__device__ __forceinline__ float bgk_collided(float f, float rho, float src,
                                              const BgkCoef<float> &k, int c, int i) {
    const float w = weight<float>(i);
    return fma(w, src, fma(w * rho - f, k.omega[c], f));
}

// Post-collision populations a level keeps of its latest row.
template <typename T>
struct BgkLevel {
    T rest[4];           // direction 0
    T xp[4], xm[4];      // directions 1 and 3, shifted to their destination column
    T along[4];          // direction that travels with the march, latest row
    T along_prev[4];     // the same of the row before
    T dead;
};

// Values that exist here, in registers: the compiler may not form them later
// or keep what they were formed from instead.
template <typename T>
__device__ __forceinline__ void pin(T &a, T &b, T &c, T &d, T &e) {
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(e));
}

// A copy in a register of its own. Without it the row that goes up takes over
// the level's registers and the level moves on to others, which costs every
// value a second register around the row loop (42 a level instead of 21).
__device__ __forceinline__ float copied(float v) {
    float r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ double copied(double v) {
    double r;
    asm volatile("v_mov_b64 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// One chunk of one strip. In the functions below, UP says that the march goes
// to decreasing rows, and EDGE that a no-flux wall touches the strip or the
// chunk (the others do without the selects).
template <typename T, int K>
struct BgkMarch {
    const T *__restrict__ f_in;
    const T *__restrict__ d_in;
    T *__restrict__ f_out;
    T *__restrict__ d_out;
    GridDesc g;
    BgkCoef<T> k;
    unsigned xoff;     // byte offset of this lane's memory column
    unsigned xout;     // byte offset of its output column
    bool out_col;      // the column is an output column of the strip
    bool at_left, at_right;
    int j0, dir, tend; // first level-0 row, its direction, number of level-0 rows
};

template <typename T>
struct BgkRow {
    T f[4][5];
    T dead;
};

// The 20 planes of a row lie plane elements apart. Their addresses are formed
// one after the other from the one before, behind an empty asm that keeps the
// compiler from forming all of them ahead: 42 row addresses do not fit the
// scalar registers, and spilling them cost 60 vector registers a level.
template <typename T>
__device__ __forceinline__ const T *next_plane(const T *p, long long plane) {
    p += plane;
    asm("" : "+s"(p));
    return p;
}
template <typename T>
__device__ __forceinline__ T *next_plane(T *p, long long plane) {
    p += plane;
    asm("" : "+s"(p));
    return p;
}

template <typename T, int K>
__device__ __forceinline__ void bgk_fetch(BgkRow<T> &r, const BgkMarch<T, K> &a, int t) {
    const long long row =
        (long long)__builtin_amdgcn_readfirstlane(map_index(a.j0 + a.dir * t, a.g.ny, a.g.bc)) *
        a.g.nx;
    const T *p = a.f_in + row;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            r.f[c][i] = *(const T *)((const char *)p + a.xoff);
            p = next_plane(p, a.g.plane);
        }
    r.dead = *(const T *)((const char *)(a.d_in + row) + a.xoff);
}

// Row number `row` of level L arrives in r: collide it, complete the row
// before it at level L + 1 (returned in r), and keep what its own completion
// needs.
template <typename T, int K, bool UP, bool EDGE>
__device__ __forceinline__ void bgk_level(BgkLevel<T> &s, BgkRow<T> &r, const BgkMarch<T, K> &a,
                                          int row) {
    constexpr int WITH = UP ? 4 : 2, AGAINST = UP ? 2 : 4;
    const bool enters = EDGE && row == (UP ? a.g.ny - 1 : 0);  // first row of the domain
    const bool left = EDGE && row == (UP ? -1 : a.g.ny);       // first row beyond it
    T rho[4], src[4];
    bgk_sources(r.f, a.k, rho, src);
    const T dead = fma(a.k.k.kD, rho[2], r.dead);
    r.dead = copied(s.dead);
    s.dead = dead;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        // one compartment after the other, so that what a level keeps is all
        // that is live between levels
        __builtin_amdgcn_sched_barrier(0);
        const T rest = copied(s.rest[c]), xp = copied(s.xp[c]), xm = copied(s.xm[c]);
        const T with = copied(s.along_prev[c]);
        const T against = bgk_collided(r.f[c][AGAINST], rho[c], src[c], a.k, c, AGAINST);
        const T east = bgk_collided(r.f[c][1], rho[c], src[c], a.k, c, 1);
        const T west = bgk_collided(r.f[c][3], rho[c], src[c], a.k, c, 3);
        s.rest[c] = bgk_collided(r.f[c][0], rho[c], src[c], a.k, c, 0);
        s.xp[c] = lane_from_left(east);
        s.xm[c] = lane_from_right(west);
        if constexpr (EDGE) {
            s.xp[c] = a.at_left ? west : s.xp[c];
            s.xm[c] = a.at_right ? east : s.xm[c];
        }
        T back = against;
        if constexpr (EDGE) {
            s.along_prev[c] = enters ? against : s.along[c];
            back = left ? s.along[c] : against;
        } else {
            s.along_prev[c] = s.along[c];
        }
        s.along[c] = bgk_collided(r.f[c][WITH], rho[c], src[c], a.k, c, WITH);
        r.f[c][0] = rest;
        r.f[c][1] = xp;
        r.f[c][3] = xm;
        r.f[c][WITH] = with;
        r.f[c][AGAINST] = back;
        pin(r.f[c][0], r.f[c][1], r.f[c][2], r.f[c][3], r.f[c][4]);
        pin(s.rest[c], s.xp[c], s.xm[c], s.along_prev[c], s.along[c]);
    }
}

template <typename T, int K>
__device__ __forceinline__ void bgk_store(const BgkRow<T> &r, const BgkMarch<T, K> &a, int row) {
    if (!a.out_col)
        return;
    const long long off = (long long)__builtin_amdgcn_readfirstlane(row) * a.g.nx;
    T *p = a.f_out + off;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            *(T *)((char *)p + a.xout) = r.f[c][i];
            p = next_plane(p, a.g.plane);
        }
    *(T *)((char *)(a.d_out + off) + a.xout) = r.dead;
}

// One level-0 row r (number t of the chunk) through the levels. The first 2K
// rows fill them; from then on every row yields an output row.
template <typename T, int K, bool UP, bool EDGE>
__device__ __forceinline__ void bgk_row(BgkLevel<T> (&lv)[K], BgkRow<T> &r,
                                        const BgkMarch<T, K> &a, int t) {
    const int row = a.j0 + a.dir * t;
#pragma unroll
    for (int l = 0; l < K; ++l) {
        bgk_level<T, K, UP, EDGE>(lv[l], r, a, row - a.dir * l);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (t >= 2 * K && t < a.tend)
        bgk_store(r, a, row - a.dir * K);
}

template <typename T, int K, bool UP, bool EDGE>
__device__ __forceinline__ void bgk_rows(const BgkMarch<T, K> &a) {
    BgkLevel<T> lv[K];
#pragma unroll
    for (int l = 0; l < K; ++l) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            lv[l].rest[c] = lv[l].xp[c] = lv[l].xm[c] = lv[l].along[c] = lv[l].along_prev[c] = T(0);
        lv[l].dead = T(0);
    }
    BgkRow<T> r0, r1;
    bgk_fetch(r0, a, 0);
    for (int t = 0; t < a.tend; t += 2) {
        bgk_fetch(r1, a, t + 1);
        bgk_row<T, K, UP, EDGE>(lv, r0, a, t);
        bgk_fetch(r0, a, t + 2);
        bgk_row<T, K, UP, EDGE>(lv, r1, a, t + 1);
    }
}

template <typename T, int K>
__global__ __launch_bounds__(BLOCK_THREADS) __attribute__((amdgpu_waves_per_eu(2)))
void bgk_march_kernel(const T *__restrict__ f_in, const T *__restrict__ d_in,
                      T *__restrict__ f_out, T *__restrict__ d_out, GridDesc g, BgkCoef<T> k,
                      int rows_per_wave, int strips, int total_waves) {
    const int wave = __builtin_amdgcn_readfirstlane(
        xcd_tile(blockIdx.x, gridDim.x) * WAVES_PER_BLOCK + (threadIdx.x >> 6));
    if (wave >= total_waves)
        return;  // whole wavefront leaves together
    const int strip = __builtin_amdgcn_readfirstlane(wave % strips);
    const int chunk = __builtin_amdgcn_readfirstlane(wave / strips);
    const int y0 = chunk * rows_per_wave, y1 = min(y0 + rows_per_wave, g.ny);
    const bool up = (chunk & 1) != 0;
    const int lane = threadIdx.x & 63;
    BgkMarch<T, K> a;
    a.f_in = f_in;
    a.d_in = d_in;
    a.f_out = f_out;
    a.d_out = d_out;
    a.g = g;
    a.k = k;
    const int x = strip * (64 - 2 * K) + lane - K;
    a.xoff = (unsigned)map_index(x, g.nx, g.bc) * (unsigned)sizeof(T);
    a.xout = (unsigned)x * (unsigned)sizeof(T);
    a.out_col = lane >= K && lane < 64 - K && x < g.nx;
    a.at_left = x == 0;
    a.at_right = x == g.nx - 1;
    a.dir = up ? -1 : 1;
    a.j0 = up ? y1 - 1 + K : y0 - K;
    a.tend = y1 - y0 + 2 * K;
    const bool edge =
        g.bc == SSLBM_NOFLUX && (y0 < K || y1 + K > g.ny ||
                                 __builtin_amdgcn_ballot_w64(a.at_left || a.at_right) != 0);
    if (up) {
        if (edge)
            bgk_rows<T, K, true, true>(a);
        else
            bgk_rows<T, K, true, false>(a);
    } else {
        if (edge)
            bgk_rows<T, K, false, true>(a);
        else
            bgk_rows<T, K, false, false>(a);
    }
}

}  // namespace sslbm
