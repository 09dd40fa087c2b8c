// tile_core.h -- steps of the SSLBM SEIRD update on a tile held in registers:
// the pass for grids that cannot give every SIMD of the GPU a long march
// (march_core.h).
//
// A workgroup of 16 wavefronts owns 64 columns x 16 R rows, R rows of a column
// a lane, and takes K steps of it between one read and one write of HBM; a
// halo of K cells on every side is recomputed by the neighbouring tiles. East
// and west neighbours come through DPP wave shifts, north and south ones from
// the lane's own rows; the first and last row of every wavefront go through
// LDS once a step, in two buffers by step parity, so that a step costs one
// barrier. K is a run-time number: nothing a lane holds depends on it.
//
// What bounds it: on the smallest grids the launch and the barriers (0.78 us a
// step), then vector issue. The march it replaces there waits for one row of
// loads after the other and computes K levels one after the other on one
// wavefront per SIMD. Per step against the best march shape: FP32 128^2
// 1.12 -> 0.78 us, 256^2 1.26 -> 0.87, 512^2 1.82 -> 1.33, 768^2 2.47 -> 1.89,
// 1024^2 3.22 -> 3.08; FP64 128^2 1.41 -> 1.07, 256^2 1.57 -> 1.30,
// 512^2 2.47 -> 2.11.
#pragma once

#include <hip/hip_runtime.h>

#include "march_core.h"

namespace sslbm {

template <typename T, bool DD>
struct TileEdges {
    T row[2][TILE_WAVES][2][DD ? 5 : 4][64];  // [step parity][wavefront][first, last row]
};

// K steps in -> out of the tile whose first output cell is (x0, y0), with the
// grid g and coefficients k. Every thread of the workgroup calls it.
template <typename T, int R, bool DD>
__device__ __forceinline__ void tile_pass(const T *__restrict__ in, T *__restrict__ out,
                                          const GridDesc &g, const Coef<T> &k, int K, int x0,
                                          int y0, TileEdges<T, DD> &e) {
    constexpr int F = DD ? 5 : 4, W = TILE_WAVES, RT = R * W;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int first = wave * R;
    const int x = x0 - K + lane, yl = y0 - K + first;
    T s[5][R];
    const int xm = map_index(x, g.nx, g.bc);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const long long row = (long long)map_index(yl + r, g.ny, g.bc) * g.nx;
#pragma unroll
        for (int c = 0; c < 5; ++c)
            s[c][r] = in[c * g.plane + row + xm];
    }
    const int up = wave > 0 ? wave - 1 : 0, down = wave < W - 1 ? wave + 1 : W - 1;
    for (int step = 1; step <= K; ++step) {
        const int p = step & 1;
#pragma unroll
        for (int c = 0; c < F; ++c) {
            e.row[p][wave][0][c][lane] = s[c][0];
            e.row[p][wave][1][c][lane] = s[c][R - 1];
        }
        __syncthreads();
        // a wavefront none of whose rows stays exact has nothing left to do
        // but to meet the others at the barrier
        if (first + R <= step || first >= RT - step)
            continue;
        T north[F], below[F];
#pragma unroll
        for (int c = 0; c < F; ++c) {
            north[c] = e.row[p][up][1][c][lane];
            below[c] = e.row[p][down][0][c][lane];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            T cen[5], nb[5], o[5];
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                cen[c] = s[c][r];
                if (c < F) {
                    const T south = r + 1 < R ? s[c][r + 1 < R ? r + 1 : 0] : below[c];
                    const T own[1] = {s[c][r]};
                    nb[c] = (north[c] + south) + east_west<T, 1>(own, 0);
                    north[c] = cen[c];
                } else {
                    nb[c] = T(0);
                }
            }
            seird_update<T, DD>(cen, nb, k, o);
#pragma unroll
            for (int c = 0; c < 5; ++c)
                s[c][r] = o[c];
        }
    }
    if (lane < K || lane >= 64 - K || x >= g.nx)
        return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = first + r;
        if (row >= K && row < RT - K && yl + r < g.ny) {
            const long long cell = (long long)(yl + r) * g.nx + x;
#pragma unroll
            for (int c = 0; c < 5; ++c)
                out[c * g.plane + cell] = s[c][r];
        }
    }
}

}  // namespace sslbm
