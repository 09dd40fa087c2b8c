// sslbm_internal.h -- declarations shared by the host API and the kernel
// translation units of libsslbm.so (not installed, not part of the ABI).
#pragma once

#include <hip/hip_runtime_api.h>

#include <vector>

#include "sslbm.h"

namespace sslbm {

// Grid description passed by value to every kernel.
struct GridDesc {
    int nx, ny;
    long long plane;  // nx * ny
    int bc;           // SSLBM_PERIODIC or SSLBM_NOFLUX
};

// Per-step constants, derived once on the host in FP64 and rounded to the
// arithmetic type at launch:
//   dl[C] = d[C] dt / dx^2 (lattice diffusivity, tau = 1/2 + 3 dl),
//   bdt = beta dt, kE = alpha dt, kI = gamma dt,
//   kR = (1 - phi) gamma dt, kD = phi gamma dt   (Eq. sources, Eq. rhoD),
//   omega[C] = 1 / tau[C] (BGK collision frequency).
struct StepCoef {
    double dl[5];
    double bdt, kE, kI, kR, kD;
    double omega[4];
    bool diffuse_d;  // d[4] != 0
};

// Launch shape of the y-marching kernel.
struct MarchShape {
    int rows_per_wave;  // output rows each wavefront produces
    int cols_per_lane;  // adjacent columns per lane: 1 or 2
};

// ---- host helpers (sslbm_api.cpp) ---------------------------------------
// Validate parameters and derive the per-step constants (SSLBM status code).
sslbm_status derive_coef(const sslbm_params *p, StepCoef *k);
// How a run of nsteps splits into passes of at most K steps: the fewest
// passes, made even where that leaves every pass a step (so that ping-pong
// buffers end where they started), with the steps spread as evenly as possible over them (the
// first `longer` passes take one step more than the rest). A pass costs
// about the same HBM traffic whatever its depth, so a short tail pass would
// waste most of one.
struct PassPlan {
    long long count = 0;   // passes
    int base = 0;          // steps of the shorter passes
    long long longer = 0;  // passes with base + 1 steps (the first ones)
    int steps(long long i) const { return i < longer ? base + 1 : base; }
};
PassPlan plan_passes(long long nsteps, int K);
// The same without a pass more to make their number even.
PassPlan fewest_passes(long long nsteps, int K);

// One pass of k steps (1 <= k <= the register limit), in -> out, with the
// context's pass shape (SSLBM status code).
sslbm_status run_pass(sslbm_ctx *c, const void *in, void *out, int k, hipStream_t s);
// One pass of 4 steps in -> out writing the state after 2 steps to mid.
sslbm_status run_pass_mid2(sslbm_ctx *c, const void *in, void *mid, void *out, hipStream_t s);

// ---- launchers (sslbm_kernels.hip) --------------------------------------
// K steps in one pass: in -> out (no overlap). K in 1..SSLBM_MAX_BLOCKING.
hipError_t launch_march(int dtype, const void *in, void *out, const GridDesc &g,
                        const StepCoef &k, int K, const MarchShape &shape, hipStream_t s);
// Largest steps-per-pass whose kernel fits the register budget.
int march_max_depth(int dtype, int cols_per_lane);
// A pass of K steps in -> out that also writes the state after MID steps to
// mid (no overlap among the three); K = 4, MID = 2 only (else
// hipErrorNotSupported).
hipError_t launch_march_mid(int dtype, const void *in, void *mid, void *out, const GridDesc &g,
                            const StepCoef &k, int K, int MID, const MarchShape &shape,
                            hipStream_t s);
// Output columns of one wavefront strip at K steps per pass.
int strip_width(int K, int cols_per_lane);
// Wavefronts of the K-step pass kernel resident on the current device at
// once (occupancy x CUs), 0 when no device can be queried.
int march_resident_waves(int dtype, int K, int cols_per_lane, bool diffuse_d);

// ---- register tiles (tile_kernels.hip) -----------------------------------
// Wavefronts of a tile's workgroup: a tile has 64 columns x TILE_WAVES R rows.
constexpr int TILE_WAVES = 16;
// Most steps a tile takes in one pass (its halo leaves 32 of 64 columns).
constexpr int TILE_MAX_DEPTH = 16;
// Tile height (rows a lane) and steps per pass for a run of nsteps on grids of
// n sizes that advance together; rows = 0: the grids are too large, march.
struct TilePlan {
    int rows = 0;
    int depth = 0;
    double us = 0.0;   // estimated time of the run
    bool few = false;  // so few tiles that half of the CUs hold them
};
struct GridSize {
    int nx, ny;
    int count;  // grids of this size
};
// The passes of such a run are plan_passes' (an even number), or with
// fewest = true as few as the depth allows.
TilePlan tile_plan(int dtype, const GridSize *sizes, int n, long long nsteps, bool fewest = false);
long long tile_count(int nx, int ny, int R, int K);
// Estimated time in us of one march pass of K steps by `waves` wavefronts of H
// rows, on grids small enough for tiles.
double march_us(int dtype, int K, int cols_per_lane, int H, long long waves);
// Whether a long run on n grid sizes is faster with tiles than with marches of
// march_us a step (asked where tiles are not few: runs of every length then take
// the same kind of pass).
bool tiles_pay(int dtype, const GridSize *sizes, int n, double march_us);
// Runs of up to so many steps are estimated by themselves: the time in us of the
// tile passes `plan` over n grid sizes, and of one march pass over grids of so
// many cells. Grids of fewer than SHORT_RUN_SIDE cells one way (`thin`) have an
// estimate in FP64 only.
constexpr int SHORT_RUN = 24, SHORT_RUN_SIDE = 64;
double short_tiles_us(int dtype, const GridSize *sizes, int n, int R, const PassPlan &plan,
                      bool thin = false);
double short_march_us(int dtype, int K, int cols_per_lane, int H, long long waves,
                      long long cells, bool thin = false);
// Compute units of the current device (256 where it cannot be asked).
int compute_units();
// K steps in -> out (no overlap) with R rows a lane.
hipError_t launch_tile(int dtype, const void *in, void *out, const GridDesc &g, const StepCoef &k,
                       int K, int R, hipStream_t s);

// ---- segments of a recorded run (sslbm_api.cpp) ---------------------------
// n >= 1 steps from one buffer to another: the passes' shape, which a caller
// with many segments of the same length works out once, and the segment.
struct SegmentShape {
    TilePlan tiles;  // rows = 0: a march
    int depth = 0;   // most steps a pass
};
SegmentShape segment_shape(const sslbm_ctx *c, long long n);
// src -> dst in the fewest passes, through tmp0 and tmp1 (states of their own;
// src, dst, tmp0 and tmp1 do not overlap, except that tmp1 may be dst).
sslbm_status run_segment(sslbm_ctx *c, const SegmentShape &shape, const void *src, void *dst,
                         void *tmp0, void *tmp1, long long n, hipStream_t s);

// ---- launchers (bgk_kernels.hip) ----------------------------------------
hipError_t launch_bgk_init(int dtype, const void *rho, void *f, void *rhoD, const GridDesc &g,
                           hipStream_t s);
hipError_t launch_bgk_step(int dtype, const void *f_in, const void *rhoD_in, void *f_out,
                           void *rhoD_out, const GridDesc &g, const StepCoef &k, hipStream_t s);
// Steps per pass bgk_run takes on this grid, and one pass of K steps.
int bgk_depth(int dtype, const GridDesc &g);
hipError_t launch_bgk_pass(int dtype, const void *f_in, const void *rhoD_in, void *f_out,
                           void *rhoD_out, const GridDesc &g, const StepCoef &k, int K,
                           hipStream_t s);
hipError_t launch_bgk_density(int dtype, const void *f, const void *rhoD, void *rho,
                              const GridDesc &g, hipStream_t s);

// ---- launchers (reduce_kernels.hip) -------------------------------------
// Number of partial blocks the total reduction uses (partials: blocks x 5 doubles).
int total_blocks(const GridDesc &g);
hipError_t launch_total(int dtype, const void *rho, const GridDesc &g, double *partials,
                        int blocks, double *out5_device, hipStream_t s);

}  // namespace sslbm

// The state behind the opaque sslbm_ctx handle.
struct sslbm_ctx {
    int nx = 0, ny = 0, dtype = 0, bc = 0;
    sslbm_params p{};
    sslbm::StepCoef coef{};
    sslbm_launch launch{};  // requested pass shape; zero fields = automatic
    sslbm_launch tuned{};   // march shape the tuner found, reported while launch is all automatic
    int last_hip = 0;
    double *partials = nullptr;  // device buffer of sslbm_total
    int partial_blocks = 0;
    int partial_device = -1;
    double *adj_partials = nullptr;  // device slots of sslbm_adjoint_step
    long long adj_slots = 0;
    int adj_device = -1;
};
