// ensemble_api.cpp -- host side of the ensemble entry points in sslbm.h:
// validation, the state layout, size classes, tile tables, the per-class
// pass-shape tuner and HIP graph capture. Validation and layout queries need
// no GPU; device tables are built on first use.
//
// Size classes. Instances are grouped at creation:
//  * on chip: the five fields fit ENS_LDS_BYTES of LDS (64 x 64 in FP32).
//    One launch of the LDS-resident kernel advances all of them by every
//    step of a run (one workgroup per instance, read and written once).
//  * march classes, one per power-of-two bucket of the longest side (up to
//    2, 4, ..., 512, 1024, ...): passes of the tile-table kernel with a pass
//    shape (steps per pass, rows per wavefront, columns per lane) of their
//    own, automatic or tuned per class.
// A run is one or more chains of launches, side by side on streams of their
// own, forked from and joined back to the caller's stream (or parallel
// branches of one HIP graph); chains never wait for each other. The on-chip
// class is a chain. The march classes are
//  * one chain of register-tile passes over all of them, where their shapes
//    are automatic and they hold too few cells for marches;
//  * one chain of passes over all of them, where they have the same steps per
//    pass and columns per lane (the automatic shapes do, as a rule): one
//    launch per pass fills the GPU by itself, while a stream per class shares
//    hardware queues with the others, so that classes wait for each other
//    (96 grids of 64^2 to 512^2, the smallest on chip, FP32: 4.9 ms for 200
//    steps with three march chains, 3.5 ms with one);
//  * one such chain with one column per lane and one with two, on large
//    ensembles some of whose classes have grids of odd rows;
//  * else a chain per class.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <tuple>
#include <vector>

#include "ensemble_internal.h"
#include "sslbm.h"
#include "sslbm_internal.h"

namespace {

constexpr int MAX_ENS_SIDE = 1 << 16;
constexpr int MAX_INSTANCES = 1 << 20;
constexpr long long ALIGN_ELEMS = 4;

struct TileTable {
    sslbm::EnsTile *dev = nullptr;
    int count = 0;
    int V = 0;  // columns per lane of a march table
};

struct GraphKey {
    long long nsteps;
    void *rho, *scratch;
    bool operator<(const GraphKey &o) const {
        return std::tie(nsteps, rho, scratch) < std::tie(o.nsteps, o.rho, o.scratch);
    }
};

struct EnsClass {
    bool on_chip = false;
    int bucket = 0;  // march classes: longest side in (2^(bucket-1), 2^bucket]
    std::vector<int> insts;
    long long cells = 0;
    int max_side = 0;
    bool even_rows = true;  // every row length even (two columns per lane possible)
    std::vector<sslbm::GridSize> sizes;  // distinct sizes of the instances
    sslbm_launch launch{};  // requested pass shape, zero fields automatic
    hipStream_t stream = nullptr;
    hipEvent_t done = nullptr;
};

// One chain of passes over some march classes: register tiles (tiles.rows > 0),
// or marches of K steps with V columns per lane and H rows of each class.
struct Chain {
    std::vector<int> classes;
    sslbm::TilePlan tiles;
    int K = 0, V = 0;
    std::vector<int> H;
    int depth() const { return tiles.rows ? tiles.depth : K; }
};

}  // namespace

struct sslbm_ensemble {
    int count = 0, dtype = 0, bc = 0;
    std::vector<int> nx, ny;
    std::vector<long long> offset;
    long long elements = 0;
    std::vector<sslbm::StepCoef> coef;
    bool diffuse_d = false;
    std::vector<EnsClass> classes;  // march classes by bucket, then the on-chip class
    std::vector<int> class_of;      // class of every instance
    int march_max_side = 0;
    size_t lds_bytes = 0;  // the largest on-chip instance
    int last_hip = 0;
    int device = -1;
    void *insts = nullptr;    // device instance table
    int *lds_list = nullptr;  // device list of the on-chip instances
    bool tiles_tuned = false;  // automatic shapes because tiles were the fastest when timed
    std::vector<sslbm::GridSize> march_sizes;  // distinct sizes of the march classes' grids
    // tables of a chain's passes: {steps, columns per lane, then class and rows
    // per wavefront of each march class}, or {steps, 0, rows a lane, classes}
    std::map<std::vector<int>, TileTable> tiles;
    hipStream_t stream = nullptr;  // graph and tuning stream
    hipEvent_t ev_in = nullptr, ev_out = nullptr, ev_fork = nullptr;
    std::map<GraphKey, hipGraphExec_t> graphs;
    // the chains of the last run, which the next one most often repeats
    std::mutex planned_lock;
    long long planned_steps = -1;
    bool planned_pairs = false;
    std::vector<Chain> planned;
    int tiles_pay[2] = {-1, -1};  // by pair alignment: tiles are faster (-1: not yet known)
};

namespace {

sslbm_status hip_status(sslbm_ensemble *e, hipError_t err) {
    if (err == hipSuccess)
        return SSLBM_OK;
    e->last_hip = (int)err;
    return SSLBM_E_HIP;
}

size_t elem_bytes(const sslbm_ensemble *e) { return e->dtype == SSLBM_F32 ? 4 : 8; }

bool valid_class(const sslbm_ensemble *e, int c) {
    return c >= 0 && c < (int)e->classes.size();
}

// Tiles of one pass of k steps of class c: every instance of the class cut
// into strips of strip_width(k, V) output columns and chunks of H output rows.
void march_tiles(const sslbm_ensemble *e, int c, int k, int H, int V,
                 std::vector<sslbm::EnsTile> *t) {
    const int w = sslbm::strip_width(k, V);
    for (int i : e->classes[c].insts)
        for (int y0 = 0; y0 < e->ny[i]; y0 += H)
            for (int x0 = 0; x0 < e->nx[i]; x0 += w)
                t->push_back({i, x0, y0, std::min(y0 + H, e->ny[i]), (y0 / H) & 1});
}

// Register tiles of one pass of k steps of class c, R rows a lane.
void register_tiles(const sslbm_ensemble *e, int c, int k, int R,
                    std::vector<sslbm::EnsTile> *t) {
    const int w = 64 - 2 * k, h = sslbm::TILE_WAVES * R - 2 * k;
    for (int i : e->classes[c].insts)
        for (int y0 = 0; y0 < e->ny[i]; y0 += h)
            for (int x0 = 0; x0 < e->nx[i]; x0 += w)
                t->push_back({i, x0, y0, 0, 0});
}

// Columns per lane actually usable: two need every row length of the class
// even, pair-aligned buffers and a depth within the two-column register budget.
int usable_cols(const sslbm_ensemble *e, int c, int V, int k, bool pairs_ok) {
    if (V == 2 && (!pairs_ok || !e->classes[c].even_rows ||
                   k > sslbm::march_max_depth(e->dtype, 2)))
        return 1;
    return V;
}

// Strips of w output columns and chunks of H output rows of grids of some sizes.
long long count_tiles(const std::vector<sslbm::GridSize> &sizes, int w, int H) {
    long long n = 0;
    for (const sslbm::GridSize &z : sizes)
        n += (long long)((z.nx + w - 1) / w) * ((z.ny + H - 1) / H) * z.count;
    return n;
}

// Automatic columns per lane of grids of some sizes that share a launch: two
// halve the shifts per cell (about 5%: 40 grids of 512^2 555 against 527 GLUPS),
// unless their strips, twice as wide, cover more columns past the edges than
// that (256^2: 399 against 454; 64^2 to 512^2 mixed: 481 against 487).
int auto_cols(const sslbm_ensemble *e, const std::vector<sslbm::GridSize> &sizes, int K) {
    if (e->dtype != SSLBM_F32 || K > sslbm::march_max_depth(e->dtype, 2))
        return 1;
    long long covered[2] = {0, 0};
    for (int V = 1; V <= 2; ++V) {
        const int w = sslbm::strip_width(K, V);
        for (const sslbm::GridSize &z : sizes)
            covered[V - 1] += (long long)((z.nx + w - 1) / w) * 64 * V * z.ny * z.count;
    }
    return covered[1] <= covered[0] + covered[0] / 32 ? 2 : 1;
}

long long cells_of(const std::vector<sslbm::GridSize> &sizes) {
    long long n = 0;
    for (const sslbm::GridSize &z : sizes)
        n += (long long)z.nx * z.ny * z.count;
    return n;
}

// The fewest rows per wavefront, at least `least`, for which the tiles of grids
// of some sizes number at most `tiles` (the highest grid's rows if none are).
int rows_for(const std::vector<sslbm::GridSize> &sizes, int w, long long tiles, int least,
             int most) {
    int lo = least, hi = std::max(least, most);
    while (lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (count_tiles(sizes, w, mid) <= tiles)
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// Automatic rows per wavefront of passes of K steps over grids of some sizes:
// the fewest for which all their tiles are resident at once, the same rows for
// every class of a pass (it lasts as long as its longest march; with rows by
// each class's share of the GPU the smallest class had the tallest ones, and 96
// grids of 64^2 to 512^2 ran at 390 GLUPS, 481 so). Where that gives chunks of fewer than
// 16 rows, a wavefront less per SIMD on taller ones may be faster, as estimated
// (FP32, 60 steps: 8 grids of 512^2 330 us at 12 rows and two wavefronts a SIMD,
// 392 at 16; 6 of them 325 at 12 rows, 290 at 16 and one wavefront).
int auto_rows(const sslbm_ensemble *e, const std::vector<sslbm::GridSize> &sizes, int K, int V) {
    long long resident = sslbm::march_resident_waves(e->dtype, K, V, e->diffuse_d);
    if (resident <= 0) {
        (void)hipGetLastError();  // the query's error is not the launch's
        resident = 2 * 4 * 256;
    }
    const int w = sslbm::strip_width(K, V), least = 2 * K, most = e->march_max_side;
    int best = rows_for(sizes, w, resident, least, most);
    if (best >= 16)
        return best;
    double best_us = 0.0;
    const int simds = 4 * sslbm::compute_units();
    for (long long share = resident / simds; share >= 1; --share) {
        const int rows = rows_for(sizes, w, share * simds, least, most);
        const double us = sslbm::march_us(e->dtype, K, V, rows, count_tiles(sizes, w, rows));
        if (best_us == 0.0 || us < best_us) {
            best_us = us;
            best = rows;
        }
    }
    return best;
}

// Sizes of the march classes whose rows are all even (even = true), or of the
// others.
std::vector<sslbm::GridSize> sizes_by_parity(const sslbm_ensemble *e, bool even) {
    std::vector<sslbm::GridSize> out;
    for (const EnsClass &cl : e->classes)
        if (!cl.on_chip && cl.even_rows == even)
            out.insert(out.end(), cl.sizes.begin(), cl.sizes.end());
    return out;
}

// Whether classes of even rows take two columns per lane in a chain of their
// own while others, which cannot, keep one. One launch for all leaves every
// class at one column, but two chains share the GPU badly where passes are
// short: of 97 mixes of 4 to 30 million cells, 60 steps, two chains were up to
// 29% slower at 4 million (256^2 beside 301^2 606 us, one chain 470) and even on
// the mean at 12 million (60 rows a wavefront), but up to 15% faster at 30
// million (130 to 200 rows: 21 grids of 1024^2 and 29 of 511^2 3066 us, one
// chain 3640) and 7% at 86 rows, unless the even grids are few or do not gain by
// two columns.
bool cols_by_class(const sslbm_ensemble *e, int K, bool pairs_ok) {
    constexpr int TALL = 80;
    if (!pairs_ok || e->dtype != SSLBM_F32)
        return false;
    const std::vector<sslbm::GridSize> even = sizes_by_parity(e, true);
    if (even.empty() || cells_of(even) * 4 < cells_of(e->march_sizes) ||
        sizes_by_parity(e, false).empty() || auto_cols(e, even, K) == 1)
        return false;
    return auto_rows(e, e->march_sizes, K, 1) >= TALL;
}

// Rows of one of two chains: the fewest for which its tiles fit its share of
// the resident wavefronts, by cells.
int shared_rows(const sslbm_ensemble *e, bool even, int K, int V) {
    const std::vector<sslbm::GridSize> sizes = sizes_by_parity(e, even);
    const double share = (double)cells_of(sizes) / (double)cells_of(e->march_sizes);
    const double resident = (double)sslbm::march_resident_waves(e->dtype, K, V, e->diffuse_d);
    const long long tiles = std::max(64ll, (long long)(share * (resident > 0 ? resident : 2048.)));
    return rows_for(sizes, sslbm::strip_width(K, V), tiles, 2 * K, e->march_max_side);
}

// Pass shape of march class c: requested fields, automatic ones filled in.
// Automatic: six steps in FP32, five in FP64; columns and rows as above, over
// every march class (over class c alone where it runs alone). With a diffusing
// D too five steps in FP64, although that kernel spills and small single grids
// take four: 60 steps of 96 grids of 64^2 to 512^2 2025 us, 2403 at four; 200 of
// 128^2 1076 and 1108; four win only below 3 million cells (8 of 512^2 573, 545).
sslbm_launch resolve(const sslbm_ensemble *e, int c, bool pairs_ok = true, bool alone = false) {
    const EnsClass &cl = e->classes[c];
    sslbm_launch r = cl.launch;
    if (r.steps_per_pass == 0)
        r.steps_per_pass = e->dtype == SSLBM_F32 ? 6 : 5;
    const int K = r.steps_per_pass;
    if (r.cols_per_lane == 0 && !alone && cols_by_class(e, K, pairs_ok)) {
        r.cols_per_lane = cl.even_rows ? 2 : 1;
        if (r.rows_per_wave == 0)
            r.rows_per_wave = shared_rows(e, cl.even_rows, K, r.cols_per_lane);
    }
    if (r.cols_per_lane == 0) {
        r.cols_per_lane = auto_cols(e, alone ? cl.sizes : e->march_sizes, K);
        for (int i = 0; i < (int)e->classes.size(); ++i)
            if (!e->classes[i].on_chip && !alone)
                r.cols_per_lane =
                    std::min(r.cols_per_lane, usable_cols(e, i, r.cols_per_lane, K, pairs_ok));
    }
    r.cols_per_lane = usable_cols(e, c, r.cols_per_lane, K, pairs_ok);
    if (r.rows_per_wave == 0)
        r.rows_per_wave = auto_rows(e, alone ? cl.sizes : e->march_sizes, K, r.cols_per_lane);
    return r;
}

// The march class with the most cells (-1 if none).
int main_class(const sslbm_ensemble *e) {
    int best = -1;
    for (int c = 0; c < (int)e->classes.size(); ++c)
        if (!e->classes[c].on_chip && (best < 0 || e->classes[c].cells > e->classes[best].cells))
            best = c;
    return best;
}

// One more grid of nx x ny in a list of distinct sizes; `at` finds a size's
// entry in the list of owner `id`.
void count_size(std::vector<sslbm::GridSize> *sizes,
                std::map<std::tuple<int, int, int>, size_t> *at, int id, int nx, int ny) {
    const auto it = at->emplace(std::make_tuple(id, nx, ny), sizes->size());
    if (it.second)
        sizes->push_back(sslbm::GridSize{nx, ny, 0});
    ++(*sizes)[it.first->second].count;
}

// Graphs and plans made with shapes that changed.
void drop_plans(sslbm_ensemble *e) {
    {
        std::lock_guard<std::mutex> guard(e->planned_lock);
        e->planned_steps = -1;
        e->tiles_pay[0] = e->tiles_pay[1] = -1;
    }
    for (auto &g : e->graphs)
        (void)hipGraphExecDestroy(g.second);
    e->graphs.clear();
}

sslbm_status ensure_device_tables(sslbm_ensemble *e) {
    int dev = 0;
    sslbm_status st = hip_status(e, hipGetDevice(&dev));
    if (st != SSLBM_OK)
        return st;
    if (e->insts && e->device == dev)
        return SSLBM_OK;
    if (e->insts)
        return SSLBM_E_UNSUPPORTED;  // an ensemble stays on the device it first ran on
    const size_t rec = sslbm::ensemble_instance_bytes(e->dtype);
    std::vector<unsigned char> host(rec * e->count);
    for (int i = 0; i < e->count; ++i)
        sslbm::ensemble_pack_instance(e->dtype, host.data() + rec * i, e->offset[i], e->nx[i],
                                      e->ny[i], e->coef[i]);
    st = hip_status(e, hipMalloc(&e->insts, host.size()));
    if (st != SSLBM_OK)
        return st;
    st = hip_status(e, hipMemcpy(e->insts, host.data(), host.size(), hipMemcpyHostToDevice));
    if (st != SSLBM_OK)
        return st;
    for (const EnsClass &cl : e->classes) {
        if (!cl.on_chip)
            continue;
        st = hip_status(e, hipMalloc((void **)&e->lds_list, sizeof(int) * cl.insts.size()));
        if (st != SSLBM_OK)
            return st;
        st = hip_status(e, hipMemcpy(e->lds_list, cl.insts.data(), sizeof(int) * cl.insts.size(),
                                     hipMemcpyHostToDevice));
        if (st != SSLBM_OK)
            return st;
    }
    st = hip_status(e, hipStreamCreateWithFlags(&e->stream, hipStreamNonBlocking));
    if (st == SSLBM_OK)
        st = hip_status(e, hipEventCreateWithFlags(&e->ev_in, hipEventDisableTiming));
    if (st == SSLBM_OK)
        st = hip_status(e, hipEventCreateWithFlags(&e->ev_out, hipEventDisableTiming));
    if (st == SSLBM_OK)
        st = hip_status(e, hipEventCreateWithFlags(&e->ev_fork, hipEventDisableTiming));
    for (EnsClass &cl : e->classes) {
        if (st == SSLBM_OK)
            st = hip_status(e, hipStreamCreateWithFlags(&cl.stream, hipStreamNonBlocking));
        if (st == SSLBM_OK)
            st = hip_status(e, hipEventCreateWithFlags(&cl.done, hipEventDisableTiming));
    }
    if (st != SSLBM_OK)
        return st;
    e->device = dev;
    return SSLBM_OK;
}

// Estimated time of a step by a chain's marches.
double march_step_us(const sslbm_ensemble *e, const Chain &ch) {
    const int w = sslbm::strip_width(ch.K, ch.V);
    long long waves = 0;
    int rows = 0;
    for (size_t i = 0; i < ch.classes.size(); ++i) {
        waves += count_tiles(e->classes[ch.classes[i]].sizes, w, ch.H[i]);
        rows = std::max(rows, ch.H[i]);
    }
    return sslbm::march_us(e->dtype, ch.K, ch.V, rows, waves) / ch.K;
}

// Whether a run of a few steps is estimated to be faster by a chain's marches.
bool short_marches(const sslbm_ensemble *e, const std::vector<sslbm::GridSize> &sizes,
                   const Chain &ch, const sslbm::TilePlan &tiles, long long nsteps) {
    if (nsteps > sslbm::SHORT_RUN)
        return false;
    for (const sslbm::GridSize &z : sizes)
        if (std::min(z.nx, z.ny) < sslbm::SHORT_RUN_SIDE)
            return false;
    auto one = [&](int k) {
        const int w = sslbm::strip_width(k, ch.V);
        long long waves = 0;
        int rows = 0;
        for (size_t i = 0; i < ch.classes.size(); ++i) {
            waves += count_tiles(e->classes[ch.classes[i]].sizes, w, ch.H[i]);
            rows = std::max(rows, ch.H[i]);
        }
        return sslbm::short_march_us(e->dtype, k, ch.V, rows, waves, cells_of(sizes));
    };
    const sslbm::PassPlan plan = sslbm::plan_passes(nsteps, ch.K);
    double march = (double)(plan.count - plan.longer) * one(plan.base);
    if (plan.longer)
        march += (double)plan.longer * one(plan.base + 1);
    return sslbm::short_tiles_us(e->dtype, sizes.data(), (int)sizes.size(), tiles.rows,
                                 sslbm::plan_passes(nsteps, tiles.depth)) > 1.03 * march;
}

// Tiles of a chain whose shapes are all automatic: as for a single grid, none
// where its grids are too large for them or the march is estimated to be faster
// (an answer for runs of every length, kept in *pay, -1 before).
sslbm::TilePlan chain_tiles(const sslbm_ensemble *e, const std::vector<sslbm::GridSize> &sizes,
                            const Chain &ch, long long nsteps, int *pay) {
    const int n = (int)sizes.size();
    if (*pay == 0)
        return sslbm::TilePlan();
    const sslbm::TilePlan tiles = sslbm::tile_plan(e->dtype, sizes.data(), n, nsteps);
    if (tiles.rows == 0 || tiles.few || e->tiles_tuned)
        return tiles;
    if (short_marches(e, sizes, ch, tiles, nsteps))
        return sslbm::TilePlan();
    if (*pay < 0)
        *pay = sslbm::tiles_pay(e->dtype, sizes.data(), n, march_step_us(e, ch)) ? 1 : 0;
    return *pay ? tiles : sslbm::TilePlan();
}

// The march chains of a run of nsteps.
std::vector<Chain> march_chains(const sslbm_ensemble *e, long long nsteps, bool pairs_ok,
                                int *pay) {
    std::vector<Chain> out;
    bool automatic = true, alike = true;
    sslbm_launch joint[2] = {};  // the shapes of classes with automatic ones, by even rows
    for (int c = 0; c < (int)e->classes.size(); ++c) {
        const EnsClass &cl = e->classes[c];
        if (cl.on_chip)
            continue;
        const bool own = cl.launch.steps_per_pass == 0 && cl.launch.rows_per_wave == 0 &&
                         cl.launch.cols_per_lane == 0;
        automatic = automatic && own;
        sslbm_launch &kept = joint[cl.even_rows];
        const sslbm_launch r = own && kept.steps_per_pass ? kept : resolve(e, c, pairs_ok);
        if (own)
            kept = r;
        Chain ch;
        ch.classes = {c};
        ch.K = r.steps_per_pass;
        ch.V = r.cols_per_lane;
        ch.H = {r.rows_per_wave};
        alike = alike && (out.empty() || (out[0].K == ch.K && out[0].V == ch.V));
        out.push_back(ch);
    }
    // classes alike in one chain; automatic shapes are alike but for the columns
    // of even rows (cols_by_class): two chains
    if (alike || automatic) {
        std::vector<Chain> merged;
        for (const Chain &ch : out) {
            auto m = std::find_if(merged.begin(), merged.end(),
                                  [&](const Chain &o) { return o.K == ch.K && o.V == ch.V; });
            if (m == merged.end()) {
                merged.push_back(ch);
            } else {
                m->classes.push_back(ch.classes[0]);
                m->H.push_back(ch.H[0]);
            }
        }
        out.swap(merged);
    }
    if (automatic && out.size() == 1)
        out[0].tiles = chain_tiles(e, e->march_sizes, out[0], nsteps, pay);
    return out;
}

// The same, kept from the last run: working out the shapes of many sizes takes
// longer than a short run of a small ensemble (20 grids of 65^2 to 160^2, 6
// steps in FP32: 14 us with the plan kept, 23 planned anew each time).
std::vector<Chain> run_chains(sslbm_ensemble *e, long long nsteps, bool pairs_ok) {
    std::lock_guard<std::mutex> guard(e->planned_lock);
    if (e->planned_steps != nsteps || e->planned_pairs != pairs_ok) {
        e->planned = march_chains(e, nsteps, pairs_ok, &e->tiles_pay[pairs_ok]);
        e->planned_steps = nsteps;
        e->planned_pairs = pairs_ok;
    }
    return e->planned;
}

// The chain of one march class run on its own.
Chain class_chain(const sslbm_ensemble *e, int c, long long nsteps, bool pairs_ok) {
    const EnsClass &cl = e->classes[c];
    const sslbm_launch r = resolve(e, c, pairs_ok, true);
    int pay = -1;
    Chain ch;
    ch.classes = {c};
    ch.K = r.steps_per_pass;
    ch.V = r.cols_per_lane;
    ch.H = {r.rows_per_wave};
    if (cl.launch.steps_per_pass == 0 && cl.launch.rows_per_wave == 0 &&
        cl.launch.cols_per_lane == 0)
        ch.tiles = chain_tiles(e, cl.sizes, ch, nsteps, &pay);
    return ch;
}

// The table of a pass of k steps of a chain, built on first use.
sslbm_status chain_table(sslbm_ensemble *e, const Chain &ch, int k, bool pairs_ok,
                         TileTable **out) {
    int V = ch.V;
    for (int c : ch.classes)
        V = std::min(V, usable_cols(e, c, ch.V, k, pairs_ok));
    std::vector<int> key;
    if (ch.tiles.rows) {
        key = {k, 0, ch.tiles.rows};
        key.insert(key.end(), ch.classes.begin(), ch.classes.end());
    } else {
        key = {k, V};
        for (size_t i = 0; i < ch.classes.size(); ++i) {
            key.push_back(ch.classes[i]);
            key.push_back(ch.H[i]);
        }
    }
    auto it = e->tiles.find(key);
    if (it == e->tiles.end()) {
        std::vector<sslbm::EnsTile> t;
        for (size_t i = 0; i < ch.classes.size(); ++i) {
            if (ch.tiles.rows)
                register_tiles(e, ch.classes[i], k, ch.tiles.rows, &t);
            else
                march_tiles(e, ch.classes[i], k, ch.H[i], V, &t);
        }
        TileTable tab;
        tab.count = (int)t.size();
        tab.V = V;
        sslbm_status st =
            hip_status(e, hipMalloc((void **)&tab.dev, sizeof(sslbm::EnsTile) * t.size()));
        if (st != SSLBM_OK)
            return st;
        st = hip_status(e, hipMemcpy(tab.dev, t.data(), sizeof(sslbm::EnsTile) * t.size(),
                                     hipMemcpyHostToDevice));
        if (st != SSLBM_OK) {
            (void)hipFree(tab.dev);
            return st;
        }
        it = e->tiles.emplace(key, tab).first;
    }
    *out = &it->second;
    return SSLBM_OK;
}

// One pass of k steps of a chain, src -> dst.
sslbm_status enqueue_pass(sslbm_ensemble *e, const Chain &ch, const void *src, void *dst, int k,
                          bool pairs_ok, hipStream_t s) {
    TileTable *tab = nullptr;
    const sslbm_status st = chain_table(e, ch, k, pairs_ok, &tab);
    if (st != SSLBM_OK)
        return st;
    if (ch.tiles.rows)
        return hip_status(e, sslbm::launch_ensemble_tiles(e->dtype, src, dst, tab->dev, tab->count,
                                                          e->insts, e->bc, k, ch.tiles.rows,
                                                          e->diffuse_d, s));
    return hip_status(e, sslbm::launch_ensemble(e->dtype, src, dst, tab->dev, tab->count, e->insts,
                                                e->bc, k, tab->V, e->diffuse_d, s));
}

// Enqueue nsteps steps of a chain on stream s (tables must exist).
sslbm_status enqueue_chain(sslbm_ensemble *e, const Chain &ch, void *rho, void *scratch,
                           long long nsteps, bool pairs_ok, hipStream_t s) {
    void *src = rho, *dst = scratch;
    const sslbm::PassPlan plan = sslbm::plan_passes(nsteps, ch.depth());
    for (long long i = 0; i < plan.count; ++i) {
        const sslbm_status st = enqueue_pass(e, ch, src, dst, plan.steps(i), pairs_ok, s);
        if (st != SSLBM_OK)
            return st;
        std::swap(src, dst);
    }
    if (src != rho) {  // an odd number of passes: copy the chain's instances back
        const size_t eb = elem_bytes(e);
        for (int c : ch.classes)
            for (int i : e->classes[c].insts) {
                const size_t off = (size_t)e->offset[i] * eb;
                const sslbm_status st = hip_status(
                    e, hipMemcpyAsync(static_cast<char *>(rho) + off,
                                      static_cast<char *>(src) + off,
                                      5 * (size_t)e->nx[i] * e->ny[i] * eb,
                                      hipMemcpyDeviceToDevice, s));
                if (st != SSLBM_OK)
                    return st;
            }
    }
    return SSLBM_OK;
}

sslbm_status enqueue_on_chip(sslbm_ensemble *e, const EnsClass &cl, void *rho, long long nsteps,
                             hipStream_t s) {
    return hip_status(e, sslbm::launch_ensemble_lds(e->dtype, rho, e->lds_list,
                                                    (int)cl.insts.size(), e->insts, e->bc, nsteps,
                                                    e->diffuse_d, e->lds_bytes, s));
}

// Every chain of a run: the first march chain on s itself, every other chain
// on the stream of its (first) class, forked from and joined back to s.
sslbm_status enqueue_run(sslbm_ensemble *e, const std::vector<Chain> &chains, void *rho,
                         void *scratch, long long nsteps, bool pairs_ok, hipStream_t s) {
    const EnsClass *on_chip = nullptr;
    for (const EnsClass &cl : e->classes)
        if (cl.on_chip)
            on_chip = &cl;
    if (chains.empty())
        return on_chip ? enqueue_on_chip(e, *on_chip, rho, nsteps, s) : SSLBM_OK;
    sslbm_status st = SSLBM_OK;
    const bool forks = on_chip || chains.size() > 1;
    if (forks)
        st = hip_status(e, hipEventRecord(e->ev_fork, s));
    std::vector<const EnsClass *> side;
    if (on_chip)
        side.push_back(on_chip);
    for (size_t i = 1; i < chains.size(); ++i)
        side.push_back(&e->classes[chains[i].classes[0]]);
    for (size_t i = 0; i < side.size() && st == SSLBM_OK; ++i) {
        const EnsClass &cl = *side[i];
        st = hip_status(e, hipStreamWaitEvent(cl.stream, e->ev_fork, 0));
        if (st == SSLBM_OK)
            st = cl.on_chip ? enqueue_on_chip(e, cl, rho, nsteps, cl.stream)
                            : enqueue_chain(e, chains[i + 1 - (on_chip ? 1 : 0)], rho, scratch,
                                            nsteps, pairs_ok, cl.stream);
        if (st == SSLBM_OK)
            st = hip_status(e, hipEventRecord(cl.done, cl.stream));
    }
    if (st == SSLBM_OK)
        st = enqueue_chain(e, chains[0], rho, scratch, nsteps, pairs_ok, s);
    for (size_t i = 0; i < side.size() && st == SSLBM_OK; ++i)
        st = hip_status(e, hipStreamWaitEvent(s, side[i]->done, 0));
    return st;
}

// Build every table a run of nsteps will use (before any capture): a chain's
// run uses at most two depths, the longer and the shorter passes.
sslbm_status prepare_chains(sslbm_ensemble *e, const std::vector<Chain> &chains, long long nsteps,
                            bool pairs_ok) {
    for (const Chain &ch : chains) {
        const sslbm::PassPlan plan = sslbm::plan_passes(nsteps, ch.depth());
        for (long long i : {0ll, plan.count - 1}) {
            if (i < 0)
                continue;
            TileTable *tab = nullptr;
            const sslbm_status st = chain_table(e, ch, plan.steps(i), pairs_ok, &tab);
            if (st != SSLBM_OK)
                return st;
        }
    }
    return SSLBM_OK;
}

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

bool pairs_aligned(const sslbm_ensemble *e, const void *rho, const void *scratch) {
    const uintptr_t pair = 2 * elem_bytes(e);
    return !((uintptr_t)rho % pair) && !((uintptr_t)scratch % pair);
}

sslbm_status check_shape(const sslbm_ensemble *e, const sslbm_launch &r) {
    if (r.steps_per_pass < 0 || r.steps_per_pass > SSLBM_MAX_BLOCKING || r.rows_per_wave < 0 ||
        r.rows_per_wave > 65536 || r.cols_per_lane < 0 || r.cols_per_lane > 2)
        return SSLBM_E_ARG;
    const int K = r.steps_per_pass ? r.steps_per_pass : (e->dtype == SSLBM_F32 ? 6 : 5);
    if (K > sslbm::march_max_depth(e->dtype, 1) ||
        (r.cols_per_lane == 2 && K > sslbm::march_max_depth(e->dtype, 2)))
        return SSLBM_E_UNSUPPORTED;
    return SSLBM_OK;
}

// One pass of every march chain side by side (each on its own stream, forked
// from and joined back to the ensemble's stream), rho -> scratch, with the
// classes' current shapes: one untimed round, then three timed ones.
// Returns the joint rate in cell-updates per nanosecond (0 on error).
double joint_rate(sslbm_ensemble *e, const void *rho, void *scratch, bool pairs_ok,
                  hipEvent_t t0, hipEvent_t t1, sslbm_status *status) {
    sslbm_status st = SSLBM_OK;
    int pay = -1;
    const std::vector<Chain> chains = march_chains(e, 1000, pairs_ok, &pay);
    double work = 0.0;  // cell-updates of one round
    for (const Chain &ch : chains)
        for (int c : ch.classes)
            work += (double)e->classes[c].cells * ch.depth();
    for (int rep = 0; rep < 4 && st == SSLBM_OK; ++rep) {
        if (rep == 1)
            st = hip_status(e, hipEventRecord(t0, e->stream));
        if (st == SSLBM_OK && chains.size() > 1)
            st = hip_status(e, hipEventRecord(e->ev_fork, e->stream));
        for (size_t i = 0; i < chains.size() && st == SSLBM_OK; ++i) {
            const Chain &ch = chains[i];
            EnsClass &cl = e->classes[ch.classes[0]];
            if (i == 0) {
                st = enqueue_pass(e, ch, rho, scratch, ch.depth(), pairs_ok, e->stream);
                continue;
            }
            st = hip_status(e, hipStreamWaitEvent(cl.stream, e->ev_fork, 0));
            if (st == SSLBM_OK)
                st = enqueue_pass(e, ch, rho, scratch, ch.depth(), pairs_ok, cl.stream);
            if (st == SSLBM_OK)
                st = hip_status(e, hipEventRecord(cl.done, cl.stream));
        }
        for (size_t i = 1; i < chains.size() && st == SSLBM_OK; ++i)
            st = hip_status(
                e, hipStreamWaitEvent(e->stream, e->classes[chains[i].classes[0]].done, 0));
    }
    if (st == SSLBM_OK)
        st = hip_status(e, hipEventRecord(t1, e->stream));
    if (st == SSLBM_OK)
        st = hip_status(e, hipEventSynchronize(t1));
    float ms = 0.f;
    if (st == SSLBM_OK)
        st = hip_status(e, hipEventElapsedTime(&ms, t0, t1));
    *status = st;
    return st == SSLBM_OK && ms > 0.f ? 3.0 * work / (ms * 1e6) : 0.0;
}

// Candidate shapes of a march class: every depth and column count within
// the register budget, rows per wavefront automatic or 8 .. 128.
std::vector<sslbm_launch> candidates(const sslbm_ensemble *e, int c, bool pairs_ok) {
    std::vector<sslbm_launch> out;
    const EnsClass &cl = e->classes[c];
    for (int V = 1; V <= (pairs_ok && cl.even_rows ? 2 : 1); ++V)
        for (int K = 1; K <= sslbm::march_max_depth(e->dtype, V); ++K)
            for (int H : {0, 8, 16, 32, 64, 128})
                if (H == 0 || (H >= 2 * K && H <= cl.max_side))
                    out.push_back(sslbm_launch{K, H, V});
    return out;
}

// The tuner: first one shape for every march class (the best joint rate),
// then each class in turn, largest first, tries its candidates while the
// others keep theirs, and keeps whichever raises the joint rate. Where
// automatic shapes mean register tiles, these are tried too, last.
sslbm_status tune_classes(sslbm_ensemble *e, const void *rho, void *scratch, bool pairs_ok,
                          hipEvent_t t0, hipEvent_t t1) {
    std::vector<int> march;
    for (int c = 0; c < (int)e->classes.size(); ++c)
        if (!e->classes[c].on_chip)
            march.push_back(c);
    if (march.empty())
        return SSLBM_OK;
    std::sort(march.begin(), march.end(),
              [&](int a, int b) { return e->classes[a].cells > e->classes[b].cells; });
    sslbm_status st = SSLBM_OK;
    double best = -1.0;
    sslbm_launch common{};
    for (const sslbm_launch &cand : candidates(e, march[0], pairs_ok)) {
        for (int c : march)
            e->classes[c].launch = cand;
        const double rate = joint_rate(e, rho, scratch, pairs_ok, t0, t1, &st);
        if (st != SSLBM_OK)
            return st;
        if (rate > best) {
            best = rate;
            common = cand;
        }
    }
    for (int c : march)
        e->classes[c].launch = common;
    if (march.size() == 1)
        march.clear();
    for (int c : march) {
        sslbm_launch keep = e->classes[c].launch;
        for (const sslbm_launch &cand : candidates(e, c, pairs_ok)) {
            e->classes[c].launch = cand;
            const double rate = joint_rate(e, rho, scratch, pairs_ok, t0, t1, &st);
            if (st != SSLBM_OK)
                return st;
            if (rate > best) {
                best = rate;
                keep = cand;
            }
        }
        e->classes[c].launch = keep;
    }
    if (sslbm::tile_plan(e->dtype, e->march_sizes.data(), (int)e->march_sizes.size(), 1000).rows) {
        std::vector<sslbm_launch> keep;
        for (EnsClass &cl : e->classes) {
            keep.push_back(cl.launch);
            cl.launch = sslbm_launch{};
        }
        e->tiles_tuned = true;
        const double rate = joint_rate(e, rho, scratch, pairs_ok, t0, t1, &st);
        if (st != SSLBM_OK)
            return st;
        if (rate <= best) {
            for (size_t c = 0; c < e->classes.size(); ++c)
                e->classes[c].launch = keep[c];
            e->tiles_tuned = false;
        }
    }
    return SSLBM_OK;
}

}  // namespace

extern "C" {

sslbm_status sslbm_ensemble_create(sslbm_ensemble **out, int count, const int *nx, const int *ny,
                                   int dtype, int bc, const sslbm_params *params,
                                   int *bad_instance) {
    if (bad_instance)
        *bad_instance = -1;
    if (!out || !nx || !ny || !params || count < 1 || count > MAX_INSTANCES)
        return SSLBM_E_ARG;
    *out = nullptr;
    if (dtype != SSLBM_F32 && dtype != SSLBM_F64)
        return SSLBM_E_ARG;
    if (bc != SSLBM_PERIODIC && bc != SSLBM_NOFLUX)
        return SSLBM_E_ARG;
    sslbm_ensemble *e = new (std::nothrow) sslbm_ensemble();
    if (!e)
        return SSLBM_E_NOMEM;
    e->count = count;
    e->dtype = dtype;
    e->bc = bc;
    long long off = 0;
    for (int i = 0; i < count; ++i) {
        sslbm::StepCoef k;
        sslbm_status st = SSLBM_OK;
        if (nx[i] < 1 || ny[i] < 1 || nx[i] > MAX_ENS_SIDE || ny[i] > MAX_ENS_SIDE)
            st = SSLBM_E_ARG;
        else
            st = sslbm::derive_coef(&params[i], &k);
        if (st != SSLBM_OK) {
            if (bad_instance)
                *bad_instance = i;
            delete e;
            return st;
        }
        e->nx.push_back(nx[i]);
        e->ny.push_back(ny[i]);
        e->coef.push_back(k);
        e->offset.push_back(off);
        e->diffuse_d = e->diffuse_d || k.diffuse_d;
        off += (5ll * nx[i] * ny[i] + ALIGN_ELEMS - 1) / ALIGN_ELEMS * ALIGN_ELEMS;
    }
    e->elements = off;

    // size classes: on chip, else by the power-of-two bucket of the longest side
    const size_t eb = elem_bytes(e);
    std::map<int, int> bucket_class;
    std::vector<int> on_chip;
    for (int i = 0; i < count; ++i) {
        const size_t bytes = 5 * (size_t)nx[i] * ny[i] * eb;
        if (bytes <= (size_t)sslbm::ENS_LDS_BYTES) {
            on_chip.push_back(i);
            e->lds_bytes = std::max(e->lds_bytes, bytes);
            continue;
        }
        const int side = std::max(nx[i], ny[i]);
        int b = 0;
        while ((1 << b) < side)
            ++b;
        bucket_class[b] = 0;
    }
    for (auto &bc_pair : bucket_class) {
        bc_pair.second = (int)e->classes.size();
        EnsClass cl;
        cl.bucket = bc_pair.first;
        e->classes.push_back(cl);
    }
    if (!on_chip.empty()) {
        EnsClass cl;
        cl.on_chip = true;
        e->classes.push_back(cl);
    }
    e->class_of.assign(count, -1);
    std::map<std::tuple<int, int, int>, size_t> at_class, at_all;
    for (int i = 0; i < count; ++i) {
        int c;
        if (5 * (size_t)nx[i] * ny[i] * eb <= (size_t)sslbm::ENS_LDS_BYTES) {
            c = (int)e->classes.size() - 1;
        } else {
            const int side = std::max(nx[i], ny[i]);
            int b = 0;
            while ((1 << b) < side)
                ++b;
            c = bucket_class[b];
        }
        EnsClass &cl = e->classes[c];
        e->class_of[i] = c;
        cl.insts.push_back(i);
        cl.cells += (long long)nx[i] * ny[i];
        cl.max_side = std::max(cl.max_side, std::max(nx[i], ny[i]));
        cl.even_rows = cl.even_rows && nx[i] % 2 == 0;
        if (!cl.on_chip) {
            e->march_max_side = std::max(e->march_max_side, std::max(nx[i], ny[i]));
            count_size(&cl.sizes, &at_class, c, nx[i], ny[i]);
            count_size(&e->march_sizes, &at_all, 0, nx[i], ny[i]);
        }
    }
    *out = e;
    return SSLBM_OK;
}

long long sslbm_ensemble_offset(const sslbm_ensemble *e, int instance) {
    if (!e || instance < 0 || instance >= e->count)
        return -1;
    return e->offset[instance];
}

long long sslbm_ensemble_elements(const sslbm_ensemble *e) { return e ? e->elements : -1; }

int sslbm_ensemble_class_count(const sslbm_ensemble *e) {
    return e ? (int)e->classes.size() : SSLBM_E_ARG;
}

int sslbm_ensemble_instance_class(const sslbm_ensemble *e, int instance) {
    if (!e || instance < 0 || instance >= e->count)
        return SSLBM_E_ARG;
    return e->class_of[instance];
}

sslbm_status sslbm_ensemble_class_info(const sslbm_ensemble *e, int cls,
                                       sslbm_ensemble_class *info) {
    if (!e || !info || !valid_class(e, cls))
        return SSLBM_E_ARG;
    const EnsClass &cl = e->classes[cls];
    info->on_chip = cl.on_chip ? 1 : 0;
    info->instances = (int)cl.insts.size();
    info->cells = cl.cells;
    info->max_side = cl.max_side;
    info->launch = cl.on_chip ? sslbm_launch{0, 0, 0} : resolve(e, cls);
    return SSLBM_OK;
}

sslbm_status sslbm_ensemble_set_class_launch(sslbm_ensemble *e, int cls,
                                             const sslbm_launch *shape) {
    if (!e || !shape || !valid_class(e, cls))
        return SSLBM_E_ARG;
    const sslbm_status st = check_shape(e, *shape);
    if (st != SSLBM_OK)
        return st;
    if (e->classes[cls].on_chip)
        return SSLBM_E_UNSUPPORTED;
    e->classes[cls].launch = *shape;
    e->tiles_tuned = false;
    drop_plans(e);
    return SSLBM_OK;
}

sslbm_status sslbm_ensemble_set_launch(sslbm_ensemble *e, const sslbm_launch *shape) {
    if (!e || !shape)
        return SSLBM_E_ARG;
    const sslbm_status st = check_shape(e, *shape);
    if (st != SSLBM_OK)
        return st;
    for (EnsClass &cl : e->classes)
        if (!cl.on_chip)
            cl.launch = *shape;
    e->tiles_tuned = false;
    drop_plans(e);
    return SSLBM_OK;
}

sslbm_status sslbm_ensemble_get_launch(const sslbm_ensemble *e, sslbm_launch *shape) {
    if (!e || !shape)
        return SSLBM_E_ARG;
    const int c = main_class(e);
    *shape = c < 0 ? sslbm_launch{0, 0, 0} : resolve(e, c);
    return SSLBM_OK;
}

static sslbm_status run_checks(sslbm_ensemble *e, void *rho, void *scratch, long long nsteps) {
    if (!e || !rho || !scratch || nsteps < 0)
        return SSLBM_E_ARG;
    const size_t bytes = elem_bytes(e) * e->elements;
    if (overlap(rho, bytes, scratch, bytes))
        return SSLBM_E_ALIAS;
    return SSLBM_OK;
}

sslbm_status sslbm_ensemble_run_class(sslbm_ensemble *e, int cls, void *rho, void *scratch,
                                      long long nsteps, void *hip_stream) {
    sslbm_status st = run_checks(e, rho, scratch, nsteps);
    if (st != SSLBM_OK)
        return st;
    if (!valid_class(e, cls))
        return SSLBM_E_ARG;
    if (nsteps == 0)
        return SSLBM_OK;
    const bool pairs_ok = pairs_aligned(e, rho, scratch);
    st = ensure_device_tables(e);
    if (st != SSLBM_OK)
        return st;
    const hipStream_t s = (hipStream_t)hip_stream;
    if (e->classes[cls].on_chip)
        return enqueue_on_chip(e, e->classes[cls], rho, nsteps, s);
    const std::vector<Chain> chain{class_chain(e, cls, nsteps, pairs_ok)};
    st = prepare_chains(e, chain, nsteps, pairs_ok);
    if (st != SSLBM_OK)
        return st;
    return enqueue_chain(e, chain[0], rho, scratch, nsteps, pairs_ok, s);
}

sslbm_status sslbm_ensemble_run(sslbm_ensemble *e, void *rho, void *scratch, long long nsteps,
                                int flags, void *hip_stream) {
    sslbm_status st = run_checks(e, rho, scratch, nsteps);
    if (st != SSLBM_OK)
        return st;
    if (flags & ~SSLBM_RUN_GRAPH)
        return SSLBM_E_ARG;
    if (nsteps == 0)
        return SSLBM_OK;
    const bool pairs_ok = pairs_aligned(e, rho, scratch);
    st = ensure_device_tables(e);
    if (st != SSLBM_OK)
        return st;
    const std::vector<Chain> chains = run_chains(e, nsteps, pairs_ok);
    st = prepare_chains(e, chains, nsteps, pairs_ok);
    if (st != SSLBM_OK)
        return st;
    const hipStream_t user = (hipStream_t)hip_stream;
    if (!(flags & SSLBM_RUN_GRAPH))
        return enqueue_run(e, chains, rho, scratch, nsteps, pairs_ok, user);

    const GraphKey key{nsteps, rho, scratch};
    auto it = e->graphs.find(key);
    if (it == e->graphs.end()) {
        st = hip_status(e, hipStreamBeginCapture(e->stream, hipStreamCaptureModeThreadLocal));
        if (st != SSLBM_OK)
            return st;
        const sslbm_status run_st = enqueue_run(e, chains, rho, scratch, nsteps, pairs_ok, e->stream);
        hipGraph_t graph = nullptr;
        const hipError_t end = hipStreamEndCapture(e->stream, &graph);
        if (run_st != SSLBM_OK) {
            if (graph)
                (void)hipGraphDestroy(graph);
            return run_st;
        }
        st = hip_status(e, end);
        if (st != SSLBM_OK)
            return st;
        hipGraphExec_t exec = nullptr;
        st = hip_status(e, hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
        (void)hipGraphDestroy(graph);
        if (st != SSLBM_OK)
            return st;
        it = e->graphs.emplace(key, exec).first;
    }
    // order the graph after the caller's prior work and the caller's later
    // work after the graph
    st = hip_status(e, hipEventRecord(e->ev_in, user));
    if (st == SSLBM_OK)
        st = hip_status(e, hipStreamWaitEvent(e->stream, e->ev_in, 0));
    if (st == SSLBM_OK)
        st = hip_status(e, hipGraphLaunch(it->second, e->stream));
    if (st == SSLBM_OK)
        st = hip_status(e, hipEventRecord(e->ev_out, e->stream));
    if (st == SSLBM_OK)
        st = hip_status(e, hipStreamWaitEvent(user, e->ev_out, 0));
    return st;
}

sslbm_status sslbm_ensemble_tune(sslbm_ensemble *e, const void *rho, void *scratch,
                                 void *hip_stream, sslbm_launch *best) {
    if (!e || !rho || !scratch)
        return SSLBM_E_ARG;
    const size_t bytes = elem_bytes(e) * e->elements;
    if (overlap(rho, bytes, scratch, bytes))
        return SSLBM_E_ALIAS;
    sslbm_status st = ensure_device_tables(e);
    if (st != SSLBM_OK)
        return st;
    st = hip_status(e, hipStreamSynchronize((hipStream_t)hip_stream));
    if (st != SSLBM_OK)
        return st;
    hipEvent_t t0, t1;
    st = hip_status(e, hipEventCreate(&t0));
    if (st != SSLBM_OK)
        return st;
    st = hip_status(e, hipEventCreate(&t1));
    if (st != SSLBM_OK) {
        (void)hipEventDestroy(t0);
        return st;
    }
    const bool pairs_ok = pairs_aligned(e, rho, scratch);
    std::vector<sslbm_launch> saved;
    for (const EnsClass &cl : e->classes)
        saved.push_back(cl.launch);
    const bool saved_tiles = e->tiles_tuned;
    e->tiles_tuned = false;
    st = tune_classes(e, rho, scratch, pairs_ok, t0, t1);
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    if (st != SSLBM_OK) {
        for (size_t c = 0; c < e->classes.size(); ++c)
            e->classes[c].launch = saved[c];
        e->tiles_tuned = saved_tiles;
        return st;
    }
    drop_plans(e);
    if (best)
        sslbm_ensemble_get_launch(e, best);
    return SSLBM_OK;
}

int sslbm_ensemble_last_hip_error(const sslbm_ensemble *e) { return e ? e->last_hip : 0; }

void sslbm_ensemble_destroy(sslbm_ensemble *e) {
    if (!e)
        return;
    drop_plans(e);
    for (auto &t : e->tiles)
        (void)hipFree(t.second.dev);
    if (e->insts)
        (void)hipFree(e->insts);
    if (e->lds_list)
        (void)hipFree(e->lds_list);
    for (EnsClass &cl : e->classes) {
        if (cl.done)
            (void)hipEventDestroy(cl.done);
        if (cl.stream)
            (void)hipStreamDestroy(cl.stream);
    }
    for (hipEvent_t ev : {e->ev_in, e->ev_out, e->ev_fork})
        if (ev)
            (void)hipEventDestroy(ev);
    if (e->stream)
        (void)hipStreamDestroy(e->stream);
    delete e;
}

}  // extern "C"
