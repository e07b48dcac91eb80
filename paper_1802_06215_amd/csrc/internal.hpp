// Internal declarations shared by the host runtime and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hdx.h"

namespace hdx {

constexpr int kMaxRocks = HDX_MAX_ROCKS;
constexpr int kMaxGrid = HDX_MAX_GRID;
constexpr int kMaxPeds = HDX_MAX_PEDS;
constexpr int kMaxGoals = HDX_MAX_GOALS;
constexpr int kHorizon = HDX_MAX_HORIZON;
constexpr int kSenseEntries = 2 * (kMaxGrid - 1) * (kMaxGrid - 1) + 1;  // squared distances
constexpr int kMaxLeaf = HDX_MAX_LEAF_SCENARIOS;
constexpr int kMaxNavLeaf = HDX_MAX_NAV_LEAF_SCENARIOS;
constexpr int kNavActions = 9;
constexpr int kPedActions = 3;
constexpr int kRockTerms = 2 * kMaxGrid + 2;  // distances on a grid are below

enum : uint32_t { kTagStep = 0, kTagInit = 1, kTagPolicy = 2 };
constexpr uint64_t kEmptyKey = ~0ull;
constexpr uint64_t kPedTerminalObs = ~0ull;

// Model parameters and tables as the kernels read them (device memory, one
// per uploaded model).  Derived constants are computed once on the host.
// The header is read with scalar loads.
struct ModelHdr {
    int32_t kind, n_actions;
    // RockSample
    int32_t grid, n_rocks;
    int32_t rock_x[kMaxRocks], rock_y[kMaxRocks];
    // crowd driving
    int32_t n_peds, n_goals, n_levels;
    // multi-agent RockSample: ceil(2^16 / (5 + n_rocks)), so that robot 1's
    // action of joint action a < (5 + n_rocks)^2 is (a * joint_inv) >> 16
    int32_t joint_inv;
    float goal_x[kMaxGoals], goal_y[kMaxGoals];
    float path_len, dt, step_len, half_sigma, coll_r2, reach, ih_scale;
    float r_collision, r_step, r_goal;
    float near_d2;  // sqrt(d2) <= step_len iff d2 <= near_d2
    uint64_t fail_thr;  // action fails iff word < fail_thr (driving, navigation)
    // navigation: goal column (on the bottom row), wall row, gate columns and
    // the reading error (a neighbour's bit flips iff word < err_thr)
    int32_t nav_goal_x, nav_wall, nav_gate_x[2];
    uint64_t err_thr;
    // navigation map as rows of 16 cells, two per word: the known walls and
    // the cells off the map, and the unknown cells in runs of consecutive
    // indices on consecutive cells -- run i of word h, h's runs being
    // [nav_run_begin[h], nav_run_begin[h + 1]): first bit in its source word
    // (bits 0-4), length (5-9), first bit in word h (10-14), source word (15-16)
    uint32_t nav_wall_rows[8];
    int32_t nav_run_begin[9];
    uint32_t nav_runs[HDX_MAX_NAV_UNKNOWN];
};

struct DevModel {
    ModelHdr h;
    uint32_t sense_thr_m1[kSenseEntries];  // floor(acc(d) 2^32) - 1, by squared distance
    float gpow[kHorizon];                  // discount powers gamma^j rounded to FP32
    double gsum[kHorizon + 1];             // 1 + gamma + ... + gamma^(j-1)
    double gpow64[kRockTerms];             // gamma^d
};

struct StatesPtr {
    int32_t *w;
    float *s;
    int32_t *car;
    float *px, *py;
    uint8_t *goal;
    int64_t stride;
};

// The states from number `at` on.
inline StatesPtr states_from(StatesPtr S, int64_t at) {
    if (S.w) S.w += at;
    if (S.s) S.s += at;
    if (S.car) S.car += at;
    if (S.px) S.px += at;
    if (S.py) S.py += at;
    if (S.goal) S.goal += at;
    return S;
}
// A launch of 2^32 threads or more does not run whole, and says nothing: calls
// that give a row several threads take long arrays in launches of up to so many.
constexpr int64_t kLaunchThreads = 1ll << 31;

// One leaf as the expansion kernel sees it (built on the host from hdx_leaf).
struct LeafTask {
    const DevModel *model;
    // actions per tile, and per row that no tile crosses (two robots: robot
    // 2's actions under one of robot 1; otherwise all)
    int16_t kind, tile_actions, n_actions, row_actions;
    uint32_t k0, k1;
    int32_t policy, const_action, max_steps, max_depth;
    StatesPtr parent;
    const uint32_t *parent_ids;
    const int16_t *idx;
    int32_t n, depth, last_action, cap;
    StatesPtr out;
    uint32_t *ids_out;
    int16_t *perm;
    int32_t *n_children;
    uint64_t *child_z;
    int32_t *child_n, *child_off;
    float *child_u0, *child_l0;
    float *r_mean;
    int64_t *steps;
    StatesPtr sprime;
    float *r;
    uint64_t *z;
    float *U, *L;
    int32_t *child_of;
    unsigned char *work;  // driving: ped_work_bytes, or null
};

// A tile: actions [action, action + tile_actions) of a leaf (fewer at the
// end of the leaf's actions).
struct Tile {
    int32_t leaf, action;
};

// Work queue of the persistent launch; the last workgroup to leave resets
// it, so a captured graph can be replayed without a separate clear.
struct TileQueue {
    int32_t next, done, n_tiles, pad;
};

constexpr int32_t kStrided = -1;
// Launch schedule of the expansion kernel; results never depend on it.
struct Schedule {
    int32_t threads;     // workgroup size, a multiple of 64
    // 0: one workgroup per tile; > 0: that many workgroups per CU, which drain
    // the queue; kStrided: one per tile, and if there are more tiles when the
    // launch is replayed, a workgroup takes the one a grid further on next
    int32_t persistent;
    int32_t xcd_remap;   // keep consecutive tiles (one leaf) on one XCD
};

__host__ __device__ inline int32_t pow2_at_least(int32_t v) {
    int32_t p = 1;
    while (p < v) p <<= 1;
    return p;
}

// RockSample tile (one robot, or two): up to kRockActions actions of a leaf
// of n scenarios, the same on host (for the launch size) and device; the
// regions are described in run_tile_rocks.
constexpr int kRockActions = 5 + kMaxRocks;
constexpr int kRockSuccs = 6;              // a robot's moves, its sample, and no change
constexpr int kRockCols = kMaxRocks + 1;   // a column per rock, and one for all scenarios
constexpr int kRockSets = kMaxRocks + 2;   // live, acting, and per rock those reading it good
constexpr int kRockCells = 1024;           // x | y << 5
struct RockSucc {
    double value;            // rollout of a live scenario
    int32_t reward, steps;   // the live scenarios' rewards / 10; steps of one's rollout
};
struct RockLayout {
    uint32_t zmask, cmask, term, coef, succ, cells, state, ub, lb, cnt, sums, place, size, pre, misc, total;
};
// Words of lb: a value per scenario; where the rollouts run step by step, one
// per successor, and the effects of each cell.
__host__ __device__ inline int32_t rock_values(int32_t n, bool stepped) {
    return stepped ? kRockSuccs * n + kRockCells : n;
}
__host__ __device__ inline RockLayout make_rock_layout(int32_t n, int32_t values, bool two) {
    RockLayout L;
    uint32_t o = 0;
    auto take = [&](uint32_t bytes) {
        uint32_t at = o;
        o += (bytes + 15u) & ~15u;
        return at;
    };
    const uint32_t chunks = (uint32_t)((n + 63) / 64), splits = two ? 3 : 1, keys = two ? 9 : 3;
    L.zmask = take(8u * kMaxRocks * chunks);
    L.cmask = take(8u * (two ? 4 : 1) * chunks);
    L.term = take(8u * kRockTerms);
    L.coef = take(8u * kRockSuccs * kRockCols);
    L.succ = take((uint32_t)sizeof(RockSucc) * kRockSuccs);
    L.cells = take(4u * chunks);
    L.state = take(4u * (two ? 2 : 1) * n);
    L.ub = take(4u * n);
    L.lb = take(4u * values);
    L.cnt = take(4u * splits * (kRockSets + 1) * 32);
    L.sums = take(4u * kRockActions * keys * 2);
    L.place = take(4u * kRockActions * keys);
    L.size = take(4u * kRockActions * keys);
    L.pre = take(2u * splits * kRockSets * chunks);
    L.misc = take(4u * (1 + 2 * kRockSuccs));
    L.total = o;
    return L;
}

// Workspace of a driving leaf expanded and grouped by two kernels: per action
// and scenario the observation, U, L, reward code and steps.
inline size_t ped_work_bytes(int32_t n) { return (size_t)kPedActions * 24u * (size_t)n; }
// Before the workspaces of a call in the kernel arguments: its leaves that are
// grouped so far, and the calls that have ended, written to host memory too, so
// that the host knows which workspaces are free without an event on the caller's
// stream (which may be gone when the event is asked).
struct PedHead {
    uint32_t left, ended;
    uint32_t *host;
};
constexpr size_t kPedHeadBytes = 64;
constexpr int kPedTile = 12;  // scenarios of a driving leaf that one workgroup expands and groups
// Driving tile: the three actions of a leaf of n scenarios.
//   zkey, pos   per action: (observation, position) pairs, sorted in place,
//               p2 of them (a power of two)
//   ub, lb      per action and scenario: U and L
//   rcode       per action and scenario: which step reward
//   misc        live scenarios, rollout steps per action
struct PedLayout {
    uint32_t zkey, pos, ub, lb, rcode, misc, total;
    int32_t p2;
};
__host__ __device__ inline PedLayout make_ped_layout(int32_t n) {
    PedLayout L;
    L.p2 = pow2_at_least(n < 64 ? 64 : n);
    uint32_t o = 0;
    auto take = [&](uint32_t bytes) {
        uint32_t at = o;
        o += (bytes + 15u) & ~15u;
        return at;
    };
    L.zkey = take(8u * kPedActions * L.p2);
    L.pos = take(2u * kPedActions * L.p2);
    L.ub = take(4u * kPedActions * n);
    L.lb = take(4u * kPedActions * n);
    L.rcode = take(1u * kPedActions * n);
    L.misc = take(4u * (1 + kPedActions));
    L.total = o;
    return L;
}

// Navigation tile: na actions of a leaf of n scenarios, run by `waves`
// wavefronts.  Regions:
//   gsum, ub    discount sums and the bound by distance
//   code        per (action, scenario): NavCode
//   val         per (action, scenario): rollout value, for the policies that
//               run step by step (the default policy's follows from the code)
//   rows, perm  while scenarios are stepped, each wavefront's map rows;
//               afterwards the grouped order of each action
//   cnt, meta   per action and observation: scenario count, then the next
//               place in the grouped order; child index << 16 | count
//   chunk_r     per action and 64-scenario chunk: step reward sum
constexpr int kNavKeys = 257;  // 256 readings and the terminal one
constexpr int kNavSums = 128;  // discount sums staged in LDS
constexpr int kNavRowBytes = 64 * 8 * 4;  // one wavefront's map rows
struct NavLayout {
    uint32_t gsum, ub, code, val, rows, perm, cnt, meta, chunk_r, misc, total;
};
// pairs = na * n; stepped: the rollouts run step by step
__host__ __device__ inline NavLayout make_nav_layout(uint32_t pairs, uint32_t na, uint32_t chunks, uint32_t waves,
                                                     bool stepped) {
    NavLayout L;
    uint32_t o = 0;
    auto take = [&](uint32_t bytes) {
        uint32_t at = o;
        o += (bytes + 15u) & ~15u;
        return at;
    };
    L.gsum = take(8u * (kNavSums + 1));
    L.ub = take(4u * 32);
    L.misc = take(16);
    L.chunk_r = take(4u * na * chunks);
    L.cnt = take(4u * na * kNavKeys);
    L.meta = take(4u * na * kNavKeys);
    L.code = take(4u * pairs);
    L.val = stepped ? take(4u * pairs) : L.code;
    L.rows = take(kNavRowBytes * waves > 2u * pairs ? kNavRowBytes * waves : 2u * pairs);
    L.perm = L.rows;
    L.total = o;
    return L;
}
// Words that a navigation tile holds per (action, scenario): its codes, and
// beside them the rollouts' values where those run step by step, each of the two
// rounded as make_nav_layout rounds them.
inline int32_t nav_values(int32_t n, int32_t actions, bool stepped) {
    return stepped ? 2 * ((n * actions + 3) & ~3) : n * actions;
}
constexpr int32_t kMaxDynamicLds = 160 * 1024 - 256;
// Dynamic LDS of a workgroup for navigation leaves of up to n_max scenarios and
// tiles of up to `values` words (nav_values); counters for all nine actions.
inline uint32_t nav_lds(int32_t n_max, int32_t values, int32_t threads) {
    const uint32_t b = make_nav_layout((uint32_t)values, kNavActions, (uint32_t)(n_max + 63) / 64,
                                       (uint32_t)threads / 64, false).total;
    return b < (uint32_t)kMaxDynamicLds ? b : (uint32_t)kMaxDynamicLds;
}
// Actions per navigation tile of a leaf of n scenarios, at most `most`: as
// many as its LDS holds beside 16 wavefronts.
inline int32_t nav_tile_actions(int32_t n, int32_t policy, int32_t most) {
    for (int32_t w = most; w > 1; --w)
        if (kNavActions % w == 0 &&
            make_nav_layout((uint32_t)nav_values(n, w, policy != HDX_POLICY_DEFAULT), kNavActions,
                            (uint32_t)(n + 63) / 64, 16, false).total <= (uint32_t)kMaxDynamicLds)
            return w;
    return 1;
}

// The most words that a tile of a leaf of up to n scenarios holds, whatever its
// policy and its actions: what a launch is sized for that the caller captured.
inline int32_t most_values(bool nav, int32_t n) { return nav ? nav_values(n, kNavActions, true) : rock_values(n, true); }

// Kernel variant a set of leaves needs: mode 0 RockSample only, 1 driving
// only, 2 both; pm = pedestrian capacity of the register state; n_max sizes
// the LDS carve-up.
struct Variant {
    int32_t mode, pm, n_max;
    // driving only: the kernel instance with 8 or 16 lanes per scenario
    int32_t group = 0;
    // the most words of a tile: navigation nav_values, RockSample rock_values
    int32_t pairs = 1;
    // driving only: the leaves have workspaces
    bool rows = false;
};
Variant pick_variant(int32_t has_rs, int32_t has_ped, int32_t ped_max, int32_t n_max, int32_t has_mars,
                     int32_t has_nav);
int32_t variant_max_threads(const Variant &v);
// Lanes a leaf of n scenarios can use.
int32_t variant_lanes(const Variant &v, int32_t n);

// Kernel launchers (kernels.hip).  The expansion kernel reads the tile
// count from d_queue->n_tiles; n_tiles here only sizes a non-persistent grid.
hipError_t launch_expand(const LeafTask *d_tasks, const Tile *d_tiles, TileQueue *d_queue, int32_t n_tiles,
                         const Variant &v, const Schedule &sch, int32_t n_cu, hipStream_t stream);

// Tiles are launched in groups.  A group holds tiles of one model variant
// (0 RockSample, 1-3 driving with up to 8, 16, 32 pedestrians, 4
// multi-agent RockSample, 5 navigation), so
// RockSample tiles never run in the register budget of the driving model,
// and gets an LDS carve-up and workgroup size for its own largest leaf.  By
// default all leaves of a variant form one group (one dispatch, no fork and
// join between dispatches), filed under the size class of its largest leaf;
// split plans give each size class of leaf (n <= 64, 128, 256, 512, 1024,
// and larger) a group of its own, so small leaves do not pay for the largest one's
// footprint, and launch the groups side by side.  Inside a group the tiles
// are ordered largest leaf first (long tiles start early, short ones fill
// the tail), a leaf's tiles in action order, and interleaved so that the
// tiles of one leaf go to one XCD.  Group g = variant *
// kSizeClasses + size class; the tile array is ordered by group; group g
// owns tiles [begin[g], begin[g] + count[g]) and the queue d_queues[g].
constexpr int kSizeClasses = 6;
constexpr int kXcds = 8;  // accelerator dies, each with its own L2
constexpr int kModelVariants = 6;
constexpr int kGroups = kModelVariants * kSizeClasses;
__host__ __device__ inline int size_class(int32_t n) {
    int c = 0;
    while (c < kSizeClasses - 1 && n > (64 << c)) ++c;
    return c;
}
inline int model_variant(int32_t kind, int32_t n_peds) {
    return kind == HDX_ROCKSAMPLE ? 0 : kind == HDX_MARS ? 4 : kind == HDX_NAV ? 5 : n_peds <= 8 ? 1 : n_peds <= 16 ? 2 : 3;
}
inline Variant group_variant(int g) {
    const int v = g / kSizeClasses;
    if (v == 4) return Variant{3, 1, 1};
    if (v == 5) return Variant{4, 1, 1};
    return v == 0 ? Variant{0, 1, 1} : Variant{1, v == 1 ? 8 : v == 2 ? 16 : 32, 1};
}
struct ClassPlan {
    int64_t begin[kGroups], count[kGroups];
    int32_t n_max[kGroups], pairs[kGroups];
    bool rows = false;  // the driving leaves have workspaces
};
// Reorder tiles[0, n_tiles) by group, largest leaf first inside a group
// (variant[leaf] is the leaf's model variant); fills plan.
void plan_classes(const LeafTask *tasks, const int8_t *variant, Tile *tiles, int64_t n_tiles, ClassPlan *plan,
                  bool split);
// One launch per non-empty group in mask (bit g = group g); lds_n[g] and, but
// for driving, lds_pairs[g] size group g's LDS (at least its n_max and pairs);
// sch[g] is its schedule (its width capped at what the group's leaves and model
// need).
hipError_t launch_classes(const LeafTask *d_tasks, const Tile *d_tiles, TileQueue *d_queues, const ClassPlan &plan,
                          const int32_t *lds_n, const int32_t *lds_pairs, const Schedule *sch, int32_t n_cu,
                          hipStream_t stream, uint64_t mask = ~0ull);
// Default schedule of a group whose largest leaf has v.n_max scenarios.  Few
// tiles (a call far smaller than the GPU): a lane for every scenario (driving:
// its lanes), so each tile ends sooner.  Otherwise half a lane per scenario,
// for RockSample four wavefronts at most (2048 leaves of 31..500 scenarios: 61,
// 38, 31 and 39 us at 1, 2, 4 and 8) and, with fewer tiles than eight per CU,
// at least (72 leaves of 67: 11.5 us at one wavefront, 8.3 at four); driving a
// quarter of its lanes with more than one tile per CU (512 leaves of 125..500
// scenarios: 500 us at 512 lanes, 526 at 1024), else half (256 leaves among
// others: 930 and 769 us).  Workgroups in tile order, one per tile.
Schedule class_default_schedule(const Variant &v, int64_t tiles, int32_t n_cu, bool few);
hipError_t configure_expand_kernels();

// Up to kArgLeaves leaves passed by value in the kernel arguments (the
// pack stays under the 4 KB kernel-argument limit).
constexpr int kArgLeaves = 11;
struct ArgPack {
    int32_t n_leaves;
    int32_t tile_end[kArgLeaves];
    LeafTask t[kArgLeaves];
};
hipError_t launch_expand_args(const ArgPack &pack, const Variant &v, const Schedule &sch, hipStream_t stream);

struct SampleArgs {
    const DevModel *model;
    uint32_t k0, k1;
    int32_t K;
    int32_t x0, y0;  // RockSample: robot cell; multi-agent: x0 is the robots' row
    uint64_t rock_thr[kMaxRocks];
    float s0;
    int32_t level0;
    float px0[kMaxPeds], py0[kMaxPeds];
    uint64_t goal_thr[kMaxPeds][kMaxGoals];  // cumulative thresholds
    int32_t n_unknown;                       // navigation: unknown cells
    uint64_t cell_thr[HDX_MAX_NAV_UNKNOWN];  // navigation: P(occupied) thresholds
    StatesPtr out;
};
// Staged in device memory (d_args) before the launch.
hipError_t launch_sample(const SampleArgs *d_args, int32_t K, hipStream_t stream);

struct BoundsArgs {
    const DevModel *model;
    uint32_t k0, k1;
    int32_t policy, const_action, max_steps, max_depth;
    StatesPtr states;
    const uint32_t *ids;
    const int32_t *depths;
    int64_t n;
    float *U, *L;
    int32_t *steps;
};
hipError_t launch_bounds(const BoundsArgs &args, int32_t kind, int32_t n_peds, hipStream_t stream);

hipError_t launch_philox(const uint32_t *ctr, int64_t count, uint32_t k0, uint32_t k1, uint32_t *out,
                         hipStream_t stream);

hipError_t launch_fp32_selftest(const float *a, const float *b, const float *c, int64_t n, float *out,
                                hipStream_t stream);

}  // namespace hdx

// The description a model was uploaded from (host side, runtime.cpp).
const hdx_model_desc *hdx_internal_desc(const hdx_model *m);
void hdx_internal_set_error(hdx_ctx *ctx, const char *msg);
void hdx_internal_quiesce(hdx_ctx *ctx);
const hdx::DevModel *hdx_internal_devmodel(const hdx_model *m);
