// HIP kernels for gfx950: scenario sampling, fused leaf expansion (update,
// expand, group by observation, bounds, rollouts, reductions) and
// stand-alone rollout bounds.
//
// Leaf expansion (Sec. III-D, Eq. 10-13) runs one workgroup per tile, a tile
// being some or all actions of a leaf: what does not depend on the action --
// the gather, the update step by the last action, the random numbers of a
// depth -- is done once for a tile's actions.  Each model has a tile of its
// own (run_tile_rocks, run_tile_ped, run_tile_nav): a lane, or a few, per
// scenario for the step, the bounds and the rollout, then the scenarios
// grouped by observation per action.
// The floating-point order depends only on the data, never on the workgroup
// size, the actions per tile or the schedule.
#include <algorithm>
#include <type_traits>

#include "models.hpp"

namespace hdx {

namespace {

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// Sum of v over the 64 lanes (all active), in one fixed order: inclusive
// prefix sums inside each row of 16 lanes (row shifts by 1, 2, 4, 8), then
// the row totals carried by the row broadcasts of lanes 15 and 31; the total
// is lane 63's prefix.  Lanes without a source add +0.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_src(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, true));
}
__device__ __forceinline__ float wave_total(float v) {
    v = v + dpp_src<0x111, 0xf>(v);  // row_shr:1
    v = v + dpp_src<0x112, 0xf>(v);  // row_shr:2
    v = v + dpp_src<0x114, 0xf>(v);  // row_shr:4
    v = v + dpp_src<0x118, 0xf>(v);  // row_shr:8
    v = v + dpp_src<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v = v + dpp_src<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// The same for integers (exact): the wavefront's sum, on every lane.
__device__ __forceinline__ int wave_total_i(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ bool has_states(const StatesPtr &S) { return S.w != nullptr || S.s != nullptr; }

// A value from the lane CTRL names (0 where there is none).
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_srci(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, true);
}
// One step of a segmented inclusive scan of two sums: f set where the
// segment's first lane has been reached.
template <int CTRL, int ROWS>
__device__ __forceinline__ void seg_step(float &u, float &l, int &f) {
    const float ou = dpp_src<CTRL, ROWS>(u), ol = dpp_src<CTRL, ROWS>(l);
    const int of = dpp_srci<CTRL, ROWS>(f);
    u = f ? u : ou + u;
    l = f ? l : ol + l;
    f |= of;
}

// LDS traffic of one wavefront stays in order; this keeps the compiler from
// moving it.
__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// The value of another lane of the lane's quad (quad_perm kCtrl).
template <int kCtrl>
__device__ __forceinline__ double quad_swap(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, kCtrl, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), kCtrl, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The descriptor again, so that what is read through it from here on is not
// read (and held in scalar registers, which run out) from the start.
__device__ __forceinline__ const HDX_CONST LeafTask *reread(const HDX_CONST LeafTask *T) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+s"(T));
#endif
    return T;
}
// v with lane i's value set to x (both uniform).
__device__ __forceinline__ uint64_t set_lane(uint64_t v, int i, uint64_t x) {
    return __builtin_amdgcn_inverse_ballot_w64(1ull << i) ? x : v;
}
// The scenarios of chunk t of a leaf of n.
__device__ __forceinline__ uint64_t chunk_mask(int n, int t) {
    return t * 64 + 64 <= n ? ~0ull : (1ull << (n & 63)) - 1ull;
}
// Lane t's mask, in scalar registers.
__device__ __forceinline__ uint64_t lane_mask(uint64_t v, int t) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, t);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), t);
    return ((uint64_t)hi << 32) | lo;
}
// A mask that all lanes read, in scalar registers.
__device__ __forceinline__ uint64_t uniform_mask(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
// base + the bits of a mask below this lane.
__device__ __forceinline__ int rank_in(uint64_t mask, int base) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, (uint32_t)base));
}
// A chunk's scenarios by observation key: from the live ones, those whose
// acting robot acts, those robot 1 read good (ga) and bad (gb), and those
// that read good (z); terminal scenarios read nothing.
template <bool kTwo, int K>
__device__ __forceinline__ void rock_keys(uint64_t (&keys)[K], uint64_t valid, uint64_t live, uint64_t act, uint64_t ga,
                                          uint64_t gb, uint64_t z, bool sense) {
    if constexpr (!kTwo) {
        keys[0] = sense ? valid & ~live : valid;
        keys[1] = sense ? z : 0;
        keys[2] = sense ? live & ~z : 0;
    } else {
        const uint64_t s[3] = {live & ~(ga | gb), ga, gb};
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            keys[3 * r] = sense ? s[r] & ~act : s[r];
            keys[3 * r + 1] = sense ? s[r] & z : 0;
            keys[3 * r + 2] = sense ? s[r] & act & ~z : 0;
        }
        keys[0] |= valid & ~live;
    }
}

// A thread's place in work that is to begin on other wavefronts than the work
// beside it: halves changed about within the largest power of two that divides
// the workgroup, so that every place is some thread's at any multiple of 64
// (tid ^ nt / 2 leaves places out at 192), with a scalar operand.
__device__ __forceinline__ int swapped_half(int tid, int nt) { return tid ^ ((nt & -nt) >> 1); }

// cell_effects of every cell, by the whole workgroup, with barriers.
__device__ __forceinline__ void stage_effects(const MView &M, uint32_t *effects) {
    for (int i = threadIdx.x; i < kRockCells; i += blockDim.x) effects[i] = cell_effects(M, i);
    __syncthreads();
    if ((int)threadIdx.x < M.h->n_rocks)
        effects[M.h->rock_x[threadIdx.x] | (M.h->rock_y[threadIdx.x] << 5)] |= rock_effect((int)threadIdx.x);
    __syncthreads();
}

// Rollout step by step (constant or random policy) of the lane's robots, at
// most R steps from depth d0, accumulated in FP32 in step order.  Lanes come in
// groups of `width`, all of one scenario, whose random actions are the same for
// whatever state it is in: lane c of a group draws those of depths c, width + c,
// ... and the others read them from it.  Called by all lanes of a wavefront.
template <class Ops>
__device__ __forceinline__ float rock_rollout(const MView &M, const uint32_t *effects, const RolloutParams &P, uint32_t id,
                                              int d0, int R, typename Ops::Team t, int width, int c, int &steps) {
    const Modulus pick((uint32_t)P.n_actions);
    const int first = lane_id() - c, grid = M.h->grid;
    float value = 0.0f;
    steps = 0;
    bool alive = t.any(grid);
    int drawn = 0, at = width;
    float powers = 0.0f;  // lane i: 10 gamma^i of the current 64 depths
    for (int j = 0;; ++j, ++at) {
        alive &= j < R;
        if (!__ballot(alive)) break;
        if ((j & 63) == 0) powers = 10.0f * M.gpow(min(j + lane_id(), kHorizon - 1));
        const float ten = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(powers), j & 63));
        int a = P.const_action;
        if (P.policy == HDX_POLICY_RANDOM) {
            if (at == width) {
                drawn = (int)pick(philox(id, (uint32_t)(d0 + j + c), 0, kTagPolicy, P.k0, P.k1).x);
                at = 0;
            }
            a = width > 1 ? __shfl(drawn, first + at, 64) : drawn;
        }
        const float v = value + Ops::act(M, effects, t, a, ten);
        value = alive ? v : value;
        steps += alive ? 1 : 0;
        alive &= t.any(grid);
    }
    return value;
}

// RockSample, one robot (RsOps) or two (MarsOps): nb actions of one leaf from
// action a_first on.  With two robots a tile stays within one action a1 of
// robot 1, which acts first and with the same outcome for all of them; what
// follows is then robot 2's actions on what robot 1 left, as with one robot.
//
// What bounds it: instruction issue, in the grouped order of the readings (a
// place per action and scenario) and in the masks that give it.
//  - The gather, the update step and the random block of a scenario are the
//    same for all actions, and a sense leaves the state as it is, so all
//    senses share one successor: six successors per scenario (four moves, a
//    sample, none) where one action per tile took 20 steps, bounds and
//    rollouts for 15 rocks.
//  - Readings are held as 64-bit masks, a word per 64-scenario chunk and rock:
//    a rank is a count of bits below a lane, a child's size a count of bits.
//  - Robot cells are deterministic, so the live scenarios of a leaf share
//    them.  Then the bound of a scenario is a sum of terms of its good rocks,
//    the same terms for all, and a child's sum of bounds is each term times
//    the number of its scenarios with that rock good: popcounts of the
//    reading's mask with the rock's, summed as integers, and one dot product
//    in FP64.  The default rollout moves east, so its value is the same for
//    all live scenarios of a successor, in closed form.
//  - Leaves whose scenarios differ in their cells, and the other rollout
//    policies, take per-scenario values instead, summed per chunk by DPP row
//    reductions, chunks in order.  Rollouts step by step run a lane per scenario
//    and successor (rock_rollout): the successors share their random actions,
//    and small leaves fill a wavefront.
// Integers and fixed orders throughout: results do not depend on the width or
// on how many actions a tile takes.
// Measured, one action per tile before and now: 2048 leaves of 31..500
// scenarios with 20 actions 96 -> 34 us, 8192 leaves of 6..100 with 13
// 119 -> 43, 128 leaves of 31..500 with 625 joint actions 375 -> 74; 1206 leaves
// of two scenarios with random rollouts 180 -> 51; a single leaf of 500 with 20
// actions (one action per tile) 7.9 -> 7.9, mostly the launch (its tile 14.7
// -> 12.6 thousand cycles, one of a leaf of 67 on four wavefronts 20 -> 9.5,
// with the successors and the children on several wavefronts).
// (rock_set: a child's live scenarios under one reading of robot 1, as the set
// `from` without the set `minus`; -1 none.)
struct RockSet {
    int from, minus;
};
template <bool kTwo>
__device__ __forceinline__ RockSet rock_set(int b, int z2) {
    constexpr int kAct = kTwo ? 1 : 0;  // one robot: a live one acts
    if (b < 5) return RockSet{z2 == 0 ? 0 : -1, -1};
    const int z = 2 + b - 5;
    return RockSet{z2 == 1 ? z : z2 == 2 ? kAct : kTwo ? 0 : -1, z2 == 1 ? -1 : z2 == 2 ? z : kTwo ? kAct : -1};
}

template <class Ops>
__device__ __forceinline__ void run_tile_rocks(const HDX_CONST LeafTask *T, const int a_first, const int nb,
                                               unsigned char *lds) {
    constexpr bool kTwo = Ops::kTwo;
    constexpr int kKeys = kTwo ? 9 : 3;
    constexpr int kSplits = kTwo ? 3 : 1;  // robot 1 read nothing, good, bad
    const int n = T->n, cap = T->cap, nch = (n + 63) >> 6;
    const int tid = threadIdx.x, nt = blockDim.x, lane = lane_id(), wid = tid >> 6, nw = nt >> 6;
    const MView M = make_view(T->model);
    const int per = T->row_actions, m = per - 5;
    const int a1 = kTwo ? (a_first * M.h->joint_inv) >> 16 : 0;
    const int b0 = kTwo ? a_first - a1 * per : a_first, b1 = b0 + nb;  // the acting robot's actions
    const int j0 = b0 > 5 ? b0 - 5 : 0, j1 = b1 - 5;                  // senses j0 <= j < j1
    const bool split = kTwo && a1 >= 5;                                // robot 1 reads
    const bool stepped = T->policy != HDX_POLICY_DEFAULT;
    const RockLayout Ly = make_rock_layout(n, rock_values(n, stepped), kTwo);
    uint64_t *zmask = (uint64_t *)(lds + Ly.zmask);  // [rock][chunk]: scenarios that read it good
    uint64_t *cmask = (uint64_t *)(lds + Ly.cmask);  // [live, acting, robot 1 good, bad][chunk]
    int32_t *cells = (int32_t *)(lds + Ly.cells);    // per chunk: the live scenarios' cells, -1 none, -2 several
    int32_t *state = (int32_t *)(lds + Ly.state);
    float *ub = (float *)(lds + Ly.ub), *lb = (float *)(lds + Ly.lb);  // (lb: per successor if they run step by step)
    uint32_t *effects = (uint32_t *)(lb + kRockSuccs * n);  // (there only then)
    // [split][set][column]: scenarios of a split and a set (0 live, 1 acting, 2 + j those reading rock j good) that
    // hold column i (rock i good; column kRockCols - 1: all)
    int32_t *cnt = (int32_t *)(lds + Ly.cnt);
    double *term = (double *)(lds + Ly.term);  // 10 gamma^d
    double *coef = (double *)(lds + Ly.coef);  // [successor][column]: bound's terms
    float *sums = (float *)(lds + Ly.sums);    // [action][key][U, L]: per-scenario values summed
    int32_t *place = (int32_t *)(lds + Ly.place);  // [action][key]: child's offset | its index << 16
    int32_t *size = (int32_t *)(lds + Ly.size);    // [action][key]: child's scenarios
    RockSucc *succ = (RockSucc *)(lds + Ly.succ);
    uint16_t *pre = (uint16_t *)(lds + Ly.pre);  // [split][row][chunk]: scenarios of earlier chunks
    int32_t *misc = (int32_t *)(lds + Ly.misc);  // robot 1's rewards / 10; then per successor rewards / 10, steps
    constexpr int kSetSize = 32, kSplitSize = (kRockSets + 1) * kSetSize;

    RolloutParams RP;
    RP.k0 = T->k0;
    RP.k1 = T->k1;
    RP.policy = T->policy;
    RP.const_action = T->const_action;
    RP.max_steps = T->max_steps;
    RP.max_depth = T->max_depth;
    RP.n_actions = T->n_actions;
    const int depth = T->depth, last_action = T->last_action;
    const int R = rollout_length(RP, depth + 1);
    const StatesPtr parent = load_states(&T->parent);
    const StatesPtr leaf_out = load_states(&T->out);
    const bool draw = j1 > j0 || split;
    // lane i's rock, a chunk's scenarios and the terms 10 gamma^d by distance: loads that wait for nothing here
    const int rock_x = M.h->rock_x[lane < kMaxRocks ? lane : 0], rock_y = M.h->rock_y[lane < kMaxRocks ? lane : 0];
    typename Ops::State ahead;  // the next chunk's parent state and id
    uint32_t id_ahead = 0;
    auto gather = [&](int t) {
        const int k = t * 64 + lane;
        Ops::make_terminal(ahead);
        if (k < n) {
            // 32-bit unsigned offsets let the loads take a scalar base
            const uint32_t p = (uint16_t)T->idx[(uint32_t)k];
            id_ahead = T->parent_ids[p];
            Ops::load(M, parent, p, ahead);
        }
    };
    gather(wid);
    for (int i = tid; i < kSplits * kSplitSize; i += nt) cnt[i] = 0;
    for (int d = tid; d < kRockTerms; d += nt) term[d] = 10.0 * M.gpow_exact(d);
    if (tid < 1 + 2 * kRockSuccs) misc[tid] = 0;
    __syncthreads();

    // -- gather + update, robot 1's action, readings (Eq. 10) ------------------
    for (int t = wid; t < nch; t += nw) {
        const int k = t * 64 + lane;
        const bool valid = k < n;
        typename Ops::State st = ahead;
        const uint32_t id = id_ahead;
        gather(t + nw);
        if (valid) {
            if (last_action >= 0) Ops::move(M, st, last_action);
            if (a_first == 0) {
                Ops::store(M, leaf_out, k, st);
                T->ids_out[k] = id;
            }
        }
        const bool live = valid && !Ops::terminal(st);
        const uint64_t lv = __ballot(live);
        // the shared cell and from it the threshold of lane i's rock, a load in flight while what follows is computed
        int cell = -1;
        uint32_t thr_i = 0;
        auto locate = [&]() {
            if (!lv) return;
            const int leader = __ffsll((unsigned long long)lv) - 1;
            cell = __builtin_amdgcn_readlane(Ops::cell(st), leader);
            if (__ballot(live && Ops::cell(st) != cell)) cell = -2;
            if (cell >= 0 && j1 > j0 && lane < m) {
                const int dx = Ops::cell_x(cell) - rock_x, dy = Ops::cell_y(cell) - rock_y;
                thr_i = M.thr[(uint32_t)(dx * dx + dy * dy)];
            }
        };
        if constexpr (!kTwo) locate();
        uint4 u = make_uint4(0, 0, 0, 0);
        if (draw && lv) u = philox(id, (uint32_t)depth, 0, kTagStep, RP.k0, RP.k1);
        int z1 = 0;
        uint64_t act = lv;
        uint32_t word = u.x;
        if constexpr (kTwo) {
            float r1 = 0.0f;
            if (live) r1 = Ops::template act<0, true>(M, st, a1, u.x, z1);
            word = u.y;
            act = __ballot(live && !Ops::template gone<1>(st));
            const int r = wave_total_i((int)r1);
            if (lane == 0 && r != 0) atomicAdd(&misc[0], r / 10);
            if (valid) {
                state[k] = Ops::with_reward(st.p, r1);
                state[n + k] = st.rk;
            }
        } else {
            if (valid) state[k] = st.w;
        }
        if constexpr (kTwo) locate();
        const uint64_t ga = split ? __ballot(z1 == 1) : 0, gb = split ? __ballot(z1 == 2) : 0;
        const uint64_t g0 = lv & ~(ga | gb);
        if (lane == 0) {
            cells[t] = cell;
            cmask[t] = lv;
            if constexpr (kTwo) {
                cmask[nch + t] = act;
                cmask[2 * nch + t] = ga;
                cmask[3 * nch + t] = gb;
            }
        }
        if (!lv) {
            if (lane >= j0 && lane < j1) zmask[lane * nch + t] = 0;
            continue;
        }
        // lanes i and 32 + i: column i's mask, the live scenarios with rock i good (the last column: all)
        const uint32_t rocks = live ? Ops::rocks(st) : 0u;
        uint64_t good = 0;
#pragma unroll 4
        for (int i = 0; i < m; ++i) good = set_lane(good, i, __ballot((rocks >> i) & 1u));
        uint64_t col = __shfl(good, lane & 31, 64);
        if ((lane & 31) == kRockCols - 1) col = lv;
        // count two sets at once, the first in the lower lanes
        auto count = [&](int set, uint64_t s0, uint64_t s1) {
            const uint64_t v = (lane < 32 ? s0 : s1) & col;
            int32_t *c = cnt + (set + (lane >> 5)) * kSetSize + (lane & 31);
            if (!split) {
                atomicAdd(c, __popcll(v));
            } else {
                atomicAdd(c + kSplitSize, __popcll(v & ga));
                atomicAdd(c + 2 * kSplitSize, __popcll(v & gb));
                if (g0) atomicAdd(c, __popcll(v & g0));
            }
        };
        count(0, lv, act);
        // a reading is good if it is correct of a good rock or wrong of a bad one
        auto reading = [&](int j) -> uint64_t {
            uint32_t thr;
            if (cell >= 0) {
                thr = (uint32_t)__builtin_amdgcn_readlane((int)thr_i, j);
            } else {
                const int c = live ? Ops::cell(st) : 0;
                const int dx = Ops::cell_x(c) - M.h->rock_x[j], dy = Ops::cell_y(c) - M.h->rock_y[j];
                thr = M.thr[(uint32_t)(dx * dx + dy * dy)];
            }
            return act & ~(__ballot(word <= thr) ^ lane_mask(good, j));
        };
        uint64_t zl = 0;  // lane j: the scenarios that read rock j good
#pragma unroll 2
        for (int j = j0; j < j1; j += 2) {
            const uint64_t za = reading(j), zb = j + 1 < j1 ? reading(j + 1) : 0;
            zl = set_lane(set_lane(zl, j, za), j + 1, zb);
            count(2 + j, za, zb);
        }
        if (lane >= j0 && lane < j1) zmask[lane * nch + t] = zl;
    }
    __syncthreads();
    T = reread(T);

    // -- does the leaf share its cells? ------------------------------------------
    int cell = -1;
    {
        const int c = lane < nch ? cells[lane] : -1;
        const uint64_t some = __ballot(c >= 0);
        if (some) cell = __builtin_amdgcn_readlane(c, __ffsll((unsigned long long)some) - 1);
        if (__ballot(c == -2 || (c >= 0 && c != cell))) cell = -2;
    }
    const bool shared = cell != -2, shared_l = shared && RP.policy == HDX_POLICY_DEFAULT;
    int live_n = 0;
#pragma unroll
    for (int sp = 0; sp < kSplits; ++sp) live_n += cnt[sp * kSplitSize + kRockCols - 1];

    // -- per-scenario values where they are needed --------------------------------
    const bool values = !shared || !shared_l || T->U != nullptr || T->L != nullptr;
    // the successors this tile's actions lead to
    const int c0 = b0 < 5 ? b0 : 5, c1 = b1 < kRockSuccs ? b1 : kRockSuccs, nc = c1 - c0;
    if (values) {
        for (int i = tid; i < kRockActions * kKeys * 2; i += nt) sums[i] = 0.0f;
        if (stepped) {
            stage_effects(M, effects);
            // a lane per scenario and successor, the successors of a scenario side by side
            const int per_wave = 64 / nc, i = lane / nc, c = lane - i * nc;
            for (int k0 = wid * per_wave; k0 < n; k0 += nw * per_wave) {
                const int k = k0 + i;
                const bool mine = i < per_wave && k < n;
                typename Ops::State st;
                Ops::make_terminal(st);
                uint32_t id = 0;
                if (mine) {
                    Ops::from_words(st, state[k], kTwo ? state[n + k] : 0);
                    id = T->parent_ids[(uint16_t)T->idx[(uint32_t)k]];
                }
                typename Ops::Team team = Ops::team(M, st);
                team.hop(effects, M.h->grid, kTwo ? 1 : 0, c0 + c, 0.0f);  // (5: no effect)
                int ns;
                const float L = rock_rollout<Ops>(M, effects, RP, id, depth + 1, R, team, nc, c, ns);
                if (mine) {
                    lb[(c0 + c) * n + k] = L;
                    atomicAdd(&misc[2 + 2 * (c0 + c)], ns);
                }
            }
            __syncthreads();
        }
        for (int c = c0; c < c1; ++c) {
            const int lo = c < 5 ? c : (b0 > 5 ? b0 : 5), hi = c < 5 ? c + 1 : b1;  // its actions
            float *const lc = lb + (stepped ? c * n : 0);
            typename Ops::WaveUpper wave_upper;
            int steps = 0, rewards = 0;
            for (int t = wid; t < nch; t += nw) {
                const int k = t * 64 + lane;
                typename Ops::State st;
                Ops::make_terminal(st);
                if (k < n) Ops::from_words(st, state[k], kTwo ? state[n + k] : 0);
                if (!Ops::terminal(st)) {
                    if (c < 5 && Ops::acting(st)) rewards += (int)Ops::mover(M, st, c);
                    Ops::settle(st);
                }
                const float U = Ops::upper_wave(M, st, wave_upper);
                if (k < n) {
                    int ns = 0;
                    const float L = stepped ? lc[k] : Ops::rollout_east(M, st, R, ns);
                    steps += ns;
                    ub[k] = U;
                    lc[k] = L;
                    for (int b = lo; b < hi; ++b) {
                        const int64_t at = (int64_t)(a_first + b - b0) * n + k;
                        if (T->U) T->U[at] = U;
                        if (T->L) T->L[at] = L;
                    }
                }
            }
            steps = wave_total_i(steps);
            rewards = wave_total_i(rewards) / 10;
            if (lane == 0) {
                atomicAdd(&misc[1 + 2 * c], rewards);
                if (!stepped) atomicAdd(&misc[2 + 2 * c], steps);
            }
            __syncthreads();
            // sums per child of its actions, one wavefront per action
            for (int b = lo + wid; b < hi; b += nw) {
                for (int t = 0; t < nch; ++t) {
                    const int k = t * 64 + lane;
                    const float u = k < n ? ub[k] : 0.0f, l = k < n ? lc[k] : 0.0f;
                    uint64_t keys[kKeys];
                    rock_keys<kTwo>(keys, chunk_mask(n, t), cmask[t], kTwo ? cmask[nch + t] : 0,
                                    kTwo ? cmask[2 * nch + t] : 0, kTwo ? cmask[3 * nch + t] : 0,
                                    b >= 5 ? zmask[(b - 5) * nch + t] : 0, b >= 5);
#pragma unroll
                    for (int q = 0; q < kKeys; ++q)
                        if (keys[q]) {
                            const bool mine = __builtin_amdgcn_inverse_ballot_w64(keys[q]);
                            const float su = wave_total(mine ? u : 0.0f), sl = wave_total(mine ? l : 0.0f);
                            if (lane == 0) {
                                float *s = sums + ((b - b0) * kKeys + q) * 2;
                                s[0] = s[0] + su;
                                s[1] = s[1] + sl;
                            }
                        }
                }
            }
            __syncthreads();
        }
    }

    // -- the successors of the shared cells: bound terms, rollout, reward ----
    if (shared) {
        // 32 lanes per successor c, lane i of them column i
        for (int c = c0 + (tid >> 5); c < c1; c += nt >> 5) {
            const int i = lane & 31;
            typename Ops::State sc;
            Ops::from_cell(sc, cell < 0 ? 0 : cell);
            const bool acts = cell >= 0 && Ops::acting(sc);
            const bool leaves = acts && Ops::walk(M, sc, c);  // moves the robot if c is a move
            const bool ends = cell < 0 || Ops::ended(sc);
            const int rx = __shfl(rock_x, i, 64), ry = __shfl(rock_y, i, 64);
            // a sampled rock is bad from now on
            const bool sampled = c == 4 && acts && i < m && Ops::at(sc, rx, ry);
            double v = 0.0;
            if (i < m && !sampled) v = term[Ops::rock_distance(sc, rx, ry)];
            if (i == kRockCols - 1) v = Ops::exits(M, sc, term);
            if (i < kRockCols) coef[c * kRockCols + i] = ends ? 0.0 : v;
            // the rewards of the live scenarios: ten for leaving; for a sample ten each way by the rock's quality
            int reward = leaves ? live_n : 0;
            const uint64_t hit = __ballot(sampled) >> (lane & 32);
            if ((uint32_t)hit) {
                const int q = __ffs((int)(uint32_t)hit) - 1;
                int good = 0;
#pragma unroll
                for (int sp = 0; sp < kSplits; ++sp) good += cnt[sp * kSplitSize + q];
                reward = 2 * good - live_n;
            }
            if (i == 0) {
                RockSucc s;
                s.value = 0.0;
                s.steps = 0;
                if (!ends) Ops::move_east(M, sc, R, term, s.value, s.steps);
                s.reward = reward;
                succ[c] = s;
            }
        }
    }
    // -- sizes and places of the children: 16 lanes per action, lane q of them key q ----
    for (int i = (nw - 1 - wid) * 4 + (lane >> 4); i < ((nb + 3) & ~3); i += nw * 4) {
        const int q = lane & 15, b = b0 + i;
        // of the live scenarios with robot 1's reading z1: all for a move; for a sense those reading good, reading
        // bad, and (robot 2 gone) reading nothing
        const int z1 = kTwo ? q / 3 : 0, z2 = kTwo ? q - 3 * z1 : q;
        int N = 0;
        if (i < nb && q < kKeys) {
            const RockSet w = rock_set<kTwo>(b, z2);
            const int32_t *row = cnt + z1 * kSplitSize + kRockCols - 1;
            if (w.from >= 0) N = row[w.from * kSetSize] - (w.minus >= 0 ? row[w.minus * kSetSize] : 0);
            if (q == 0) N += n - live_n;  // terminal scenarios read nothing
        }
        const int present = N > 0 ? 1 : 0;
        // inclusive prefixes over the 16 lanes: scenarios and children
        int incl = N | (present << 16);
        incl += dpp_srci<0x111, 0xf>(incl);
        incl += dpp_srci<0x112, 0xf>(incl);
        incl += dpp_srci<0x114, 0xf>(incl);
        incl += dpp_srci<0x118, 0xf>(incl);
        if (i < nb && q < kKeys) {
            place[i * kKeys + q] = ((incl & 0xFFFF) - N) | (((incl >> 16) - present) << 16);
            size[i * kKeys + q] = N;
        }
        if (i < nb && q == 15) T->n_children[a_first + i] = incl >> 16;
    }
    // scenarios in earlier chunks: of each split those reading rock j good (row j), acting (row kMaxRocks), and not
    // (row kMaxRocks + 1; with the terminal ones, which read nothing)
    for (int e = swapped_half(tid, nt); e < kSplits * 32; e += nt) {
        const int sp = e >> 5, row = e & 31;
        if (row < kRockSets && (row >= kMaxRocks || (row >= j0 && row < j1))) {
            uint16_t *out = pre + (sp * kRockSets + row) * nch;
            int run = 0;
#pragma unroll 4
            for (int t = 0; t < nch; ++t) {
                out[t] = (uint16_t)run;
                const uint64_t live = cmask[t], act = kTwo ? cmask[nch + t] : live;
                uint64_t s = live;
                if constexpr (kTwo) {
                    const uint64_t ga = cmask[2 * nch + t], gb = cmask[3 * nch + t];
                    s = sp == 0 ? live & ~(ga | gb) : sp == 1 ? ga : gb;
                }
                uint64_t v = row < kMaxRocks ? zmask[row * nch + t] : row == kMaxRocks ? act : ~act;
                v &= s;
                if (sp == 0 && row == kMaxRocks + 1) v |= chunk_mask(n, t) & ~live;
                run += __popcll(v);
            }
        }
    }
    __syncthreads();
    T = reread(T);

    // -- children, a lane each; few of them four lanes each, a quarter of the columns and then the quad's sum (one
    // lane's twenty columns take 2700 cycles, most of them waits), on other wavefronts than the leaf's first chunks --
    auto children = [&](auto lanes) {
        constexpr int kLanes = decltype(lanes)::value, kCols = kMaxRocks / kLanes;
        for (int g = swapped_half(tid, nt); g < nb * kKeys * kLanes; g += nt) {
            const int e = g / kLanes, part = g % kLanes;
            const int i = e / kKeys, q = e - i * kKeys, b = b0 + i, a = a_first + i;
            const int c = b >= 5 ? 5 : b;
            const int N = size[e], at0 = place[e], ci = at0 >> 16;
            if (N == 0) continue;  // (a quad's lanes together)
            float u0 = 0.0f, l0 = 0.0f;
            if (shared) {
                // the terms times the counts, and 1 / N to FP64's last places (the hardware's estimate and two Newton
                // steps), so the mean is rounded once
                const int z1 = kTwo ? q / 3 : 0, z2 = kTwo ? q - 3 * z1 : q;
                const RockSet w = rock_set<kTwo>(b, z2);
                const int32_t *from = cnt + z1 * kSplitSize + (w.from >= 0 ? w.from : 0) * kSetSize;
                const int32_t *minus = cnt + z1 * kSplitSize + (w.minus >= 0 ? w.minus : 0) * kSetSize;
                const int keep = w.from >= 0 ? -1 : 0, drop = w.minus >= 0 ? -1 : 0;
                const double *f = coef + c * kRockCols;
                double v = 0.0;
#pragma unroll
                for (int j = 0; j < kCols; ++j) {  // columns past the last rock hold 0
                    const int r = part * kCols + j;
                    v = __builtin_fma(f[r], (double)((from[r] & keep) - (minus[r] & drop)), v);
                }
                if constexpr (kLanes == 4) {
                    v = v + quad_swap<0xB1>(v);  // lanes 1 0 3 2
                    v = v + quad_swap<0x4E>(v);  // lanes 2 3 0 1
                }
                const double counted = (double)((from[kMaxRocks] & keep) - (minus[kMaxRocks] & drop));  // live ones
                const double dn = (double)N;
                double rn = __builtin_amdgcn_rcp(dn);
                rn = __builtin_fma(__builtin_fma(-dn, rn, 1.0), rn, rn);
                rn = __builtin_fma(__builtin_fma(-dn, rn, 1.0), rn, rn);
                u0 = (float)(__builtin_fma(f[kMaxRocks], counted, v) * rn);
                l0 = (float)(succ[c].value * counted * rn);
            }
            if (part == 0 && ci < cap) {
                if (!shared) u0 = sums[e * 2] / (float)N;
                if (!shared_l) l0 = sums[e * 2 + 1] / (float)N;
                const int64_t at = (int64_t)a * cap + ci;
                T->child_z[at] = (uint64_t)q;
                T->child_n[at] = N;
                T->child_off[at] = at0 & 0xFFFF;
                T->child_u0[at] = u0;
                T->child_l0[at] = l0;
            }
        }
    };
    if (nb * kKeys <= 16) children(std::integral_constant<int, 4>());
    else children(std::integral_constant<int, 1>());
    for (int i = nt - 1 - tid; i < nb; i += nt) {
        const int a = a_first + i, c = b0 + i >= 5 ? 5 : b0 + i;
        const int reward = misc[0] + (values ? misc[1 + 2 * c] : succ[c].reward);
        T->r_mean[a] = n > 0 ? 10.0f * (float)reward / (float)n : 0.0f;
        T->steps[2 * a + 0] = (int64_t)live_n;
        T->steps[2 * a + 1] = values ? (int64_t)misc[2 + 2 * c] : (int64_t)succ[c].steps * live_n;
    }

    // -- grouped order ------------------------------------------------------------
    // A wavefront takes a chunk and a share of the actions: a scenario's place is
    // its child's offset, plus the child's scenarios in earlier chunks, plus the
    // bits below its lane in the child's mask.
    int32_t *const child_of = T->child_of;
    const StatesPtr sprime = load_states(&T->sprime);
    const bool pair_out = has_states(sprime);
    const bool pairs = pair_out || T->r != nullptr || T->z != nullptr || child_of != nullptr;
    const int shares = nch > 0 && nw > nch ? nw / nch : 1;
    for (int unit = wid; unit < nch * shares; unit += nw) {
        const int t = unit / shares, share = unit - t * shares;
        const int k = t * 64 + lane;
        const bool valid = k < n;
        const uint64_t live = uniform_mask(cmask[t]), act = kTwo ? uniform_mask(cmask[nch + t]) : live;
        const uint64_t all = chunk_mask(n, t);
        uint64_t s[kSplits];  // live scenarios by robot 1's reading
        s[0] = live;
        if constexpr (kTwo) {
            s[1] = split ? uniform_mask(cmask[2 * nch + t]) : 0;
            s[2] = split ? uniform_mask(cmask[3 * nch + t]) : 0;
            s[0] = live & ~(s[1] | s[2]);
        }
        // lane j: rock j's mask and earlier counts; lane i: the offsets of action i's children
        const uint64_t zl = lane >= j0 && lane < j1 ? zmask[lane * nch + t] : 0;
        int before[kSplits], acting[kSplits], idle[kSplits], offs[kSplits];
#pragma unroll
        for (int sp = 0; sp < kSplits; ++sp) {
            const uint16_t *p = pre + sp * kRockSets * nch + t;
            before[sp] = lane >= j0 && lane < j1 ? p[lane * nch] : 0;
            acting[sp] = __builtin_amdgcn_readfirstlane(p[kMaxRocks * nch]);
            idle[sp] = __builtin_amdgcn_readfirstlane(p[(kMaxRocks + 1) * nch]);
            offs[sp] = lane < nb ? (place[lane * kKeys + 3 * sp + 1] & 0xFFFF) | (place[lane * kKeys + 3 * sp + 2] << 16) : 0;
        }
        // key 0 comes first: terminal scenarios, and for a sense those that do not act
        const uint64_t none = (all & ~live) | (s[0] & ~act);
        const int pos0 = rank_in(none, idle[0]);
        int16_t *const perm = T->perm + (int64_t)a_first * n;
        // moves: one child, or one per reading of robot 1
        int pos = k;
        for (int i = share; i < nb && b0 + i < 5; i += shares) {
            if (split) {
                pos = rank_in((all & ~live) | s[0], acting[0] + idle[0]);
#pragma unroll
                for (int sp = 1; sp < kSplits; ++sp) {
                    const int p = rank_in(s[sp], (place[i * kKeys + 3 * sp] & 0xFFFF) + acting[sp] + idle[sp]);
                    pos = __builtin_amdgcn_inverse_ballot_w64(s[sp]) ? p : pos;
                }
            }
            // scalar base, 32-bit offset
            if (valid) perm[(uint32_t)(i * n + pos)] = (int16_t)k;
        }
        auto sense_place = [&](int i) -> int {
            const int j = b0 + i - 5;
            const uint64_t z = lane_mask(zl, j);
            int pos = pos0;
#pragma unroll
            for (int sp = 0; sp < kSplits; ++sp) {
                if (sp > 0 && !s[sp]) continue;
                const uint64_t good = s[sp] & z, bad = s[sp] & act & ~z;
                const int o = __builtin_amdgcn_readlane(offs[sp], i), e = __builtin_amdgcn_readlane(before[sp], j);
                const int p1 = rank_in(good, (o & 0xFFFF) + e);
                const int p2 = rank_in(bad, (int)((uint32_t)o >> 16) + acting[sp] - e);
                pos = __builtin_amdgcn_inverse_ballot_w64(good) ? p1 : pos;
                pos = __builtin_amdgcn_inverse_ballot_w64(bad) ? p2 : pos;
                if (sp > 0 && (s[sp] & ~act)) {
                    const int p0 = rank_in(s[sp] & ~act, (place[i * kKeys + 3 * sp] & 0xFFFF) + idle[sp]);
                    pos = __builtin_amdgcn_inverse_ballot_w64(s[sp] & ~act) ? p0 : pos;
                }
            }
            return pos;
        };
        const int first = b0 >= 5 ? share : 5 - b0 + share;
#pragma unroll 2
        for (int i = first; i < nb; i += shares) {
            const int q = sense_place(i);
            if (valid) perm[(uint32_t)(i * n + q)] = (int16_t)k;
        }
        if (pairs && valid)
            for (int i = share; i < nb; i += shares) {
                const int b = b0 + i, a = a_first + i;
                const bool sense = b >= 5;
                const uint64_t me = 1ull << lane;
                int key = 0;
                if constexpr (kTwo) key = (s[1] & me) ? 3 : (s[2] & me) ? 6 : 0;
                if (sense && (act & me)) key += (zmask[(b - 5) * nch + t] & me) ? 1 : 2;
                typename Ops::State st;
                Ops::from_words(st, state[k], kTwo ? state[n + k] : 0);
                float r = 0.0f;
                if (!Ops::terminal(st)) {
                    if (!sense && Ops::acting(st)) r = Ops::mover(M, st, b);
                    Ops::settle(st);
                    if constexpr (kTwo) r = Ops::reward_of(state[k]) + r;
                }
                const int64_t pk = (int64_t)a * n + k;
                if (pair_out) Ops::store(M, sprime, pk, st);
                if (T->r) T->r[pk] = r;
                if (T->z) T->z[pk] = (uint64_t)key;
                if (child_of) child_of[pk] = place[i * kKeys + key] >> 16;
            }
    }
    __syncthreads();  // LDS is reused by the next tile
}

// Navigation: na actions [a0, a0 + na) of one leaf.
//
// What bounds it: instruction issue (the walks and the random blocks); the
// map, the update step, the random numbers of the step and the failure words
// of the rollouts are the same for all nine actions of a scenario, so a tile
// takes as many actions as its LDS holds (nav_tile_actions) and a lane does a
// scenario's actions one after another.  What an action yields is a word
// (NavCode) in LDS; rollouts of the default policy are settled from the walk
// and the failure words (NavOps::walk); rollouts step by step run a lane per
// scenario and action, which share their random words (153 leaves of two
// scenarios, random rollouts: 36 us with a tile per action, 70 with a lane
// running three actions in turn, 26 so).  Measured on 1024 leaves of 125..2000
// scenarios: 0.37 ms (1.1e8 VALU instructions of a wavefront, 0.48 of the
// issue slots) against 3.26 ms with one action per tile and every rollout
// step taken; eleven leaves of one to five scenarios 16 against 67 us.
//
// Grouping, one wavefront per action, so no barrier is needed between its
// passes: a count per observation (each key is its own table index), one
// scan over the keys for child offsets and indices, the grouped order -- a
// scenario's rank among the 64 of its chunk from one ballot per key bit --
// and segmented DPP scans over 64-aligned chunks of the grouped order, a
// child's chunk partials added in chunk order.  The floating-point order
// depends on the data alone, never on the width or the actions per tile.
struct NavCode {
    // bits 0-8 observation, 9-13 distance, 14-15 how the walk ends,
    // 16 settled, 17-29 moves of the walk; once settled, depths to its end
    // (stepped policies: steps of the rollout)
    static constexpr uint32_t kSettled = 1u << 16, kMax = 0x1fffu;
    __device__ static uint32_t make(uint32_t z, int d, int kind, bool settled, int m) {
        return z | ((uint32_t)d << 9) | ((uint32_t)kind << 14) | (settled ? kSettled : 0u) | ((uint32_t)m << 17);
    }
    __device__ static uint32_t obs(uint32_t c) { return c & 511u; }
    __device__ static int dist(uint32_t c) { return (int)((c >> 9) & 31u); }
    __device__ static int kind(uint32_t c) { return (int)((c >> 14) & 3u); }
    __device__ static int count(uint32_t c) { return (int)((c >> 17) & kMax); }
};

__device__ __forceinline__ void run_tile_nav(const HDX_CONST LeafTask *T, const int a0, const int na, unsigned char *lds) {
    using Ops = NavOps;
    const int n = T->n, cap = T->cap, nch = (n + 63) >> 6;
    const int tid = threadIdx.x, nt = blockDim.x, lane = lane_id(), wid = tid >> 6, nw = nt >> 6;
    const bool stepped = T->policy != HDX_POLICY_DEFAULT;
    const NavLayout Ly = make_nav_layout((uint32_t)(na * n), (uint32_t)na, (uint32_t)nch, (uint32_t)nw, stepped);
    double *gsum = (double *)(lds + Ly.gsum);
    float *ub = (float *)(lds + Ly.ub);
    uint32_t *code = (uint32_t *)(lds + Ly.code);
    float *val = (float *)(lds + Ly.val);
    uint32_t *rows = (uint32_t *)(lds + Ly.rows) + wid * (kNavRowBytes / 4) + lane;
    uint16_t *perm = (uint16_t *)(lds + Ly.perm);
    int32_t *cnt = (int32_t *)(lds + Ly.cnt);
    uint32_t *meta = (uint32_t *)(lds + Ly.meta);
    float *chunk_r = (float *)(lds + Ly.chunk_r);
    int32_t *expanded = (int32_t *)(lds + Ly.misc);
    const MView M = make_view(T->model);

    for (int j = tid; j <= kNavSums; j += nt) gsum[j] = M.gpow_sum(j);
    for (int d = tid; d <= Ops::kNoDistance; d += nt)
        ub[d] = d == Ops::kNoDistance ? 0.0f : 20.0f * M.gpow(d > 0 ? d - 1 : 1);
    for (int i = tid; i < na * kNavKeys; i += nt) cnt[i] = 0;
    if (tid == 0) *expanded = 0;
    __syncthreads();

    RolloutParams RP;
    RP.k0 = T->k0;
    RP.k1 = T->k1;
    RP.policy = T->policy;
    RP.const_action = T->const_action;
    RP.max_steps = T->max_steps;
    RP.max_depth = T->max_depth;
    RP.n_actions = T->n_actions;
    const int depth = T->depth, last_action = T->last_action;
    const int R = rollout_length(RP, depth + 1);
    const StatesPtr parent = load_states(&T->parent);
    const StatesPtr leaf_out = load_states(&T->out);
    const StatesPtr sprime = load_states(&T->sprime);
    const bool pair_out = has_states(sprime);

    // -- gather + update + expand + bounds + rollouts (Eq. 10, 12, 13) ------
    int my_exp = 0;
    for (int base = wid * 64; base < n; base += nt) {
        const int k = base + lane;
        const bool valid = k < n;
        Ops::State st;
        Ops::make_terminal(st);
        uint32_t id = 0;
        if (valid) {
            const uint32_t p = (uint16_t)T->idx[(uint32_t)k];
            id = T->parent_ids[p];
            Ops::load(M, parent, p, st);
        }
        Ops::make_rows(M, st, rows);
        if (last_action >= 0 && !Ops::terminal(st)) {
            float r0;
            Ops::move(M, rows, st, last_action,
                      last_action == 0 ? 0u : philox(id, (uint32_t)(depth - 1), 0, kTagStep, RP.k0, RP.k1).x, r0);
        }
        if (a0 == 0 && valid) {
            Ops::store(M, leaf_out, k, st);
            T->ids_out[k] = id;
        }
        const bool live = valid && !Ops::terminal(st);
        my_exp += live ? 1 : 0;
        uint32_t u_fail = 0, err = 0, around = 0;
        if (live) {
            u_fail = philox(id, (uint32_t)depth, 0, kTagStep, RP.k0, RP.k1).x;
            err = Ops::reading_errors(M, id, (uint32_t)depth, RP.k0, RP.k1);
            around = Ops::neighbours(M, rows, st.p & 15, (st.p >> 4) & 15);
        }
        const Ops::Target target = Ops::target_of(M, st);
        int need = 0;  // moves of the longest walk to settle
        for (int i = 0; i < na; ++i) {
            const int a = a0 + i;
            float r = 0.0f;
            uint32_t z = Ops::kTerminalObs;
            int d = Ops::kNoDistance, kind = Ops::kStuck, m = 0;
            bool settled = true;
            Ops::State s1 = st;
            if (live) {
                Ops::move(M, s1, a, u_fail, a == 0 ? 0 : (int)((around >> (a - 1)) & 1u), r);
                if (!Ops::terminal(s1)) {
                    const int x = s1.p & 15, y = (s1.p >> 4) & 15;
                    z = Ops::neighbours(M, rows, x, y) ^ err;
                    d = Ops::distance(M, s1);
                    if (R > 0 && !stepped) {
                        kind = Ops::walk(M, rows, target, x, y, R, m);
                        settled = kind == Ops::kOver || m == 0;
                        need = settled || need > m ? need : m;
                    } else {
                        kind = Ops::kOver;
                    }
                }
            }
            if (valid) {
                code[i * n + k] = NavCode::make(z, d, kind, settled, m);
                if (stepped) val[i * n + k] = __int_as_float(s1.p);  // for its rollout below
                const int64_t pk = (int64_t)a * n + k;
                if (pair_out) Ops::store(M, sprime, pk, s1);
                if (T->r) T->r[pk] = r;
                if (T->z) T->z[pk] = z;
                if (T->U) T->U[pk] = ub[d];
            }
            // mean step reward: sum of this 64-scenario chunk (lanes past n add 0)
            const float r_chunk = __ballot(r != 0.0f) ? wave_total(r) : 0.0f;
            if (lane == 0) chunk_r[i * nch + (base >> 6)] = r_chunk;
        }
        if (stepped) {
            // a lane per scenario and action, the actions of a scenario side by side
            const int per_wave = 64 / na, i = lane / na, c = lane - i * na;
            for (int l0 = 0; l0 < 64 && base + l0 < n; l0 += per_wave) {
                const int l = (l0 + i) & 63, kk = base + l;
                const bool mine = i < per_wave && l0 + i < 64 && kk < n;
                const int32_t p = mine ? __float_as_int(val[c * n + kk]) : 1 << 30;
                int ns;
                const float L = Ops::rollout_steps(M, RP, rows - lane + l, p, (uint32_t)__shfl((int)id, l, 64), depth + 1,
                                                   R, na, c, ns);
                if (mine) {
                    val[c * n + kk] = L;
                    code[c * n + kk] |= (uint32_t)ns << 17;
                }
            }
        }
        // the depth at which each walk's moves have all succeeded
        for (int from = 0; from < R && __ballot(need > 0);) {
            uint64_t F;
            const int j = Ops::failures(M, id, depth + 1, from, R, need, RP.k0, RP.k1, F);
            const int got = j - __popcll(F);
            if (need > 0) {
                for (int i = 0; i < na; ++i) {
                    const uint32_t c = code[i * n + k];
                    if (c & NavCode::kSettled) continue;
                    const int m = NavCode::count(c);
                    const bool done = m <= got;
                    const int v = done ? from + Ops::depths_until(F, m) : m - got;
                    code[i * n + k] =
                        (c & ~(NavCode::kMax << 17)) | ((uint32_t)v << 17) | (done ? NavCode::kSettled : 0u);
                }
            }
            need -= got;
            from += j;
        }
    }
    my_exp = wave_total_i(my_exp);
    if (lane == 0 && my_exp) atomicAdd(expanded, my_exp);
    __syncthreads();

    // -- grouping and per-child sums, one wavefront per action -----------------
    for (int i = wid; i < na; i += nw) {
        const int a = a0 + i;
        const uint32_t *codes = code + i * n;
        int32_t *next = cnt + i * kNavKeys;
        uint32_t *info = meta + i * kNavKeys;
        uint16_t *order = perm + i * n;
        for (int k = lane; k < n; k += 64) atomicAdd(&next[NavCode::obs(codes[k])], 1);
        wave_fence();
        // lane l owns keys 5 l .. 5 l + 4: packed scenario count and presence
        constexpr int kPer = (kNavKeys + 63) / 64;
        int c[kPer], sum = 0;
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int v = lane * kPer + e;
            c[e] = v < kNavKeys ? next[v] : 0;
            sum += c[e] + (c[e] > 0 ? 1 << 16 : 0);
        }
        int incl = sum;
        incl += dpp_srci<0x111, 0xf>(incl);
        incl += dpp_srci<0x112, 0xf>(incl);
        incl += dpp_srci<0x114, 0xf>(incl);
        incl += dpp_srci<0x118, 0xf>(incl);
        incl += dpp_srci<0x142, 0xa>(incl);
        incl += dpp_srci<0x143, 0xc>(incl);
        int run = incl - sum;
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int v = lane * kPer + e;
            if (c[e] > 0) {
                const int o = run & 0xFFFF, ci = run >> 16;
                next[v] = o;
                info[v] = ((uint32_t)ci << 16) | (uint32_t)c[e];
                if (ci < cap) {
                    const int64_t q = (int64_t)a * cap + ci;
                    T->child_z[q] = (uint64_t)v;
                    T->child_n[q] = c[e];
                    T->child_off[q] = o;
                }
                run += c[e] + (1 << 16);
            }
        }
        if (lane == 63) T->n_children[a] = incl >> 16;
        wave_fence();
        int32_t *const child_of = T->child_of;
        for (int t = 0; t < nch; ++t) {
            const int k = t * 64 + lane;
            const bool valid = k < n;
            const uint32_t key = valid ? NavCode::obs(codes[k]) : 511u;
            // the lanes of this chunk with the same key
            uint64_t same = ~0ull;
#pragma unroll
            for (int b = 0; b < 9; ++b) {
                const bool on = (key >> b) & 1u;
                const uint64_t bal = __ballot(on);
                same &= on ? bal : ~bal;
            }
            const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            if (valid) {
                const int at = next[key] + rank;
                order[at] = (uint16_t)k;
                if (child_of) child_of[(int64_t)a * n + k] = (int32_t)(info[key] >> 16);
                wave_fence();
                if (rank == 0) next[key] = at + __popcll(same);
            }
            wave_fence();
        }
        int steps = 0;
        float carry_u = 0.0f, carry_l = 0.0f;  // sums so far of a child that the last chunk did not end
        for (int t = 0; t < nch; ++t) {
            const int q = t * 64 + lane;
            const bool valid = q < n;
            const int k = valid ? order[q] : 0;
            const uint32_t cd = codes[k];
            const uint32_t key = NavCode::obs(cd);
            float u = 0.0f, l = 0.0f;
            int end = 0;
            uint32_t inf = 0;
            if (valid) {
                end = next[key];
                inf = info[key];
                u = ub[NavCode::dist(cd)];
                int s = 0;
                if (NavCode::dist(cd) != Ops::kNoDistance) {
                    if (stepped) {
                        l = val[i * n + k];
                        s = NavCode::count(cd);
                    } else {
                        const int kind = (cd & NavCode::kSettled) ? NavCode::kind(cd) : (int)Ops::kOver;
                        l = Ops::walk_value(kind, NavCode::count(cd), R,
                                            [&](int j) { return j <= kNavSums ? gsum[j] : M.gpow_sum(j); }, s);
                    }
                }
                steps += s;
                T->perm[(int64_t)a * n + q] = (int16_t)k;
                if (T->L) T->L[(int64_t)a * n + k] = l;
            }
            const int count = (int)(inf & 0xFFFFu);
            const int start = end - count;  // the child's first place
            int f = (!valid || q == start || lane == 0) ? 1 : 0;
            const bool carried = start < t * 64;  // the child began in an earlier chunk
            seg_step<0x111, 0xf>(u, l, f);
            seg_step<0x112, 0xf>(u, l, f);
            seg_step<0x114, 0xf>(u, l, f);
            seg_step<0x118, 0xf>(u, l, f);
            seg_step<0x142, 0xa>(u, l, f);
            seg_step<0x143, 0xc>(u, l, f);
            if (valid && carried) {
                u = carry_u + u;
                l = carry_l + l;
            }
            if (valid && q + 1 == end) {
                const int ci = (int)(inf >> 16);
                if (ci < cap) {
                    T->child_u0[(int64_t)a * cap + ci] = u / (float)count;
                    T->child_l0[(int64_t)a * cap + ci] = l / (float)count;
                }
            }
            carry_u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(u), 63));
            carry_l = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l), 63));
        }
        steps = wave_total_i(steps);
        if (lane == 0) {
            float tr = 0.0f;
            for (int t = 0; t < nch; ++t) tr = tr + chunk_r[i * nch + t];
            T->r_mean[a] = n > 0 ? tr / (float)n : 0.0f;
            T->steps[2 * a + 0] = (int64_t)*expanded;
            T->steps[2 * a + 1] = (int64_t)steps;
        }
    }
    __syncthreads();  // LDS is reused by the next tile
}

// One compare-exchange of a bitonic network over (key, position) pairs in
// LDS: elements i and i + stride of a run sorted in blocks of `size`.
__device__ __forceinline__ void exchange(uint64_t *keys, uint16_t *vals, int i, int stride, int size) {
    const uint64_t ka = keys[i], kb = keys[i + stride];
    const uint32_t va = vals[i], vb = vals[i + stride];
    const bool less = kb < ka || (kb == ka && vb < va);
    if (less == ((i & size) == 0)) {
        keys[i] = kb;
        keys[i + stride] = ka;
        vals[i] = (uint16_t)vb;
        vals[i + stride] = (uint16_t)va;
    }
}

// Sort the (key, position) pairs of the three actions, p2 (a power of two of
// at least 64) each, ascending.  Strides below 64 stay inside the 128
// elements (64 of a run of 64) that one wavefront handles, so only longer
// ones need a barrier.
__device__ __forceinline__ void sort_actions(uint64_t *zk, uint16_t *pos, int p2) {
    const int lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int block = p2 < 128 ? p2 : 128, blocks = kPedActions * p2 / block, half = p2 >> 1;
    const int log_half = 31 - __clz(half);
    for (int size = 2; size <= p2; size <<= 1) {
        int stride = size >> 1;
        for (; stride >= block; stride >>= 1) {
            for (int e = threadIdx.x; e < kPedActions * half; e += blockDim.x) {
                const int a = e >> log_half, q = e & (half - 1);
                const int i = ((q & ~(stride - 1)) << 1) | (q & (stride - 1));
                exchange(zk + a * p2, pos + a * p2, i, stride, size);
            }
            __syncthreads();
        }
        // the strides inside a block; every size up to a block at once
        const int top = size < block ? block : size;
        for (int b = wid; b < blocks; b += nw) {
            const int at = b * block, a = at / p2, o = at - a * p2;
            for (int sz = size < block ? 2 : size; sz <= top; sz <<= 1)
                for (int st = sz >> 1 < block ? sz >> 1 : block >> 1; st > 0; st >>= 1) {
                    if (lane < block >> 1)
                        exchange(zk + a * p2, pos + a * p2, o + (((lane & ~(st - 1)) << 1) | (lane & (st - 1))), st, sz);
                    wave_fence();
                }
        }
        __syncthreads();
        if (size < block) size = block;
    }
}

// Driving: the three actions of one leaf, a scenario on G lanes (PedLanes).
//
// What bounds it: instruction issue, two thirds of it the random blocks and
// the walks of the pedestrians.  These are the same for the three actions, so
// each pedestrian's step is taken once for all of them.  Four lanes per
// scenario with up to PM / 4 pedestrians each leave the work of a scenario
// within a few percent of one lane's (the cars are repeated on four lanes,
// their failure words drawn one depth per lane) and give four times the
// wavefronts at a third of the registers; 8 or 16 lanes (one or two pedestrians
// each) cost a quarter more work and are for leaves too few or too small to
// fill the GPU otherwise.
//
// A leaf's scenarios need each other only for the grouping.  Leaves enough to
// fill the GPU take a workgroup each for the whole (run_tile_ped; 512 leaves of
// 125..500 scenarios with 16 pedestrians and rollouts of 50 steps 0.51 ms, 2.4e8
// VALU instructions of a wavefront, 0.77 of the issue slots).  Fewer leave CUs
// idle and wait for the largest, and take two kernels: the scenarios of all
// leaves on whatever CUs are free (ped_rows), which leave each pair's
// observation, bounds, reward and steps in a workspace, and a workgroup per leaf
// that groups them.  One leaf of 500 scenarios takes 52 us so and 430 whole, 256
// of 50..500 among 768 RockSample leaves 485 and 620; at 512 leaves it
// is 618 and 505.  Leaves of up to kPedTile scenarios, three wavefronts, stay on
// one workgroup and one launch; so do, whole, those of persistent schedules and
// captured launches, which are to serve other leaves too.
//
// Grouping: (observation, position) pairs of the three actions sorted in LDS
// (the observations are hashes, most of them distinct), then one wavefront
// per action walks the grouped order with segmented DPP scans over 64-aligned
// chunks, a child's chunk partials added in chunk order.

// Scenarios begin + lane / G, + stride, ... of a leaf; a pair's results go to
// sink.stepped and, after its rollout, sink.rolled.
template <int G, int PP, class Sink>
__device__ __forceinline__ void ped_scenarios(const HDX_CONST LeafTask *T, int begin, int stride, Sink &sink) {
    constexpr int A = kPedActions;
    const int n = T->n, lane = lane_id();
    const MView M = make_view(T->model);
    RolloutParams RP;
    RP.k0 = T->k0;
    RP.k1 = T->k1;
    RP.policy = T->policy;
    RP.const_action = T->const_action;
    RP.max_steps = T->max_steps;
    RP.max_depth = T->max_depth;
    RP.n_actions = T->n_actions;
    const PedConst C = ped_const(M);
    const int depth = T->depth, last_action = T->last_action, P = C.n_peds;
    const int d0 = depth + 1, R = rollout_length(RP, d0);
    const StatesPtr parent = load_states(&T->parent);
    const StatesPtr leaf_out = load_states(&T->out);
    const StatesPtr sprime = load_states(&T->sprime);
    const bool pair_out = has_states(sprime);
    const int j = lane & (G - 1), first = lane & ~(G - 1);  // lane of the group, its first lane
    const int car = min(lane & 3, A - 1);                   // the action whose car this lane owns
    for (int base = begin; base < n; base += stride) {
        const int k = base + lane / G;
        const bool valid = k < n;
        PedLanes<G, PP> E;
        E.clear();
        uint32_t id = 0, goals = 0;  // four bits per slot
        float s = 0.0f, lv = 0.0f;
        bool live = false;
        int car_in = 0;
        if (valid) {
            const uint32_t p = (uint16_t)T->idx[(uint32_t)k];
            id = T->parent_ids[p];
            s = parent.s[p];
            car_in = parent.car[p];
            lv = (float)(car_in & 0xff);
            live = !((car_in >> 8) & 1);
#pragma unroll
            for (int q = 0; q < PP; ++q) {
                const int ped = q * G + j;
                if (ped < P) {
                    const int g = parent.goal[ped * parent.stride + p];
                    E.px[q] = parent.px[ped * parent.stride + p];
                    E.py[q] = parent.py[ped * parent.stride + p];
                    E.gx[q] = M.h->goal_x[g];
                    E.gy[q] = M.h->goal_y[g];
                    goals |= (uint32_t)g << (4 * q);
                }
            }
        }
        if (last_action >= 0) {
            if (live) {
                const bool failed = philox(id, (uint32_t)(depth - 1), 0, kTagStep, RP.k0, RP.k1).x < C.fail_thr;
                lv = ped_level(C, lv, (float)(1 - last_action), failed);
                s = ped_advance(C, s, lv);
                E.walk(C, j, id, (uint32_t)(depth - 1), RP.k0, RP.k1);
            }
            const uint32_t see = E.template look<A>(C, s, car);
            live &= !((lv > 0.0f) & ((see & 1u) != 0)) & !(s >= C.path_len);
        }
        if (valid) {
            if (j == 0) {
                leaf_out.s[k] = s;
                leaf_out.car[k] = (int)lv | (live ? 0 : 0x100);
                T->ids_out[k] = id;
            }
#pragma unroll
            for (int q = 0; q < PP; ++q) {
                const int ped = q * G + j;
                if (ped < P) {
                    leaf_out.px[ped * leaf_out.stride + k] = E.px[q];
                    leaf_out.py[ped * leaf_out.stride + k] = E.py[q];
                    leaf_out.goal[ped * leaf_out.stride + k] = (uint8_t)((goals >> (4 * q)) & 15u);
                }
            }
        }
        // the step of this lane's action
        if (live) {
            const bool failed = philox(id, (uint32_t)depth, 0, kTagStep, RP.k0, RP.k1).x < C.fail_thr;
            lv = ped_level(C, lv, (float)(1 - car), failed);
            s = ped_advance(C, s, lv);
            E.walk(C, j, id, (uint32_t)depth, RP.k0, RP.k1);
        }
        uint32_t see = E.template look<A>(C, s, car);
        const bool hit0 = (lv > 0.0f) & ((see & 1u) != 0), there0 = s >= C.path_len;
        const int code = !live ? 0 : hit0 ? 2 : there0 ? 3 : 1;
        const bool alive = live & !hit0 & !there0;
        const bool term = !alive;
        // the observation: a hash chained over the level and the floored positions, in pedestrian order
        uint64_t z = kPedTerminalObs;
        {
            uint64_t h = hash_field(0x243F6A8885A308D3ull, (int32_t)lv);
#pragma unroll
            for (int q = 0; q < PP; ++q) {
                if (q * G < P) {
                    const int fx = (int32_t)floorf(E.px[q]), fy = (int32_t)floorf(E.py[q]);
                    for (int i = 0; i < G && q * G + i < P; ++i) {
                        h = hash_field(h, __shfl(fx, first + i, 64));
                        h = hash_field(h, __shfl(fy, first + i, 64));
                    }
                }
            }
            if (alive) z = h == kPedTerminalObs ? kPedTerminalObs - 1 : h;
        }
        const float U = ped_upper(M, s, term ? 1 : 0);
        if (pair_out && valid) {
            if (j < A) {
                const int64_t at = (int64_t)j * n + k;
                sprime.s[at] = s;
                sprime.car[at] = (int)lv | (term ? 0x100 : 0);
            }
#pragma unroll
            for (int q = 0; q < PP; ++q) {
                const int ped = q * G + j;
                if (ped < P)
                    for (int a = 0; a < A; ++a) {
                        const int64_t at = ped * sprime.stride + (int64_t)a * n + k;
                        sprime.px[at] = E.px[q];
                        sprime.py[at] = E.py[q];
                        sprime.goal[at] = (uint8_t)((goals >> (4 * q)) & 15u);
                    }
            }
        }
        const bool mine = valid && j < A;
        const int64_t at = (int64_t)j * n + k;
        if (mine) {
            sink.stepped(j, k, z, U, code);
            if (T->r) T->r[at] = code == 0 ? 0.0f : code == 1 ? C.r_step : code == 2 ? C.r_hit : C.r_goal;
            if (T->z) T->z[at] = z;
            if (T->U) T->U[at] = U;
        }
        // the rollouts of the three actions together
        int steps;
        const float value = ped_rollout<A>(M, C, RP, E, car, id, d0, R, s, lv, see, alive, steps);
        if (mine) {
            sink.rolled(j, k, value, steps);
            if (T->L) T->L[at] = value;
        }
    }
}

// The tile of a leaf in LDS.
struct PedTile {
    uint64_t *zk;
    uint16_t *pos;
    float *ub, *lb;
    uint8_t *rc;
    int32_t *count;  // live scenarios, then rollout steps per action
    int32_t n, p2;
    int exp = 0, steps = 0;
    __device__ __forceinline__ PedTile(int n_, unsigned char *lds) : n(n_) {
        const PedLayout Ly = make_ped_layout(n);
        zk = (uint64_t *)(lds + Ly.zkey);
        pos = (uint16_t *)(lds + Ly.pos);
        ub = (float *)(lds + Ly.ub);
        lb = (float *)(lds + Ly.lb);
        rc = (uint8_t *)(lds + Ly.rcode);
        count = (int32_t *)(lds + Ly.misc);
        p2 = Ly.p2;
    }
    __device__ __forceinline__ void clear() {  // then a barrier
        const int tid = threadIdx.x, nt = blockDim.x;
        if (tid < 1 + kPedActions) count[tid] = 0;
        for (int i = tid; i < kPedActions * p2; i += nt)
            if ((i & (p2 - 1)) >= n) {
                zk[i] = kEmptyKey;
                pos[i] = 0xFFFFu;
            }
    }
    __device__ __forceinline__ void stepped(int a, int k, uint64_t z, float U, int code) {
        zk[a * p2 + k] = z;
        pos[a * p2 + k] = (uint16_t)k;
        ub[a * n + k] = U;
        rc[a * n + k] = (uint8_t)code;
        exp += a == 0 && code != 0 ? 1 : 0;
    }
    __device__ __forceinline__ void rolled(int a, int k, float L, int ns) {
        lb[a * n + k] = L;
        steps += ns;
    }
};

// Sort and children of a filled tile.
__device__ __forceinline__ void group_children(const HDX_CONST LeafTask *T, const PedTile &tile) {
    constexpr int A = kPedActions;
    const int n = tile.n, cap = T->cap, p2 = tile.p2;
    const int lane = lane_id(), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint64_t *const zk = tile.zk;
    uint16_t *const pos = tile.pos;
    const float *ub = tile.ub, *lb = tile.lb;
    const uint8_t *rc = tile.rc;
    const int32_t *count = tile.count;
    const PedConst C = ped_const(make_view(T->model));
    // -- observations ascending, positions ascending within one ----------------
    sort_actions(zk, pos, p2);

    // -- children and their sums, one wavefront per action -----------------------
    for (int a = wid; a < A; a += nw) {
        const uint64_t *z = zk + a * p2;
        const uint16_t *order = pos + a * p2;
        float carry_u = 0.0f, carry_l = 0.0f, tr = 0.0f;  // a child's sums so far; the rewards'
        int children = 0, open = 0;                       // children so far; the open child's first place
        int32_t *const child_of = T->child_of;
        for (int t = 0; t * 64 < n; ++t) {
            const int i = t * 64 + lane;
            const bool valid = i < n;
            const int k = valid ? order[i] : 0;
            const uint64_t key = valid ? z[i] : 0;
            const bool head = valid && (i == 0 || z[i - 1] != key);
            const bool last = valid && (i + 1 == n || z[i + 1] != key);
            const uint64_t heads = __ballot(head);
            const uint64_t mine = heads & (~0ull >> (63 - lane));  // heads at or below this lane
            const int start = mine ? t * 64 + 63 - __clzll((long long)mine) : open;
            const int ci = children + __popcll(mine) - 1;
            float u = valid ? ub[a * n + k] : 0.0f, l = valid ? lb[a * n + k] : 0.0f;
            int f = (head || !valid || lane == 0) ? 1 : 0;
            seg_step<0x111, 0xf>(u, l, f);
            seg_step<0x112, 0xf>(u, l, f);
            seg_step<0x114, 0xf>(u, l, f);
            seg_step<0x118, 0xf>(u, l, f);
            seg_step<0x142, 0xa>(u, l, f);
            seg_step<0x143, 0xc>(u, l, f);
            if (mine == 0) {
                u = carry_u + u;
                l = carry_l + l;
            }
            if (valid) {
                T->perm[(int64_t)a * n + i] = (int16_t)k;
                if (child_of) child_of[(int64_t)a * n + k] = ci;
            }
            if (last && ci < cap) {
                const int64_t at = (int64_t)a * cap + ci;
                const int cn = i + 1 - start;
                T->child_z[at] = key;
                T->child_n[at] = cn;
                T->child_off[at] = start;
                T->child_u0[at] = u / (float)cn;
                T->child_l0[at] = l / (float)cn;
            }
            carry_u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(u), 63));
            carry_l = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(l), 63));
            children += __popcll(heads);
            open = __builtin_amdgcn_readlane(start, 63);
            // mean step reward: this 64-scenario chunk in scenario order
            const int c = valid ? rc[a * n + i] : 0;
            const float r = c == 0 ? 0.0f : c == 1 ? C.r_step : c == 2 ? C.r_hit : C.r_goal;
            tr = tr + (__ballot(r != 0.0f) ? wave_total(r) : 0.0f);
        }
        if (lane == 0) {
            T->n_children[a] = children;
            T->r_mean[a] = n > 0 ? tr / (float)n : 0.0f;
            T->steps[2 * a + 0] = (int64_t)count[0];
            T->steps[2 * a + 1] = (int64_t)count[1 + a];
        }
    }
    __syncthreads();  // LDS is reused by the next tile
}


// A whole leaf on one workgroup.
template <int G, int PP>
__device__ __forceinline__ void run_tile_ped(const HDX_CONST LeafTask *T, unsigned char *lds) {
    const int wid = threadIdx.x >> 6, j = lane_id() & (G - 1);
    PedTile tile(T->n, lds);
    tile.clear();
    __syncthreads();
    ped_scenarios<G, PP>(T, wid * (64 / G), blockDim.x / G, tile);
    if (j < kPedActions && tile.exp) atomicAdd(&tile.count[0], tile.exp);
    if (j < kPedActions && tile.steps) atomicAdd(&tile.count[1 + j], tile.steps);
    __syncthreads();
    group_children(T, tile);
}

// A leaf's pairs between the two kernels, in its workspace: observation, U, L,
// reward code and steps.
struct PedEntries {
    uint64_t *z;
    float *u, *l;
    int32_t *code, *steps;
    int32_t n;
    __device__ __forceinline__ explicit PedEntries(const HDX_CONST LeafTask *T) : n(T->n) {
        const int pairs = kPedActions * n;
        z = (uint64_t *)T->work;
        u = (float *)(z + pairs);
        l = u + pairs;
        code = (int32_t *)(l + pairs);
        steps = code + pairs;
    }
    __device__ __forceinline__ void stepped(int a, int k, uint64_t z_, float U, int code_) {
        const int at = a * n + k;
        z[at] = z_;
        u[at] = U;
        code[at] = code_;
    }
    __device__ __forceinline__ void rolled(int a, int k, float L, int ns) {
        const int at = a * n + k;
        l[at] = L;
        steps[at] = ns;
    }
};

// The scenarios of workgroup `chunk` of a leaf.
template <int G, int PP>
__device__ __forceinline__ void ped_chunk(const HDX_CONST LeafTask *T, int chunk) {
    const int begin = chunk * (int)(blockDim.x / G) + (int)(threadIdx.x >> 6) * (64 / G);
    if (begin >= T->n) return;
    PedEntries entries(T);
    ped_scenarios<G, PP>(T, begin, T->n, entries);  // one round
}

// The children of a leaf whose scenarios are in its workspace.
__device__ __forceinline__ void run_tile_ped_grouping(const HDX_CONST LeafTask *T, unsigned char *lds) {
    PedTile tile(T->n, lds);
    tile.clear();
    __syncthreads();
    const PedEntries E(T);
    for (int a = 0; a < kPedActions; ++a) {
        tile.exp = tile.steps = 0;
        for (int k = threadIdx.x; k < tile.n; k += blockDim.x) {
            const int at = a * tile.n + k;
            tile.stepped(a, k, E.z[at], E.u[at], E.code[at]);
            tile.rolled(a, k, E.l[at], E.steps[at]);
        }
        const int exp = wave_total_i(tile.exp), steps = wave_total_i(tile.steps);
        if (lane_id() == 0) {
            if (exp) atomicAdd(&tile.count[0], exp);
            if (steps) atomicAdd(&tile.count[1 + a], steps);
        }
    }
    __syncthreads();
    group_children(T, tile);
}

__device__ __forceinline__ int remap_xcd(int b, int grid) {
    // workgroups are dealt to the 8 XCDs round-robin; give each XCD a
    // contiguous run of tiles so the tiles of one leaf share an L2
    const int x = b & 7, slot = b >> 3, base = grid >> 3, extra = grid & 7;
    return x * base + min(x, extra) + slot;
}

// MODE 0: RockSample only; 1: crowd driving only; 2: both; 3: multi-agent
// RockSample only; 4: navigation only; 5: crowd driving, the grouping of leaves
// whose scenarios ped_rows has expanded.  Workgroups of the RockSample tiles are
// capped at 512 lanes; driving (mixed calls and the grouping too) and navigation
// take up to 1024, because one large leaf's LDS carve-up leaves room for one
// workgroup per CU.
template <int MODE>
constexpr bool rock_mode() { return MODE == 0 || MODE == 3; }
template <int MODE>
constexpr int max_threads() { return rock_mode<MODE>() ? 512 : 1024; }
// RockSample tiles: keep 7 wavefronts per SIMD resident (at most 72 VGPRs,
// no spills); the others' register state decides their own.
template <int MODE>
constexpr int min_waves() { return rock_mode<MODE>() ? 7 : 1; }

// Lanes per scenario of the driving tiles: at most four pedestrians per lane,
// or (kSpread) one or two.
template <int PM, bool kSpread>
constexpr int ped_lanes() { return !kSpread ? (PM == 32 ? 8 : 4) : PM == 8 ? 8 : 16; }

// Actions of the tile that begins at action a: no more than its row has left
// (only with two robots is a row less than all actions).
template <int MODE>
__device__ __forceinline__ int tile_width(const HDX_CONST LeafTask *T, int a) {
    const int row = T->row_actions;
    return min((int)T->tile_actions, row - (MODE == 3 ? a % row : a));
}

template <int MODE, int PM, bool kSpread>
__device__ __forceinline__ void run_mode(const HDX_CONST LeafTask *T, int a, unsigned char *lds) {
    if constexpr (MODE == 3) {
        run_tile_rocks<MarsOps>(T, a, tile_width<MODE>(T, a), lds);
    } else if constexpr (MODE == 4) {
        run_tile_nav(T, a, tile_width<MODE>(T, a), lds);
    } else if (MODE == 0 || (MODE == 2 && T->kind == HDX_ROCKSAMPLE)) {
        run_tile_rocks<RsOps>(T, a, tile_width<MODE>(T, a), lds);
    } else if constexpr (MODE == 1 || MODE == 2) {
        run_tile_ped<ped_lanes<PM, kSpread>(), PM / ped_lanes<PM, kSpread>()>(T, lds);
    } else if constexpr (MODE == 5) {
        run_tile_ped_grouping(T, lds);
    }
}

template <int MODE, int PM, bool kSpread = false>
__global__ __launch_bounds__(max_threads<MODE>(), min_waves<MODE>()) void expand_tiles(const LeafTask *tasks,
                                                                                       const Tile *tiles,
                                                                                       TileQueue *queue,
                                                                                       int32_t step,
                                                                                       int32_t xcd_remap) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int32_t s_tile;
    const int32_t n_tiles = __builtin_amdgcn_readfirstlane(queue->n_tiles);
    // step: 0 a tile per workgroup; -1 tiles from the queue; else from its own place on every step-th tile (the place
    // kept in LDS: in a register that the tiles are short of it cost every launch 0.4 to 0.8 %)
    int iter = 0;
    for (;;) {
        int t;
        if (step) {
            if (threadIdx.x == 0) s_tile = step < 0 ? atomicAdd(&queue->next, 1) : iter > 0 ? s_tile + step : (int)blockIdx.x;
            __syncthreads();
            t = __builtin_amdgcn_readfirstlane(s_tile);
            __syncthreads();
        } else {
            if (iter > 0) break;
            t = xcd_remap ? remap_xcd((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x;
        }
        ++iter;
        if (t >= n_tiles) break;
        const HDX_CONST Tile *tile = (const HDX_CONST Tile *)(tiles + t);
        const HDX_CONST LeafTask *T = (const HDX_CONST LeafTask *)(tasks + tile->leaf);
        run_mode<MODE, PM, kSpread>(T, tile->action, lds);
    }
    if (step < 0 && threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&queue->done, 1) == (int)gridDim.x - 1) {
            queue->next = 0;
            queue->done = 0;
            __threadfence();
        }
    }
}

// One of a call's leaves has ended; the last of them tells the host.
__device__ __forceinline__ void end_ped_leaf(PedHead *head, uint32_t n_leaves) {
    __threadfence();
    if (atomicAdd(&head->left, 1u) != n_leaves - 1) return;
    head->left = 0;
    const uint32_t ended = atomicAdd(&head->ended, 1u) + 1u;
    __hip_atomic_store(head->host, ended, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A few leaves carried in the kernel arguments: no descriptor staging, so
// the launch is ordered by its stream alone.  The pack is read in place in
// the kernarg segment (constant address space, scalar loads).
template <int MODE, int PM>
__global__ __launch_bounds__(max_threads<MODE>()) void expand_args(const ArgPack pack) {
    extern __shared__ __align__(16) unsigned char lds[];
#if defined(__HIP_DEVICE_COMPILE__)
    const HDX_CONST ArgPack *P = (const HDX_CONST ArgPack *)__builtin_amdgcn_kernarg_segment_ptr();
#else
    const ArgPack *P = &pack;
#endif
    // the grid is the number of tiles (never remapped or rounded up here); each read below waits for the one before
    // it, so a single leaf takes none
    const int n_leaves = P->n_leaves, t = (int)blockIdx.x;
    int i = 0;
    while (i + 1 < n_leaves && t >= P->tile_end[i]) ++i;
    const HDX_CONST LeafTask *T = &P->t[i];
    const int local = i > 0 ? t - P->tile_end[i - 1] : t;
    int a = local * T->tile_actions;
    if (MODE == 3) {
        const int per_row = (T->row_actions + T->tile_actions - 1) / T->tile_actions, row = local / per_row;
        a = row * T->row_actions + (local - row * per_row) * T->tile_actions;
    }
    run_mode<MODE, PM, true>(T, a, lds);
    if constexpr (MODE == 5)  // (a leaf is a tile; all have read their workspace)
        if (threadIdx.x == 0) end_ped_leaf((PedHead *)(P->t[0].work - kPedHeadBytes), (uint32_t)n_leaves);
}

// Driving, the scenarios of many leaves: `chunks` workgroups per tile of the
// queue (a tile is a leaf), those past the leaf's scenarios ending at once.  Two
// pedestrians per lane where the tiles take four: shorter wavefronts, five of
// them per SIMD (341 leaves of 31..500 scenarios 429 us, 491 with four).
constexpr int kPedRowThreads = 256;
template <int PM, bool kSpread>
constexpr int row_lanes() { return !kSpread && PM > 8 ? PM / 2 < 16 ? PM / 2 : 16 : ped_lanes<PM, kSpread>(); }
template <int PM, bool kSpread>
__global__ __launch_bounds__(kPedRowThreads, 5) void ped_rows(const LeafTask *tasks, const Tile *tiles,
                                                           const TileQueue *queue, int32_t chunks) {
    const int t = (int)blockIdx.x / chunks;
    if (t >= __builtin_amdgcn_readfirstlane(queue->n_tiles)) return;
    const HDX_CONST LeafTask *T = (const HDX_CONST LeafTask *)(tasks + ((const HDX_CONST Tile *)(tiles + t))->leaf);
    ped_chunk<row_lanes<PM, kSpread>(), PM / row_lanes<PM, kSpread>()>(T, (int)blockIdx.x - t * chunks);
}

// The same of a few leaves in the kernel arguments; blockIdx.y selects the leaf.
template <int PM>
__global__ __launch_bounds__(kPedRowThreads, 4) void ped_rows_args(const ArgPack pack) {
#if defined(__HIP_DEVICE_COMPILE__)
    const HDX_CONST ArgPack *P = (const HDX_CONST ArgPack *)__builtin_amdgcn_kernarg_segment_ptr();
#else
    const ArgPack *P = &pack;
#endif
    ped_chunk<row_lanes<PM, true>(), PM / row_lanes<PM, true>()>(&P->t[blockIdx.y], (int)blockIdx.x);
}

// Dynamic LDS of one workgroup for leaves of up to n_max scenarios, tiles of up
// to `pairs` words (tile_pairs).
template <int MODE>
uint32_t lds_bytes(int32_t n_max, int32_t pairs, int32_t threads) {
    if (rock_mode<MODE>()) return make_rock_layout(n_max, std::max(n_max, pairs), MODE == 3).total;
    if (MODE == 1 || MODE == 5) return make_ped_layout(n_max).total;
    if (MODE == 2)
        return std::max(make_rock_layout(n_max, std::max(n_max, pairs), false).total, make_ped_layout(n_max).total);
    return nav_lds(n_max, pairs, threads);
}

template <class K>
hipError_t allow_lds(K *kernel) {
    return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxDynamicLds);
}
template <int MODE, int PM>
hipError_t configure_t() {
    hipError_t e = allow_lds(expand_args<MODE, PM>);
    if constexpr (MODE != 2)  // calls that mix the two models launch one kernel per model
        if (e == hipSuccess) e = allow_lds(expand_tiles<MODE, PM>);
    if constexpr (MODE == 1)
        if (e == hipSuccess) e = allow_lds(expand_tiles<MODE, PM, true>);
    return e;
}

template <int MODE, int PM>
hipError_t launch_args_t(const ArgPack &pack, const Variant &v, const Schedule &sch, hipStream_t stream) {
    const int grid = pack.tile_end[pack.n_leaves - 1];
    if (grid < 1) return hipSuccess;
    const int threads = sch.threads > max_threads<MODE>() ? max_threads<MODE>() : sch.threads;
    hipLaunchKernelGGL((expand_args<MODE, PM>), dim3(grid), dim3(threads),
                       lds_bytes<MODE>(v.n_max, v.pairs, threads), stream, pack);
    return hipGetLastError();
}

template <int MODE, int PM, bool kSpread = false>
hipError_t launch_expand_t(const LeafTask *d_tasks, const Tile *d_tiles, TileQueue *d_queue, int32_t n_tiles,
                           int32_t n_max, int32_t pairs, const Schedule &sch, int32_t n_cu, hipStream_t stream) {
    // persistent: a fixed grid that drains the tile queue, so a captured
    // graph stays valid for any tile count
    const int grid = sch.persistent > 0 ? n_cu * sch.persistent : n_tiles;
    if (grid < 1) return hipSuccess;
    const int threads = sch.threads > max_threads<MODE>() ? max_threads<MODE>() : sch.threads;
    const int step = sch.persistent > 0 ? -1 : sch.persistent == kStrided ? grid : 0;
    hipLaunchKernelGGL((expand_tiles<MODE, PM, kSpread>), dim3(grid), dim3(threads),
                       lds_bytes<MODE>(n_max, pairs, threads), stream, d_tasks, d_tiles, d_queue, step, sch.xcd_remap);
    return hipGetLastError();
}

// Workgroups of ped_rows for a leaf of n scenarios.
template <int PM, bool kSpread>
int ped_chunks(int32_t n) {
    return (n * row_lanes<PM, kSpread>() + kPedRowThreads - 1) / kPedRowThreads;
}

template <int PM, bool kSpread>
hipError_t launch_ped_t(const LeafTask *d_tasks, const Tile *d_tiles, TileQueue *d_queue, int32_t n_tiles, int32_t n_max,
                        const Schedule &sch, int32_t n_cu, hipStream_t stream) {
    const int chunks = ped_chunks<PM, kSpread>(n_max);
    if (n_tiles < 1) return hipSuccess;
    if ((int64_t)chunks * n_tiles > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((ped_rows<PM, kSpread>), dim3((unsigned)(chunks * n_tiles)), dim3(kPedRowThreads), 0, stream,
                       d_tasks, d_tiles, d_queue, chunks);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_expand_t<5, 1>(d_tasks, d_tiles, d_queue, n_tiles, n_max, 0, sch, n_cu, stream) : e;
}

template <int PM>
hipError_t launch_ped_args_t(const ArgPack &pack, const Variant &v, const Schedule &sch, hipStream_t stream) {
    hipLaunchKernelGGL((ped_rows_args<PM>), dim3(ped_chunks<PM, true>(v.n_max), pack.n_leaves), dim3(kPedRowThreads),
                       0, stream, pack);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_args_t<5, 1>(pack, v, sch, stream) : e;
}

// ---------------------------------------------------------------------------
// sample_scenarios
// ---------------------------------------------------------------------------
// The arguments (belief thresholds, ~3.6 KB) are read from device memory.
__global__ void sample_kernel(const SampleArgs *args) {
    const HDX_CONST SampleArgs &A = *(const HDX_CONST SampleArgs *)args;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= A.K) return;
    const HDX_CONST ModelHdr *M = (const HDX_CONST ModelHdr *)&A.model->h;
    const StatesPtr &S = A.out;
    if (M->kind == HDX_ROCKSAMPLE) {
        int32_t w = A.x0 | (A.y0 << 5);
        uint4 u = make_uint4(0, 0, 0, 0);
        for (int i = 0; i < M->n_rocks; ++i) {
            if ((i & 3) == 0) u = philox((uint32_t)k, 0, (uint32_t)(i >> 2), kTagInit, A.k0, A.k1);
            const uint32_t word = (i & 3) == 0 ? u.x : (i & 3) == 1 ? u.y : (i & 3) == 2 ? u.z : u.w;
            if ((uint64_t)word < A.rock_thr[i]) w |= 1 << (10 + i);
        }
        S.w[k] = w;
    } else if (M->kind == HDX_MARS) {
        // the robots' row is known; rock i good as for RockSample
        int32_t rk = 0;
        uint4 u = make_uint4(0, 0, 0, 0);
        for (int i = 0; i < M->n_rocks; ++i) {
            if ((i & 3) == 0) u = philox((uint32_t)k, 0, (uint32_t)(i >> 2), kTagInit, A.k0, A.k1);
            const uint32_t word = (i & 3) == 0 ? u.x : (i & 3) == 1 ? u.y : (i & 3) == 2 ? u.z : u.w;
            if ((uint64_t)word < A.rock_thr[i]) rk |= 1 << i;
        }
        S.w[k] = A.x0;
        S.w[S.stride + k] = rk;
    } else if (M->kind == HDX_NAV) {
        // robot on row 0 at a uniform column; one gate open; other unknown
        // cells occupied at their prior (draw i = word i % 4 of block i / 4)
        uint4 u = philox((uint32_t)k, 0, 0, kTagInit, A.k0, A.k1);
        const int x = (int)(((uint64_t)u.x * (uint64_t)M->grid) >> 32);
        uint32_t m0 = u.y < 0x80000000u ? 2u : 1u, m1 = 0, m2 = 0, m3 = 0;
        for (int i = 2; i < A.n_unknown; ++i) {
            if ((i & 3) == 0) u = philox((uint32_t)k, 0, (uint32_t)(i >> 2), kTagInit, A.k0, A.k1);
            const uint32_t word = (i & 3) == 0 ? u.x : (i & 3) == 1 ? u.y : (i & 3) == 2 ? u.z : u.w;
            if ((uint64_t)word < A.cell_thr[i]) {
                const uint32_t bit = 1u << (i & 31);
                if (i < 32) m0 |= bit;
                else if (i < 64) m1 |= bit;
                else if (i < 96) m2 |= bit;
                else m3 |= bit;
            }
        }
        S.w[k] = x;
        S.w[S.stride + k] = (int32_t)m0;
        S.w[2 * S.stride + k] = (int32_t)m1;
        S.w[3 * S.stride + k] = (int32_t)m2;
        S.w[4 * S.stride + k] = (int32_t)m3;
    } else {
        S.s[k] = A.s0;
        S.car[k] = A.level0 & 0xff;
        uint4 u = make_uint4(0, 0, 0, 0);
        for (int j = 0; j < M->n_peds; ++j) {
            if ((j & 3) == 0) u = philox((uint32_t)k, 0, (uint32_t)(j >> 2), kTagInit, A.k0, A.k1);
            const uint32_t word = (j & 3) == 0 ? u.x : (j & 3) == 1 ? u.y : (j & 3) == 2 ? u.z : u.w;
            int g = M->n_goals - 1;
            for (int q = 0; q < M->n_goals - 1; ++q) {
                if ((uint64_t)word < A.goal_thr[j][q]) {
                    g = q;
                    break;
                }
            }
            S.px[j * S.stride + k] = A.px0[j];
            S.py[j * S.stride + k] = A.py0[j];
            S.goal[j * S.stride + k] = (uint8_t)g;
        }
    }
}

// ---------------------------------------------------------------------------
// rollout_bounds: one lane per state
// ---------------------------------------------------------------------------
__device__ __forceinline__ RolloutParams bounds_params(const BoundsArgs &A, const MView &M) {
    RolloutParams RP;
    RP.k0 = A.k0;
    RP.k1 = A.k1;
    RP.policy = A.policy;
    RP.const_action = A.const_action;
    RP.max_steps = A.max_steps;
    RP.max_depth = A.max_depth;
    RP.n_actions = M.h->n_actions;
    return RP;
}

// RockSample, either model: a lane per state.
template <class Ops>
__global__ __launch_bounds__(256) void bounds_rocks(const BoundsArgs A) {
    __shared__ float term[kRockTerms];  // 10 gamma^d
    __shared__ uint32_t effects[kRockCells];
    const MView M = make_view(A.model);
    for (int d = threadIdx.x; d < kRockTerms; d += blockDim.x) term[d] = 10.0f * M.gpow(d);
    stage_effects(M, effects);
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = k < A.n;
    typename Ops::State st;
    Ops::make_terminal(st);
    if (valid) Ops::load(M, A.states, k, st);
    const RolloutParams RP = bounds_params(A, M);
    const int d0 = valid ? A.depths[k] : 0, R = rollout_length(RP, d0);
    int ns;
    const float L = RP.policy == HDX_POLICY_DEFAULT
                        ? Ops::rollout_east(M, st, R, ns)
                        : rock_rollout<Ops>(M, effects, RP, valid ? A.ids[k] : 0u, d0, R, Ops::team(M, st), 1, 0, ns);
    if (!valid) return;
    A.U[k] = Ops::upper(M, st, [&](int d) { return term[d]; });
    A.L[k] = L;
    if (A.steps) A.steps[k] = ns;
}

// Driving: a state on G lanes, as in the tiles.
template <int G, int PP>
__global__ __launch_bounds__(256) void bounds_ped(const BoundsArgs A) {
    const MView M = make_view(A.model);
    const PedConst C = ped_const(M);
    const RolloutParams RP = bounds_params(A, M);
    const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
    const bool valid = k < A.n;
    const int j = lane_id() & (G - 1);
    PedLanes<G, PP> E;
    E.clear();
    float s = 0.0f, lv = 0.0f;
    bool live = false;
    uint32_t id = 0;
    int d0 = 0;
    if (valid) {
        s = A.states.s[k];
        const int32_t car = A.states.car[k];
        lv = (float)(car & 0xff);
        live = !((car >> 8) & 1);
        id = A.ids[k];
        d0 = A.depths[k];
#pragma unroll
        for (int q = 0; q < PP; ++q) {
            const int ped = q * G + j;
            if (ped < C.n_peds) {
                const int g = A.states.goal[ped * A.states.stride + k];
                E.px[q] = A.states.px[ped * A.states.stride + k];
                E.py[q] = A.states.py[ped * A.states.stride + k];
                E.gx[q] = M.h->goal_x[g];
                E.gy[q] = M.h->goal_y[g];
            }
        }
    }
    const uint32_t see = E.template look<1>(C, s, 0);
    int ns;
    const float L = ped_rollout<1>(M, C, RP, E, 0, id, d0, rollout_length(RP, d0), s, lv, see, live, ns);
    if (!valid || j != 0) return;
    A.U[k] = ped_upper(M, s, live ? 0 : 1);
    A.L[k] = L;
    if (A.steps) A.steps[k] = ns;
}

// Navigation: the map's rows in LDS, the wavefront's lanes together.
__global__ __launch_bounds__(256) void bounds_nav(const BoundsArgs A) {
    __shared__ uint32_t rows_lds[4 * kNavRowBytes / 4];
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = k < A.n;
    const MView M = make_view(A.model);
    NavOps::State st;
    NavOps::make_terminal(st);
    if (valid) NavOps::load(M, A.states, k, st);
    uint32_t *rows = rows_lds + (threadIdx.x >> 6) * (kNavRowBytes / 4) + lane_id();
    NavOps::make_rows(M, st, rows);
    const RolloutParams RP = bounds_params(A, M);
    const int d0 = valid ? A.depths[k] : 0;
    int ns = 0;
    const float L = NavOps::rollout(M, RP, rows, st, valid ? A.ids[k] : 0u, d0, rollout_length(RP, d0), valid, ns);
    if (!valid) return;
    A.U[k] = NavOps::upper(M, st);
    A.L[k] = L;
    if (A.steps) A.steps[k] = ns;
}

// FP32 rounding self-test: the operations the models' state updates use.
__global__ void fp32_selftest_kernel(const float *a, const float *b, const float *c, int64_t n, float *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = a[i], y = b[i], z = c[i];
    out[i] = __builtin_sqrtf(fabsf(x));
    out[n + i] = x / y;
    out[2 * n + i] = x * y + z;
    out[3 * n + i] = floorf(x);
}

__global__ void philox_kernel(const uint32_t *ctr, int64_t count, uint32_t k0, uint32_t k1, uint32_t *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const uint4 c = reinterpret_cast<const uint4 *>(ctr)[i];
    reinterpret_cast<uint4 *>(out)[i] = philox(c.x, c.y, c.z, c.w, k0, k1);
}

}  // namespace

hipError_t launch_fp32_selftest(const float *a, const float *b, const float *c, int64_t n, float *out,
                                hipStream_t stream) {
    const int threads = 256;
    const int64_t blocks = (n + threads - 1) / threads;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(fp32_selftest_kernel, dim3((unsigned)blocks), dim3(threads), 0, stream, a, b, c, n, out);
    return hipGetLastError();
}

Variant pick_variant(int32_t has_rs, int32_t has_ped, int32_t ped_max, int32_t n_max, int32_t has_mars,
                     int32_t has_nav) {
    Variant v;
    v.mode = has_nav ? 4 : has_mars ? 3 : !has_ped ? 0 : (has_rs ? 2 : 1);
    v.pm = !has_ped ? 1 : ped_max <= 8 ? 8 : ped_max <= 16 ? 16 : 32;
    v.n_max = n_max < 1 ? 1 : n_max;
    return v;
}

int32_t variant_max_threads(const Variant &v) { return v.mode == 0 || v.mode == 3 ? max_threads<0>() : max_threads<1>(); }

int32_t variant_lanes(const Variant &v, int32_t n) {
    if (v.mode != 1 && v.mode != 2) return n;
    return n * (!v.group ? (v.pm == 32 ? 8 : 4) : v.pm <= 8 ? 8 : 16);
}

hipError_t configure_expand_kernels() {
    hipError_t e = configure_t<0, 1>();
    if (e == hipSuccess) e = configure_t<1, 8>();
    if (e == hipSuccess) e = configure_t<1, 16>();
    if (e == hipSuccess) e = configure_t<1, 32>();
    if (e == hipSuccess) e = configure_t<5, 1>();
    if (e == hipSuccess) e = configure_t<2, 8>();
    if (e == hipSuccess) e = configure_t<2, 16>();
    if (e == hipSuccess) e = configure_t<2, 32>();
    if (e == hipSuccess) e = configure_t<3, 1>();
    if (e == hipSuccess) e = configure_t<4, 1>();
    return e;
}

hipError_t launch_expand(const LeafTask *d_tasks, const Tile *d_tiles, TileQueue *d_queue, int32_t n_tiles,
                         const Variant &v, const Schedule &sch, int32_t n_cu, hipStream_t stream) {
#define HDX_LAUNCH(M, P) launch_expand_t<M, P>(d_tasks, d_tiles, d_queue, n_tiles, v.n_max, v.pairs, sch, n_cu, stream)
#define HDX_LAUNCH_G(P) launch_expand_t<1, P, true>(d_tasks, d_tiles, d_queue, n_tiles, v.n_max, v.pairs, sch, n_cu, stream)
#define HDX_LAUNCH_ROWS(P, G) launch_ped_t<P, G>(d_tasks, d_tiles, d_queue, n_tiles, v.n_max, sch, n_cu, stream)
    if (v.mode == 0) return HDX_LAUNCH(0, 1);
    if (v.mode == 3) return HDX_LAUNCH(3, 1);
    if (v.mode == 4) return HDX_LAUNCH(4, 1);
    if (v.rows && v.n_max > kPedTile) {
        if (v.group)
            return v.pm == 8 ? HDX_LAUNCH_ROWS(8, true) : v.pm == 16 ? HDX_LAUNCH_ROWS(16, true) : HDX_LAUNCH_ROWS(32, true);
        return v.pm == 8 ? HDX_LAUNCH_ROWS(8, false) : v.pm == 16 ? HDX_LAUNCH_ROWS(16, false) : HDX_LAUNCH_ROWS(32, false);
    }
    if (v.group) return v.pm == 8 ? HDX_LAUNCH_G(8) : v.pm == 16 ? HDX_LAUNCH_G(16) : HDX_LAUNCH_G(32);
    return v.pm == 8 ? HDX_LAUNCH(1, 8) : v.pm == 16 ? HDX_LAUNCH(1, 16) : HDX_LAUNCH(1, 32);
#undef HDX_LAUNCH_G
#undef HDX_LAUNCH_ROWS
#undef HDX_LAUNCH
}

hipError_t launch_expand_args(const ArgPack &pack, const Variant &v, const Schedule &sch, hipStream_t stream) {
#define HDX_LAUNCH(M, P) launch_args_t<M, P>(pack, v, sch, stream)
    if (v.mode == 0) return HDX_LAUNCH(0, 1);
    if (v.mode == 3) return HDX_LAUNCH(3, 1);
    if (v.mode == 4) return HDX_LAUNCH(4, 1);
    if (v.mode == 1 && !(v.rows && v.n_max > kPedTile))
        return v.pm == 8 ? HDX_LAUNCH(1, 8) : v.pm == 16 ? HDX_LAUNCH(1, 16) : HDX_LAUNCH(1, 32);
    if (v.mode == 1)
        return v.pm == 8    ? launch_ped_args_t<8>(pack, v, sch, stream)
               : v.pm == 16 ? launch_ped_args_t<16>(pack, v, sch, stream)
                            : launch_ped_args_t<32>(pack, v, sch, stream);
    return v.pm == 8 ? HDX_LAUNCH(2, 8) : v.pm == 16 ? HDX_LAUNCH(2, 16) : HDX_LAUNCH(2, 32);
#undef HDX_LAUNCH
}

hipError_t launch_sample(const SampleArgs *d_args, int32_t K, hipStream_t stream) {
    const int threads = 256;
    const int blocks = (K + threads - 1) / threads;
    if (blocks < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sample_kernel, dim3(blocks), dim3(threads), 0, stream, d_args);
    return hipGetLastError();
}

namespace {
template <int PM>
hipError_t launch_bounds_ped(const BoundsArgs &args, hipStream_t stream) {
    constexpr int threads = 256, g = ped_lanes<PM, false>();
    constexpr int64_t most = kLaunchThreads / g;
    for (int64_t at = 0; at < args.n; at += most) {
        BoundsArgs part = args;
        part.states = states_from(args.states, at);
        part.ids = args.ids + at;
        part.depths = args.depths + at;
        part.U = args.U + at;
        part.L = args.L + at;
        part.steps = args.steps ? args.steps + at : nullptr;
        part.n = std::min(most, args.n - at);
        hipLaunchKernelGGL((bounds_ped<g, PM / g>), dim3((unsigned)((part.n * g + threads - 1) / threads)), dim3(threads),
                           0, stream, part);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
}  // namespace

hipError_t launch_bounds(const BoundsArgs &args, int32_t kind, int32_t n_peds, hipStream_t stream) {
    const int threads = 256;
    if (args.n <= 0) return hipSuccess;
    if (kind == HDX_PEDNAV)
        return n_peds <= 8    ? launch_bounds_ped<8>(args, stream)
               : n_peds <= 16 ? launch_bounds_ped<16>(args, stream)
                              : launch_bounds_ped<32>(args, stream);
    const dim3 grid((unsigned)((args.n + threads - 1) / threads)), block(threads);  // a lane per state
    if (kind == HDX_ROCKSAMPLE) {
        hipLaunchKernelGGL(bounds_rocks<RsOps>, grid, block, 0, stream, args);
    } else if (kind == HDX_MARS) {
        hipLaunchKernelGGL(bounds_rocks<MarsOps>, grid, block, 0, stream, args);
    } else {
        hipLaunchKernelGGL(bounds_nav, grid, block, 0, stream, args);
    }
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t *ctr, int64_t count, uint32_t k0, uint32_t k1, uint32_t *out,
                         hipStream_t stream) {
    const int threads = 256;
    const int64_t blocks = (count + threads - 1) / threads;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(philox_kernel, dim3((unsigned)blocks), dim3(threads), 0, stream, ctr, count, k0, k1, out);
    return hipGetLastError();
}

}  // namespace hdx
